"""Labels by tiles (64 x 16 x 16 vertices, 64 x 256 in 2D) against the oracle's
walked labels where the split can go wrong: tile edges and remainders, paths
that cross one tile or many (longer than the walk over the direction bytes, so
the pointer-jumping passes run), one label array alone, and pointers that are
no forest inside one tile and through several."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2601_01787_amd as pmsz
from test_gpu_parity import dev, host, random_case

pytestmark = pytest.mark.gpu


def _check(h):
    d = pmsz.directions(dev(h))
    mx, mn = pmsz.labels(d)
    rmx, rmn = oracle.labels(oracle.directions(h))
    assert np.array_equal(host(mx), rmx) and np.array_equal(host(mn), rmn)
    return pmsz.last_labels()


@pytest.mark.parametrize("shape", [(16, 16, 64), (17, 17, 65), (15, 31, 63), (33, 16, 130),
                                   (2, 40, 257), (1, 1, 65), (256, 64), (257, 65), (255, 63),
                                   (600, 129), (1, 300), (300, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_tile_edges(shape):
    _check(random_case(shape, np.float32, 3)[0])
    info = _check(random_case(shape, np.float32, 4, ties=True)[0])
    assert info["passes_max"] >= 1 and info["passes_min"] >= 1


def test_paths_through_many_tiles():
    """Ramps and a snake: integral lines of up to about 700 and 5000 steps."""
    z, y, x = np.meshgrid(np.arange(40), np.arange(50), np.arange(700), indexing="ij")
    info = _check((x + 1e-3 * y + 1e-6 * z).astype(np.float64))
    assert info["passes_max"] > 1 and info["passes_min"] > 1
    _check((z + 1e-3 * x - 1e-6 * y).astype(np.float64))
    h = np.full((40, 400), -1.0)
    step = 0
    for row in range(0, 40, 3):  # a ridge that winds through the grid
        cols = range(400) if row % 2 == 0 else range(399, -1, -1)
        for c in cols:
            step += 1
            h[row, c] = step
        for r in (row + 1, row + 2):
            if r < 40:
                step += 1
                h[r, cols[-1]] = step
    info = _check(h)
    assert info["passes_max"] > 1


def test_one_label_array_alone():
    f = random_case((20, 30, 100), np.float32, 9)[0]
    d = pmsz.directions(dev(f))
    rmx, rmn = oracle.labels(oracle.directions(f))
    lib, grid = pmsz.load(), pmsz.grid_of(d)
    ws = pmsz.workspace(grid, pmsz.WS_LABELS, d.device)
    out = torch.empty(d.shape, dtype=torch.int32, device="cuda")
    for k, ref in enumerate((rmx, rmn)):
        a = [None, None]
        a[k] = ctypes.c_void_p(out.data_ptr())

        def call(dd):
            return lib.pmsz_labels(ctypes.byref(grid), ctypes.c_void_p(dd.data_ptr()), *a,
                                   ctypes.c_void_p(ws.data_ptr()), ws.numel(), None)

        assert call(d) == 0
        assert np.array_equal(host(out), ref)
        bad = d.clone()
        bad[5, 5, 5] = 0x80 if k == 0 else 0x08  # the other label's nibble
        assert call(bad) == 1
        assert pmsz.last_labels()["passes_min" if k == 0 else "passes_max"] == 0


@pytest.mark.parametrize("ring", ["pair_across_x", "loop_in_a_tile", "loop_across_tiles",
                                  "pair_across_y", "pair_across_z"])
def test_cycles_are_refused(ring):
    nz, ny, nx = 20, 20, 80
    f = random_case((nz, ny, nx), np.float32, 6)[0]
    d = pmsz.directions(dev(f))
    if ring.startswith("pair"):
        at, code = {"x": ((3, 3, 63), 1), "y": ((3, 15, 9), 2), "z": ((15, 3, 9), 4)}[ring[-1]]
        to = tuple(a + ((code >> (2 - k)) & 1) for k, a in enumerate(at))
        d[at] = (d[at] & 0xF0) | code
        d[to] = (d[to] & 0xF0) | code | 8
    else:
        x0, x1 = (5, 50) if ring == "loop_in_a_tile" else (50, 75)
        for x in range(x0, x1):  # a rectangle, two rows high
            d[2, 4, x] = (d[2, 4, x] & 0xF0) | 1
            d[2, 5, x + 1] = (d[2, 5, x + 1] & 0xF0) | 9
        d[2, 4, x1] = (d[2, 4, x1] & 0xF0) | 2
        d[2, 5, x0] = (d[2, 5, x0] & 0xF0) | 10
    with pytest.raises(pmsz.PmszError) as e:
        pmsz.labels(d)
    assert e.value.status == 1


@pytest.mark.parametrize("shape", [(1, 1), (1, 1023), (1, 1024), (5, 205), (70, 90, 100)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_verify_counts_at_block_edges(shape, dtype):
    """Blocks of 1024 vertices, with remainders and more than one per block."""
    f, fhat, xi = random_case(shape, dtype, 12)
    g = fhat.copy()
    g.reshape(-1)[-1] = f.reshape(-1)[-1] + dtype(3 * xi)  # the last vertex: out of bound
    rep = pmsz.verify(dev(f), dev(g), dev(fhat), xi)
    assert rep == oracle.verify(f, g, fhat, xi)
    assert rep["bound_violations"] == 1


@pytest.mark.parametrize("shape", [(33, 33, 129), (18, 40, 200), (16, 16, 16), (15, 16, 16), (8, 50, 128),
                                   (3000, 16), (3000, 15), (64, 900), (63, 900), (2, 2, 5000),
                                   (5000, 3, 3)], ids=lambda s: "x".join(map(str, s)))
def test_both_sides_of_the_thin_rule(shape):
    """Grids that fill a quarter of their tiles or more, and less."""
    _check(random_case(shape, np.float32, 3)[0])
    _check(random_case(shape, np.float32, 4, ties=True)[0])
    ramp = np.arange(np.prod(shape), dtype=np.float64).reshape(shape)  # paths of full length
    info = _check(ramp)
    assert info["passes_max"] > 1 or max(shape) <= 64


@pytest.mark.parametrize("shape", [(28, 28, 100), (9, 9, 100)], ids=["tiles", "thin"])
@pytest.mark.parametrize("ring", ["pair", "loop_in_a_tile", "loop_across_tiles"])
def test_cycles_on_both_sides_of_the_thin_rule(shape, ring):
    d = pmsz.directions(dev(random_case(shape, np.float32, 6)[0]))
    x0, x1 = {"pair": (63, 64), "loop_in_a_tile": (5, 50), "loop_across_tiles": (50, 75)}[ring]
    for x in range(x0, x1):
        d[2, 4, x] = (d[2, 4, x] & 0xF0) | 1
        d[2, 4 if ring == "pair" else 5, x + 1] = (d[2, 4 if ring == "pair" else 5, x + 1] & 0xF0) | 9
    if ring != "pair":
        d[2, 4, x1] = (d[2, 4, x1] & 0xF0) | 2
        d[2, 5, x0] = (d[2, 5, x0] & 0xF0) | 10
    with pytest.raises(pmsz.PmszError) as e:
        pmsz.labels(d)
    assert e.value.status == 1


@pytest.mark.parametrize("shape", [(28, 28, 100), (9, 9, 100)], ids=["tiles", "thin"])
def test_invalid_bytes_are_counted_once(shape):
    d = pmsz.directions(dev(random_case(shape, np.float32, 6)[0]))
    d[3, 3, 3] = 0x88  # both codes
    d[3, 4, 70] = 0x08
    with pytest.raises(pmsz.PmszError, match=r"\b2 direction bytes"):
        pmsz.labels(d)


def test_thin_grid_of_more_tiles_than_a_launch_holds():
    """1 x 1 x (2^26 + 1): more than 2^22 tiles of 1024 threads each."""
    h = np.random.default_rng(5).random((2 ** 26 + 1, 1, 1), np.float32)
    _check(h)
