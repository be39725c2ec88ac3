"""Tiles marched by single waves (directions, and the sweeps of batches of 2^23
vertices or more) against the oracle where the split can go wrong: tile widths,
heights and depths and their neighbours, grids thinner than a tile's halo, ties,
an odd number of planes, both edit rules, detection boxes of a decomposed
domain, and bounds missed in the last column, line or plane."""
import numpy as np
import pytest
import torch

import oracle
import paper_2601_01787_amd as pmsz
from oracle import multiblock as mb
from test_gpu_parity import dev, host, random_case, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [1, 2, 63, 64, 65, 129])
@pytest.mark.parametrize("ny,nz", [(1, 1), (2, 3), (3, 2), (4, 34), (5, 33), (9, 5), (16, 4)])
def test_directions_at_tile_edges_3d(nx, ny, nz):
    for dtype in (np.float32, np.float64):
        for ties in (False, True):
            h = random_case((nz, ny, nx), dtype, nx + 7 * ny + nz, ties=ties)[0]
            assert np.array_equal(host(pmsz.directions(dev(h))), oracle.directions(h))


@pytest.mark.parametrize("nx", [1, 2, 3, 255, 256, 257, 511, 515])
@pytest.mark.parametrize("ny", [1, 2, 3, 17, 34, 65])
def test_directions_at_tile_edges_2d(nx, ny):
    for dtype in (np.float32, np.float64):
        for ties in (False, True):
            h = random_case((ny, nx), dtype, nx + 7 * ny, ties=ties)[0]
            assert np.array_equal(host(pmsz.directions(dev(h))), oracle.directions(h))


@pytest.mark.parametrize("shape", [(33, 509, 511), (257, 2, 16385), (1, 4099, 2049),
                                   (2051, 4101), (8388609, 1)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("mode", ["halving", "targeted"])
def test_sweeps_match_oracle(shape, dtype, mode):
    f, fhat, xi = random_case(shape, dtype, 11, ties=mode == "targeted", xi=0.01)
    g_ref, st_ref = oracle.correct(f, fhat, xi, mode=mode)
    g, st = pmsz.correct(dev(f), dev(fhat), xi, mode=mode)
    assert pmsz.last_timing()["sweeps"] >= 2
    assert st == {**st, **st_ref}
    assert same_bits(host(g), g_ref)


def test_sweeps_with_detection_boxes_match_oracle():
    f, fhat, xi = random_case((41, 459, 467), np.float32, 5, xi=0.01)
    g_ref, st_ref = mb.correct_blocks(f, fhat, xi, (2, 3, 2))
    g, st = pmsz.correct_blocks(dev(f), dev(fhat), xi, (2, 3, 2))
    for k in ("status", "phases", "local_rounds", "lowered", "steps_applied"):
        assert st[k] == st_ref[k], k
    assert same_bits(host(g), g_ref)


@pytest.mark.parametrize("shape", [(33, 509, 511), (2051, 4101)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("bad", [np.nan, 2.0])
def test_sweeps_validate_every_vertex(shape, bad):
    f, fhat, xi = random_case(shape, np.float32, 3)
    ends = [(0,) * len(shape), tuple(n - 1 for n in shape),
            (32,) + tuple(n - 1 for n in shape[1:]), tuple(n // 2 for n in shape)]
    for at in ends:
        h = fhat.copy()
        h[at] = bad if np.isnan(bad) else f[at] + bad * xi
        g = dev(h)
        _, st = pmsz.correct(dev(f), g, xi, inplace=True)
        assert st["status"] == ("NONFINITE" if np.isnan(bad) else "INPUT_BOUND"), at
        assert same_bits(host(g), h)


def test_directions_of_the_longest_row():
    """1 x (2^31 - 1): the last tile's columns end one short of 2^31."""
    n = 2 ** 31 - 1
    h = torch.empty((1, n), device="cuda").uniform_(generator=torch.Generator("cuda").manual_seed(3))
    d = pmsz.directions(h).view(-1)
    h = h.view(-1)
    for at in [*range(0, n, 1 << 28), n - 1000]:
        a, b = max(at - 1, 0), min(at + (1 << 28) + 1, n)
        v = h[a:b]
        lo, hi = torch.full_like(v[:1], -torch.inf), torch.full_like(v[:1], torch.inf)
        left, right = v[:-1], v[1:]
        # (ties: the larger index is the higher)
        up_r, up_l = torch.cat([right, lo]), torch.cat([lo, left])
        mx = torch.where((up_r >= v) & (up_r >= up_l), 1, torch.where(up_l > v, 9, 0))
        dn_r, dn_l = torch.cat([right, hi]), torch.cat([hi, left])
        mn = torch.where((dn_l <= v) & (dn_l <= dn_r), 9, torch.where(dn_r < v, 1, 0))
        want = (mx | (mn << 4)).to(torch.uint8)
        i, j = (0 if a == 0 else 1), (len(v) if b == n else len(v) - 1)
        assert torch.equal(d[a + i:a + j], want[i:j]), at


def _merged_directions(h):
    """Direction bytes by the stencil's merges, every box reduced for its own vertex;
    neighbours outside the grid are NaN, as are some values."""
    d3 = h.ndim == 3
    p = np.pad(h if d3 else h[None], 1, constant_values=np.nan)
    nz, ny, nx = (h if d3 else h[None]).shape

    def at(m, sign, code):
        dx, dy, dz = sign * (m & 1), sign * ((m >> 1) & 1), sign * (m >> 2)
        v = p[1 + dz:1 + dz + nz, 1 + dy:1 + dy + ny, 1 + dx:1 + dx + nx]
        c = np.full(v.shape, code, np.uint8)
        return v, v, c, c

    def merge(a, b, hi, lo):  # hi, lo: where b is taken
        return (np.where(hi, b[0], a[0]), np.where(lo, b[1], a[1]), np.where(hi, b[2], a[2]),
                np.where(lo, b[3], a[3]))

    def up(a, b):
        return merge(a, b, b[0] >= a[0], b[1] < a[1])

    def down(a, b):
        return merge(a, b, ~(a[0] > b[0]), ~(a[1] <= b[1]))

    def box(sign, m, bits):  # the box of the offsets m | {0 .. bits}
        if bits == 0:
            return at(m, sign, (8 | m if m else 0) if sign < 0 else m)
        bit = 1 << (bits - 1)
        if sign > 0:
            return up(box(sign, m, bits - 1), box(sign, m | bit, bits - 1))
        return down(box(sign, m | bit, bits - 1), box(sign, m, bits - 1))

    with np.errstate(invalid="ignore"):
        e = up(box(-1, 0, 3 if d3 else 2), box(1, 0, 3 if d3 else 2))
    return (e[2] | (e[3] << 4)).reshape(h.shape)


@pytest.mark.parametrize("shape", [(35, 9, 130), (5, 17, 64), (2, 3, 65), (1, 1, 9), (70, 515),
                                   (33, 256), (3, 300), (1, 5)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_directions_beside_nan(shape, dtype):
    """One NaN (in a tile, on its edge or just outside), some, many, all: the bytes
    are those of the merges, and their pointers a forest that verify takes."""
    rng = np.random.default_rng(8)
    f = random_case(shape, dtype, 8, ties=len(shape) == 2)[0]
    assert np.array_equal(_merged_directions(f), oracle.directions(f))
    n = f.size
    spots = [rng.integers(n, size=1) for _ in range(12)] + [np.array([0]), np.array([n - 1])]
    spots += [rng.integers(n, size=k) for k in (1 + n // 200, 1 + n // 3)] + [np.arange(n)]
    if len(shape) == 3 and shape[0] > 32:  # around the first tile's far corner
        spots += [np.ravel_multi_index(at, shape) for at in
                  ((32, 4, 64), (32, 3, 63), (31, 4, 63), (31, 3, 64), (31, 3, 63))]
    for at in spots:
        g = f.copy()
        g.reshape(-1)[at] = np.nan
        assert np.array_equal(host(pmsz.directions(dev(g))), _merged_directions(g)), at
        rep = pmsz.verify(dev(f), dev(g), dev(f), 0.1)
        assert rep["bound_violations"] == np.isnan(g).sum() and rep["max_abs_err"] == np.inf
