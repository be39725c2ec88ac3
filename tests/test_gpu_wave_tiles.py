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
