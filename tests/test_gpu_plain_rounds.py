"""Rounds run as plain kernels (batches of 2^23 vertices or more): the iterates under
a round limit, the last rounds of which apply nothing, and fields whose rounds
differ in kind within one batch."""
import numpy as np
import pytest

import oracle
import paper_2601_01787_amd as pmsz
from test_gpu_parity import dev, host, noise_case, random_case, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,dtype", [((33, 509, 511), np.float32), ((2051, 4101), np.float64)],
                         ids=["3d-f32", "2d-f64"])
@pytest.mark.parametrize("mode", ["halving", "targeted"])
@pytest.mark.parametrize("k", [0, 1, 2, 5])
def test_round_limit_gives_the_oracles_iterate(shape, dtype, mode, k):
    f, fhat, xi = random_case(shape, dtype, 31, xi=0.003)
    g_ref, st_ref = oracle.correct(f, fhat, xi, max_iters=k, mode=mode)
    g, st = pmsz.correct(dev(f), dev(fhat), xi, max_iters=k, mode=mode)
    assert st == {**st, **st_ref}
    assert same_bits(host(g), g_ref)


def test_fields_in_rounds_of_different_kinds():
    """A dense field (tile rounds), a nearly exact one (sparse rounds), one that
    needs no edit and one of the other dimension, together and alone."""
    cases = [random_case((2000, 3000), np.float32, 1, xi=0.05),
             random_case((60, 200, 250), np.float32, 2, xi=1e-4),
             random_case((300, 400), np.float32, 3, xi=0.01)]
    f = random_case((64, 65, 66), np.float32, 4)[0]
    cases.append((f, f.copy(), 0.01))
    fields = [(dev(f), dev(h), xi) for f, h, xi in cases]
    stats = pmsz.correct_batched(fields)
    for (f, h, xi), (_, g, _), st in zip(cases, fields, stats):
        g_ref, st_ref = oracle.correct(f, h, xi)
        assert st == {**st, **st_ref}
        assert same_bits(host(g), g_ref)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_round_handed_back_by_the_tail(dtype):
    """A small field whose target list overflows in the tail, beside a large one
    that needs no edit: the round handed back runs as a plain one, and every
    statistic is that of the field alone."""
    f, fhat, xi = noise_case(24, 0.2, 31)
    f = f.astype(dtype)
    lb, ub = oracle.bounds(f, xi)
    fhat = np.minimum(np.maximum(fhat.astype(dtype), lb), ub)
    still = random_case((2900, 2900), dtype, 5)[0]
    cases = [(still, still.copy(), 0.05), (f, fhat, xi)]
    fields = [(dev(a), dev(h), e) for a, h, e in cases]
    stats = pmsz.correct_batched(fields)
    tm, rounds = pmsz.last_timing(), pmsz.last_rounds()
    assert tm["handbacks"] > 0, tm
    for (a, h, e), (_, g, _), st in zip(cases, fields, stats):
        g_ref, st_ref = oracle.correct(a, h, e)
        assert st == {**st, **st_ref}
        assert same_bits(host(g), g_ref)
    assert sum(r["edits"] for r in rounds) == sum(st["steps_applied"] for st in stats)
