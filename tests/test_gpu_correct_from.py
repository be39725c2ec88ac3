"""pmsz_correct_from: fhat in an array of its own, copied by the first sweep
(2^23 vertices or more) or with the workspace's clear (fewer; by 16 bytes or, at
odd sizes and addresses, by words)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2601_01787_amd as pmsz
from test_gpu_parity import dev, host, random_case, same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 7, 9), (16, 16, 64), (31, 33), (33, 509, 511), (2051, 4101)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_fhat_stays_and_g_is_its_own(shape, dtype):
    f, fhat, xi = random_case(shape, dtype, 21, xi=0.01)
    d_f, d_h = dev(f), dev(fhat)
    g, st = pmsz.correct(d_f, d_h, xi)
    same = d_h.clone()
    _, st2 = pmsz.correct(d_f, same, xi, inplace=True)
    assert st == st2 and same_bits(host(g), host(same)) and same_bits(host(d_h), fhat)
    # validation failures return a copy of fhat, its NaN's bits included
    bad = fhat.copy()
    bad.reshape(-1)[-1] = np.nan
    bad.view(np.uint32).reshape(-1)[-dtype().itemsize // 4] |= 5
    g, st = pmsz.correct(d_f, dev(bad), xi)
    assert st["status"] == "NONFINITE" and same_bits(host(g), bad)
    g, st = pmsz.correct(d_f, d_h, xi, max_iters=0)
    assert st["status"] == "NOT_CONVERGED" and same_bits(host(g), fhat)


def test_fields_at_odd_addresses():
    f, fhat, xi = random_case((9, 10, 32), np.float32, 2)
    g_ref, _ = oracle.correct(f, fhat, xi)
    buf = torch.empty(2 * f.size + 8, device="cuda")
    d_f, d_h = (buf[at:at + f.size].view(f.shape) for at in (1, f.size + 2))
    d_f.copy_(dev(f))
    d_h.copy_(dev(fhat))
    g, st = pmsz.correct(d_f, d_h, xi)
    assert st["status"] == "OK" and same_bits(host(g), g_ref)


def test_overlapping_arrays_are_refused():
    buf = torch.zeros(200, device="cuda")
    f = torch.zeros((10, 10), device="cuda")
    grid, st = pmsz.grid_of(f), pmsz.Stats()
    ws = pmsz.workspace(grid, pmsz.WS_CORRECT, f.device)

    def call(at):
        return pmsz.load().pmsz_correct_from(
            ctypes.byref(grid), ctypes.c_void_p(f.data_ptr()), ctypes.c_void_p(buf.data_ptr()),
            ctypes.c_void_p(buf[at:].data_ptr()), 0.1, None, 0, ctypes.c_void_p(ws.data_ptr()),
            ws.numel(), 10, ctypes.byref(st), None)

    assert call(1) == call(99) == 1
    assert call(0) == call(100) == 0


def test_g_over_f_is_refused_where_fhat_is_separate():
    buf = torch.zeros(300, device="cuda")
    f, fhat = buf[100:200].view(10, 10), torch.zeros((10, 10), device="cuda")
    grid, st = pmsz.grid_of(f), pmsz.Stats()
    ws = pmsz.workspace(grid, pmsz.WS_CORRECT, f.device)

    def call(at, h=fhat):
        p = [ctypes.c_void_p(t.data_ptr()) for t in (f, h, buf[at:], ws)]
        return pmsz.load().pmsz_correct_from(ctypes.byref(grid), *p[:3], 0.1, None, 0, p[3],
                                             ws.numel(), 10, ctypes.byref(st), None)

    assert [call(at) for at in (1, 100, 199)] == [1, 1, 1]
    assert [call(at) for at in (0, 200)] == [0, 0]
    assert call(100, f) == 0  # all three the same array, as in a call in place


def test_derived_tensors_keep_what_a_copy_carries():
    """g starts as a clone of fhat where that is more than a copy of its memory: a
    tangent, a pending negation, a zero without memory, a subclass with a clone of
    its own, a place in an autograd graph."""
    f, fhat, xi = random_case((6, 7, 8), np.float32, 11)
    g_ref, _ = oracle.correct(f, fhat, xi)
    d_f, d_h = dev(f), dev(fhat)
    tangent = torch.ones_like(d_h)
    with torch.autograd.forward_ad.dual_level():
        dual = torch.autograd.forward_ad.make_dual(d_h, tangent)
        g, _ = pmsz.correct(d_f, dual, xi)
        g, t = torch.autograd.forward_ad.unpack_dual(g)
        assert t is not None and torch.equal(t, tangent)
        assert same_bits(host(g), g_ref)
    neg = torch._neg_view(-d_h)
    assert neg.is_neg()
    g, st = pmsz.correct(d_f, neg, xi)
    assert st["status"] == "OK" and not g.is_neg() and same_bits(host(g), g_ref)
    zeros = torch._efficientzerotensor((6, 7, 8), device="cuda")
    g, st = pmsz.correct(torch.zeros((6, 7, 8), device="cuda"), zeros, xi)
    assert st["status"] == "OK" and not host(g).any()

    class Doubled(torch.Tensor):
        def clone(self):
            return self.as_subclass(torch.Tensor) * 2

    g, _ = pmsz.correct(d_f, (d_h / 2).as_subclass(Doubled), xi)
    assert same_bits(host(g), g_ref)
    g, _ = pmsz.correct(d_f, d_h.clone().requires_grad_(), xi)
    assert g.grad_fn is not None
    assert same_bits(host(g.detach()), g_ref)
