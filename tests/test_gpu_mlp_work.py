"""ilh_mlp_backward keeps its scratch in the caller's work array: networks whose data gradients fit it at
once and deeper ones that go through it two layers at a time, at batches around the 16-row tiles and
beyond the work-groups of a launch, against the oracle (bounds as in the other MLP tests: BF16 roundings
of a data gradient); nothing past 1,024 bytes a row is touched, at a work array four bytes past an
aligned address; a fresh context's call can be captured and replayed, and two calls of one context on two
streams, each with its own arrays, do not disturb one another."""
import ctypes as C

import pytest
import torch

from gpu_common import to_dev
from paper_2609_16424_amd import learned as L
from test_gpu_mlp import _gpu_mlp, _input, _params
from test_gpu_mlp_rows import test_forward_and_gradients_at_tile_edges as _against_oracle

pytestmark = pytest.mark.gpu

DEEP = [90] + [128] * 7 + [41]


@pytest.mark.parametrize("widths,B", [(DEEP, 1), (DEEP, 17), (DEEP, 300), (DEEP, 8230), ([90, 128, 128, 128, 128, 41], 31),
                                      ([90, 128, 128, 128, 41], 33), ([49, 128, 60], 16)])
def test_gradients(widths, B):
    _against_oracle(widths, B)


def _p(t):
    return C.c_void_p(t.data_ptr())


def _case(widths, B, seed):
    """(context, mlp, arguments of a call) with the forward done."""
    W, b = _params(widths, seed)
    G, m = _gpu_mlp(widths, W, b)
    x = to_dev(_input(B, widths[0], seed), torch.float32)
    t = torch.randn(B, L.pad32(widths[-1]), device="cuda", generator=torch.Generator("cuda").manual_seed(seed))
    zs, acts, _ = m.forward(x)
    return G, m, [x, zs, acts, t]


def _call(G, m, a, B, grad, work, loss=None):
    x, zs, acts, t = a
    G._stream()
    G._check(G.lib.ilh_mlp_backward(G.ctx, m.nl, m.cw, _p(m.WT), _p(x), _p(zs), _p(acts), _p(t), B, _p(grad),
                                    _p(grad[m.nW:]), _p(work), loss))


@pytest.mark.parametrize("widths,B", [(DEEP, 1), (DEEP, 17), (DEEP, 8230), ([90, 128, 128, 128, 41], 1),
                                      ([90, 128, 128, 128, 41], 33), ([20, 20], 1), ([20, 20], 16)])
def test_work_is_not_exceeded(widths, B):
    G, m, a = _case(widths, B, 3)
    ref, out = torch.zeros_like(m.grad), torch.zeros_like(m.grad)
    _call(G, m, a, B, ref, torch.zeros(2 * B * 128, device="cuda"))
    buf = torch.full((2 * B * 128 + 65,), 1.25, device="cuda")
    _call(G, m, a, B, out, buf[1:])
    torch.cuda.synchronize()
    assert float(buf[0]) == 1.25 and bool((buf[2 * B * 128 + 1:] == 1.25).all())
    n = m.nW
    assert torch.equal(out[n:], ref[n:])  # the bias gradients have one order of summation
    assert float((out[:n] - ref[:n]).norm()) <= 1e-5 * float(ref[:n].norm())


def test_first_call_can_be_captured():
    G, m, a = _case([90, 128, 128, 128, 41], 257, 4)
    work, grad = torch.empty(2 * 257 * 128, device="cuda"), torch.empty_like(m.grad)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _call(G, m, a, 257, grad, work)
    ref = torch.empty_like(grad)
    _call(G, m, a, 257, ref, torch.empty_like(work))
    for _ in range(3):
        grad.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(grad[m.nW:], ref[m.nW:])
        assert float((grad - ref).norm()) <= 1e-5 * float(ref.norm())


def test_calls_on_two_streams():
    B = 4096
    G, m, a = _case([90, 128, 128, 128, 41], B, 5)
    b = [a[0] * 0.5, a[1] * 0.5, a[2] * 0.5, a[3]]
    refs = []
    for args in (a, b):
        refs.append(torch.empty_like(m.grad))
        _call(G, m, args, B, refs[-1], torch.empty(2 * B * 128, device="cuda"))
    outs = [torch.empty_like(m.grad) for _ in range(2)]
    works = [torch.empty(2 * B * 128, device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(20):
        for s, args, o, w in zip(streams, (a, b), outs, works):
            with torch.cuda.stream(s):
                _call(G, m, args, B, o, w)
    torch.cuda.synchronize()
    G._stream()
    for o, r in zip(outs, refs):
        assert torch.equal(o[m.nW:], r[m.nW:])
        assert float((o - r).norm()) <= 1e-5 * float(r.norm())
