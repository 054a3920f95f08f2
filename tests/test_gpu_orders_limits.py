"""Orders 1 and 4 at the limits of the strip kernels: more element rows than 65,535 (which the launch's
second grid dimension takes), and tangent coefficients that the device has no room for, where the
calls run on the element kernels, which need none.  Both are compared with those kernels (bounds: 1e-11 of
each block in FP64, 1e-5 in FP32 as in the other comparisons of the two; the same kernels 1e-13)."""
import pytest
import torch

import paper_2609_16424_amd as ilh
import seeded_inputs as si
from gpu_common import close, to_dev, to_np

pytestmark = pytest.mark.gpu


def _inputs(G, seed):
    u0 = to_np(G.init_state())
    h = 1.0 / (G.k * max(G.n))
    u = si.perturb_state(u0, seed, G.nh1, 0.05 * h, 0.05, 0.02)
    k = si.block_direction(seed + 1, G.nh1, G.nl2, 0.1 * h, 0.1, 0.1)
    dk = si.block_direction(seed + 2, G.nh1, G.nl2, h, 1.0, 1.0)
    return to_dev(u), to_dev(k), dk, 0.5 * G.dt_estimate(to_dev(u), 2.0)


def _calls(G, u, k, dk, tau):
    return [to_np(G.residual(k, u, tau)), to_np(G.jvp(k, u, tau, to_dev(dk), 64)),
            to_np(G.jvp(k, u, tau, to_dev(dk, torch.float32), 32))]


@pytest.mark.parametrize("k", [1, 4])
def test_more_element_rows_than_the_grid_takes(k):
    n = (2, 70000) if k == 1 else (1, 66000)
    G = ilh.Hydro("uniform", n, k, lo=(0.0, 0.0), hi=(1.0, n[1] / n[0]))
    args = _inputs(G, 3)
    got = _calls(G, *args)
    G.set_kernel_variant(1)
    for a, b, tol in zip(got, _calls(G, *args), (1e-11, 1e-11, 1e-5)):
        assert close(a, b, tol, G.nh1)


def _fill():
    """All but 1 to 1.5 GB of the device's memory."""
    held = []
    while True:
        free = torch.cuda.mem_get_info()[0] - (1 << 30)
        if free < (1 << 29):
            return held
        held.append(torch.empty(min(free, 16 << 30), dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("prec", [64, 32])
def test_no_room_for_the_coefficients(prec):
    n = (600, 500) if prec == 64 else (800, 700)  # 1.8 and 1.7 GB of them
    dt = torch.float64 if prec == 64 else torch.float32
    G = ilh.Hydro("tg2d", n, 4)
    u, k, dk, tau = _inputs(G, 5)
    dk = to_dev(dk, dt)
    torch.cuda.synchronize()
    held = []
    try:
        held = _fill()
        G.linearize(k, u, tau)
        got = [to_np(G.jvp_lin(dk, prec)), to_np(G.jvp_lin(2.0 * dk, prec)), to_np(G.jvp(k, u, tau, dk, prec))]
    finally:
        del held
        torch.cuda.empty_cache()
    G.set_kernel_variant(1)
    ref = to_np(G.jvp(k, u, tau, dk, prec))
    for g, f in zip(got, (1.0, 2.0, 1.0)):
        assert close(g, f * ref, 1e-13 if prec == 64 else 1e-6, G.nh1)


def test_implicit_step_with_no_room_for_the_coefficients():
    """The solver's own actions, preconditioner and linearisation ahead; its workspace is there before."""
    ref, out = [], []
    for full in (False, True):
        G = ilh.Hydro("tg2d", (600, 500), 4)
        opts = ilh.newton_options(tol=1e-8, jvp_prec=64, restart=4, gmres_maxit=40, max_newton=8)
        u = G.init_state()
        dt = 2.0 * G.dt_estimate(u, 0.5)
        if not full:
            G.set_kernel_variant(1)
        else:
            G.set_kernel_variant(1)  # allocates the solver's workspace, no coefficients
            G.implicit_step(u.clone(), dt, opts=opts)
            G.set_kernel_variant(0)
        torch.cuda.synchronize()
        held = []
        try:
            held = _fill() if full else []
            _, st = G.implicit_step(u, dt, opts=opts)
        finally:
            del held
            torch.cuda.empty_cache()
        (out if full else ref).append((to_np(u), st))
        del G
    assert out[0][1]["newton"] == ref[0][1]["newton"]
    assert close(out[0][0], ref[0][0], 1e-9)
