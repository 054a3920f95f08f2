"""The sums of squares of a Newton iteration and of a restarted cycle on vectors of every length class: one
work-group, fewer than 256, more, and the most that a sum takes (1,024, each then walking several rounds and a
remainder).  The residual norms that a solve reports are compared with torch's norms of the same residuals
(1e-13: 64-bit sums in another order), and a step solved with two-column cycles, whose restart residuals
scale every cycle, with one solved in long cycles."""
import pytest
import torch

import paper_2609_16424_amd as ilh
from gpu_common import rel, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wait", [5000.0, -1.0])
@pytest.mark.parametrize("n", [(1, 1), (8, 8), (80, 80), (160, 150), (300, 301)])
def test_reported_norms(n, wait):
    G = ilh.Hydro("tg2d", n, 3)
    G.set_step_wait(wait)
    u = G.init_state()
    dt = 2.0 * G.dt_estimate(u, 0.5)
    g = G.plain_guess(u, [], 0.5 * dt)
    _, st = G.implicit_step(u.clone(), dt, guess=g, opts=ilh.newton_options(max_newton=0, guess_fallback=0),
                            raise_on_fail=False)
    for k, name in ((torch.zeros_like(u), "res0"), (g, "res_init")):
        ref = float(torch.linalg.norm(G.residual(k, u, 0.5 * dt)))
        assert abs(st[name] - ref) <= 1e-13 * ref + 1e-12 * st["res0"] * (name == "res_init"), (name, st[name], ref)


@pytest.mark.parametrize("prec", [32, 64])
def test_short_cycles_on_long_vectors(prec):
    out = []
    for m in (2, 20):
        G = ilh.Hydro("tg2d", (200, 171), 3)
        u = G.init_state()
        dt = 2.0 * G.dt_estimate(u, 0.5)
        G.implicit_step(u, dt, opts=ilh.newton_options(tol=1e-10, jvp_prec=prec, restart=m, gmres_maxit=400))
        out.append(to_np(u))
    assert rel(out[0], out[1]) <= 1e-9
