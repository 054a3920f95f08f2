"""Krylov cycles around the largest basis the one-launch Gram-Schmidt step holds (22 vectors with one node
pair per thread, 16 with two of an FP64 basis): cycles that end in its closing step at 15, 16, 17, 22 and
23 columns, and cycles that go on with the three launches behind it.  As for the shorter cycles, the
forms add the same FP64 sums in another order: same Newton iterations, GMRES counts at most one apart
per iteration, trajectories equal to the Newton tolerance (1e-10 relative residual, 1e-9 of the state)."""
import pytest

import paper_2609_16424_amd as ilh
from gpu_common import rel, to_np

pytestmark = pytest.mark.gpu


def _run(n, k, kw, fac, wait):
    G = ilh.Hydro("tg2d", n, k)
    u = G.init_state()
    dt = fac * G.dt_estimate(u, 0.5)
    opts = ilh.newton_options(tol=1e-10, gmres_maxit=400, **kw)
    traj, stats, hist = [], [], []
    for _ in range(2):
        if wait is not None:
            G.set_step_wait(wait)
        kk, st = G.implicit_step(u, dt, guess=G.plain_guess(u, hist, 0.5 * dt), opts=opts)
        hist = (hist + [kk])[-2:]
        traj.append(to_np(u))
        stats.append(st)
    return traj, stats


@pytest.mark.parametrize("n,k,kw,fac", [
    ((9, 7), 2, dict(jvp_prec=64, gmres_rtol=1e-9, restart=15), 4.0),
    ((9, 7), 2, dict(jvp_prec=64, gmres_rtol=1e-9, restart=22), 8.0),
    ((9, 7), 2, dict(jvp_prec=64, gmres_rtol=1e-9, restart=23), 8.0),
    ((13, 6), 3, dict(jvp_prec=32, gmres_rtol=1e-5, restart=16), 8.0),
    ((13, 6), 3, dict(jvp_prec=64, gmres_rtol=1e-9, restart=64), 16.0),
    ((100, 70), 3, dict(jvp_prec=64, gmres_rtol=1e-9, restart=16), 4.0),
    ((100, 70), 3, dict(jvp_prec=64, gmres_rtol=1e-9, restart=17), 4.0),
    ((100, 70), 3, dict(jvp_prec=64, gmres_rtol=1e-9, restart=64), 8.0)])
def test_cycles_around_the_largest_basis(n, k, kw, fac):
    ref, sr = _run(n, k, kw, fac, -1.0)
    assert max(s["gmres"] / s["newton"] for s in sr) > 14  # long cycles are what runs
    for wait in (None, 0.0):
        tr, st = _run(n, k, kw, fac, wait)
        for a, b, x, y in zip(tr, ref, st, sr):
            assert x["newton"] == y["newton"], (wait, x, y)
            assert abs(x["gmres"] - y["gmres"]) <= x["newton"], (wait, x["gmres"], y["gmres"])
            assert rel(a, b) <= 1e-9, (wait, rel(a, b))
