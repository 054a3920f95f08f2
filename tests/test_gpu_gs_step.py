"""The one-launch Gram-Schmidt step (its work-groups meet inside the launch) against the three
launches it replaces, and its fallback: a step whose wait is given up is repeated with the three
launches.  All three forms run the same scheme with the same FP64 sums in another order, so they
take the same Newton iterations, GMRES counts at most one apart per Newton iteration, and their
trajectories agree to the Newton tolerance.  The meshes put one to 242 work-groups into the meeting,
with partly filled groups, every element block size the preconditioner meets (4, 8, 9, 16, 27), one,
two (FP64 basis) and three (FP32 basis) node pairs per thread, cycles longer than the 14 basis
vectors the launch holds, and vectors too wide for it."""
import pytest
import torch

import paper_2609_16424_amd as ilh
from gpu_common import rel, to_np

pytestmark = pytest.mark.gpu

CASES = {
    "one_element": ("tg2d", (1, 1), 2, dict(jvp_prec=32), 1.0),
    "q2_f32": ("tg2d", (9, 7), 2, dict(jvp_prec=32), 2.0),
    "q3_f64": ("tg2d", (13, 6), 3, dict(jvp_prec=64), 2.0),
    "q4_basis64": ("tg2d", (6, 5), 4, dict(jvp_prec=32, basis64=1), 1.0),
    "q2_3d": ("tg3d", (5, 4, 3), 2, dict(jvp_prec=32), 2.0),
    "q3_3d_f64": ("tg3d", (2, 3, 2), 3, dict(jvp_prec=64), 1.0),
    "restart20": ("tg2d", (16, 12), 2, dict(jvp_prec=32, restart=20, gmres_maxit=400), 4.0),
    "restart3": ("tg2d", (16, 12), 3, dict(jvp_prec=32, restart=3, gmres_maxit=400), 2.0),
    "uncoupled_graphs": ("tg2d", (20, 12), 3, dict(jvp_prec=32, prec_coupled=0, graphs=1), 2.0),
    "two_pairs_f64": ("tg2d", (100, 70), 3, dict(jvp_prec=64), 2.0),
    "three_pairs_f32": ("tg2d", (128, 128), 3, dict(jvp_prec=32), 4.0),
    "too_wide": ("tg2d", (160, 130), 3, dict(jvp_prec=32), 2.0),
    "triple_probe": ("triple", (28, 12), 3, dict(jvp_prec=32, prec_probe=2, prec_lag=1), 2.0),
}


def _run(case, waits, nsteps=3):
    problem, n, k, kw, fac = CASES[case]
    if problem == "triple":
        from paper_2609_16424_amd import learned as L
        G = L.make_triple(n[0], n[1], k)
    else:
        G = ilh.Hydro(problem, n, k)
    u = G.init_state()
    dt = fac * G.dt_estimate(u, 0.5)
    opts = ilh.newton_options(tol=1e-10, **kw)
    hist, traj, stats = [], [], []
    for i in range(nsteps):
        if waits is not None:
            G.set_step_wait(waits)
        g = G.plain_guess(u, hist, 0.5 * dt)
        kk, st = G.implicit_step(u, dt, guess=g, opts=opts)
        hist = (hist + [kk])[-2:]
        traj.append(to_np(u))
        stats.append(st)
    return traj, stats


@pytest.mark.parametrize("case", list(CASES))
def test_one_launch_step_matches_three_launches(case):
    ref, sr = _run(case, -1.0)
    for waits in (None, 0.0):  # the default wait, and every step given up
        tr, st = _run(case, waits)
        for a, b, x, y in zip(tr, ref, st, sr):
            assert x["newton"] == y["newton"], (case, waits, x, y)
            assert abs(x["gmres"] - y["gmres"]) <= x["newton"], (case, waits, x["gmres"], y["gmres"])
            assert rel(a, b) <= 1e-9, (case, waits, rel(a, b))


def test_two_contexts_on_two_streams():
    """Two contexts whose steps overlap on two streams (from two threads): each work-group meeting
    may have to wait for the other context's launches; both finish with the single-stream result."""
    import threading
    ref, _ = _run("three_pairs_f32", -1.0, 2)
    out = [None, None]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            out[i] = _run("three_pairs_f32", None, 2)[0]

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for o in out:
        assert o is not None
        for a, b in zip(o, ref):
            assert rel(a, b) <= 1e-9


def test_step_wait_bounds():
    G = ilh.Hydro("tg2d", (2, 2), 2)
    for bad in (2e6, float("nan")):
        with pytest.raises(ilh.IlhError):
            G.set_step_wait(bad)
