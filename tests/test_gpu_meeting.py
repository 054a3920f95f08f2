"""Which form the launches whose work-groups meet take, read from the context's counters: the one-launch
Arnoldi step is taken and not given up where the basis fits the chip, at every edge of the rule (one
element; two and three node pairs per thread; cycles longer than the launch holds; captured
steps), and not taken for vectors too wide for it; a given-up step costs its own linear solve
and then 1, 2, 4, ... later ones, after which the launch is tried again, and the caller's setting stays.
The residual norms likewise: one launch by default, two without a meeting where it is given up or not
wanted, with the same iterations and values."""
import pytest

import paper_2609_16424_amd as ilh
from gpu_common import rel, to_np
from test_gpu_gs_step import CASES

pytestmark = pytest.mark.gpu


def _steps(case, nsteps, wait=None):
    """(final state, linear solves, counters) of nsteps implicit steps without a guess."""
    problem, n, k, kw, fac = CASES[case]
    G = ilh.Hydro(problem, n, k)
    if wait is not None:
        G.set_step_wait(wait)
    u = G.init_state()
    dt = fac * G.dt_estimate(u, 0.5)
    solves = 0
    for _ in range(nsteps):
        solves += G.implicit_step(u, dt, opts=ilh.newton_options(tol=1e-10, **kw))[1]["newton"]
    return to_np(u), solves, G.meeting_counts()


@pytest.mark.parametrize("case", [c for c in CASES if c != "triple_probe"])
def test_one_launch_steps_are_taken(case):
    _, _, counts = _steps(case, 2)
    assert counts["cycles_given_up"] == 0
    assert (counts["steps"] > 0) == (case != "too_wide"), counts


def test_given_up_steps_pause_and_resume():
    ref, _, none = _steps("q2_f32", 8, -1.0)
    assert none["steps"] == 0 and none["cycles_given_up"] == 0
    u, solves, counts = _steps("q2_f32", 8, 0.0)
    assert rel(u, ref) <= 1e-9
    tries, nxt, pause = 0, 1, 1  # the 1st linear solve tries, then the 3rd, 6th, 11th, 20th, ...
    while nxt <= solves:
        tries, nxt, pause = tries + 1, nxt + 1 + pause, 2 * pause
    assert solves >= 8 and tries >= 3
    assert counts["cycles_given_up"] == tries, (solves, counts)


def test_setting_survives_a_given_up_step():
    """After the wait is allowed again the launch is taken again, without another give-up."""
    problem, n, k, kw, fac = CASES["q2_f32"]
    G = ilh.Hydro(problem, n, k)
    u = G.init_state()
    dt = fac * G.dt_estimate(u, 0.5)
    opts = ilh.newton_options(tol=1e-10, **kw)
    G.set_step_wait(0.0)
    G.implicit_step(u, dt, opts=opts)
    a = G.meeting_counts()
    assert a["cycles_given_up"] >= 1
    G.set_step_wait(5000.0)
    G.implicit_step(u, dt, opts=opts)
    b = G.meeting_counts()
    assert b["steps"] > a["steps"] and b["cycles_given_up"] == a["cycles_given_up"]


@pytest.mark.parametrize("case", ["one_element", "q2_f32", "q2_3d", "two_pairs_f64"])
def test_norms_are_formed_again_when_given_up(case):
    problem, n, k, kw, fac = CASES[case]
    runs = []
    for wait in (-1.0, 0.0, 5000.0):
        G = ilh.Hydro(problem, n, k)
        G.set_step_wait(wait)
        u = G.init_state()
        dt = fac * G.dt_estimate(u, 0.5)
        st = [G.implicit_step(u, dt, opts=ilh.newton_options(tol=1e-10, **kw))[1] for _ in range(2)]
        runs.append((to_np(u), st, G.meeting_counts()))
    (a, sa, ca), (b, sb, cb), (c, sc, cc) = runs
    assert ca["norms"] == 0 and ca["norms_given_up"] == 0
    assert cb["norms"] > 0 and cb["norms_given_up"] == cb["norms"]
    assert cc["norms"] == cb["norms"] and cc["norms_given_up"] == 0
    for x, y, z in zip(sa, sb, sc):
        assert x["newton"] == y["newton"] == z["newton"]
        # the first residuals are of the same states: the sums differ by rounding only
        assert abs(x["res_init"] - y["res_init"]) <= 1e-12 * x["res_init"]
    assert rel(b, a) <= 1e-9 and rel(c, a) <= 1e-9


def test_guess_norms_are_formed_again_when_given_up():
    from test_gpu_mlp_fused import _guess, _state
    outs = []
    for wait in (-1.0, 0.0, 5000.0):
        G = ilh.Hydro("tg2d", (13, 11), 3)
        G.set_step_wait(wait)
        u, _ = _state(G, 5)
        g, used = _guess(G, (128, 64), True, True, seed=7).guess(u, [0.5 * u], 0.01)
        outs.append((to_np(g), used, G.meeting_counts()))
    (a, na, ca), (b, nb, cb), (c, nc, cc) = outs
    assert ca["norms"] == 0 and cb["norms_given_up"] == cb["norms"] == cc["norms"] > 0 and cc["norms_given_up"] == 0
    assert na == nb == nc and (a == b).all() and (a == c).all()
