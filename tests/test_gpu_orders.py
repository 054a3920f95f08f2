"""The strip kernels of orders 1 and 4 in 2D (residual, linearisation and Jacobian action), which ran
on the generic element kernels before: against the oracle's residual and complex-step action on
meshes of one element, one element less and more than a strip (8 elements at k = 4, 32 at k = 1),
with viscosity and with the Taylor-Green source, also walked several element rows to a wave and by two
waves a strip; implicit steps against the oracle's (1e-8 of the state at a Newton tolerance of 1e-10, as
at the other orders); and the action without allocations on a
mesh whose tangent coefficients its scratch does not hold.  Bounds: 1e-12 in FP64 and 1e-5 in FP32
(those of the other orders)."""
import pytest
import torch

import paper_2609_16424_amd as ilh
from gpu_common import close, make_pair, random_dir, random_state, rel, to_dev, to_np
import seeded_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("problem,n,k,visc,rows,waves",
                         [("tg2d", (1, 1), 4, None, 0, 0), ("tg2d", (7, 2), 4, None, 0, 0),
                          ("triple", (8, 3), 4, "formula", 0, 0), ("tg2d", (9, 1), 4, "const", 0, 0),
                          ("tg2d", (1, 1), 1, None, 0, 0), ("tg2d", (31, 2), 1, None, 0, 0),
                          ("triple", (32, 3), 1, "formula", 0, 0), ("tg2d", (33, 1), 1, "const", 0, 0),
                          ("tg2d", (10, 6), 4, None, 4, 1), ("triple", (9, 7), 4, "formula", 3, 2),
                          ("tg2d", (34, 5), 1, None, 2, 1), ("triple", (35, 9), 1, "formula", 8, 2)])
def test_residual_and_action_match_oracle(problem, n, k, visc, rows, waves):
    from oracle.krylov import jvp_cs
    O, G = make_pair(problem, n, k, visc, width=0.1)
    G.set_apply_rows(rows)
    G.set_apply_waves(waves)
    u, kk, dk = random_state(O, 1), 0.1 * random_dir(O, 2), random_dir(O, 3)
    tau = 0.01 / max(n)
    r = to_np(G.residual(to_dev(kk), to_dev(u), tau))
    assert close(r, O.residual(kk, u, tau), 1e-12, O.nh1)
    jo = jvp_cs(lambda q: O.residual(q, u, tau), kk, dk)
    assert close(to_np(G.jvp(to_dev(kk), to_dev(u), tau, to_dev(dk), 64)), jo, 1e-12, O.nh1)
    assert close(to_np(G.jvp(to_dev(kk), to_dev(u), tau, to_dev(dk, torch.float32), 32)), jo, 1e-5, O.nh1)


def _inputs(G, seed):
    h = 1.0 / (G.k * max(G.n))
    u = si.perturb_state(to_np(G.init_state()), seed, G.nh1, 0.03 * h, 0.3, 0.1)
    kk = si.block_direction(seed + 1, G.nh1, G.nl2, 0.1 * h, 0.1, 0.1)
    dk = si.block_direction(seed + 2, G.nh1, G.nl2, h, 1.0, 1.0)
    return to_dev(u), to_dev(kk), dk, 0.1 * h


@pytest.mark.parametrize("k,n", [(1, (9, 5)), (4, (3, 2))])
def test_implicit_steps_match_oracle(k, n):
    from oracle import krylov
    O, G = make_pair("tg2d", n, k)
    u0 = O.init_state()
    states, _, _ = krylov.run_midpoint(O, u0, 0.01, 3)
    u = to_dev(u0)
    hist = []
    for i in range(3):
        kk, st = G.implicit_step(u, 0.01, guess=G.plain_guess(u, hist), opts=ilh.newton_options(tol=1e-10))
        hist = (hist + [kk])[-2:]
        assert rel(to_np(u), states[i + 1]) <= 1e-8


def test_action_without_allocations_beyond_the_scratch():
    """226 x 210 Q4Q3: 292 MB of tangent coefficients in FP64 (the scratch holds 268 MB), accepted on the
    element kernels as before; the transpose action stays refused at this order."""
    G = ilh.Hydro("tg2d", (226, 210), 4)
    u, kk, dk, tau = _inputs(G, 11)
    d = to_dev(dk)
    got = to_np(G.jvp_noalloc(kk, u, tau, d, 64))
    assert close(got, to_np(G.jvp(kk, u, tau, d, 64)), 1e-12, G.nh1)
    with pytest.raises(ilh.IlhError):
        G.vjp(kk, u, tau, d, 64)
