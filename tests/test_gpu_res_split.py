"""The 2D strip residual on both sides of the strip count (640) up to which two waves share a strip, with a
partly filled last strip, orders 1 to 3, with and without source, and the det J it hands to the line
search (a step), against the oracle (1e-12 of the largest entry, FP64 sums of some hundred terms)."""
import pytest

import paper_2609_16424_amd as ilh
from gpu_common import close, make_pair, random_dir, random_state, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prob,n,k,visc", [("tg2d", (13, 320), 3, None), ("tg2d", (13, 321), 3, None),
                                           ("triple", (13, 321), 3, "formula"), ("tg2d", (17, 320), 2, "formula"),
                                           ("tg2d", (17, 321), 2, None), ("tg2d", (33, 320), 1, None),
                                           ("tg2d", (33, 321), 1, "const")])
def test_residual_both_sides_of_the_split(prob, n, k, visc):
    O, G = make_pair(prob, n, k, visc)
    u = random_state(O, 81)
    kk = 0.1 * random_dir(O, 82)
    r = to_np(G.residual(to_dev(kk), to_dev(u), 1e-4))
    ref = O.residual(kk, u, 1e-4)
    assert close(r, ref, 1e-12), rel(r, ref)


@pytest.mark.parametrize("n", [(13, 50), (13, 330)])
def test_step_takes_the_same_trials(n):
    """Implicit steps with the det J of the strip residual on both sides: no halving, converged, and the
    same state to the Newton tolerance whichever residual kernel ran (the element kernels' run)."""
    out = []
    for variant in ("lin", "generic"):
        G = ilh.Hydro("tg2d", n, 2)
        G.set_kernel_variant(variant)
        u = G.init_state()
        dt = 2.0 * G.dt_estimate(u, 0.5)
        _, st = G.implicit_step(u, dt, guess=G.plain_guess(u, [], 0.5 * dt), opts=ilh.newton_options(tol=1e-10, jvp_prec=64))
        assert st["halvings"] == 0 and st["res_final"] <= 1e-10 * st["res0"]
        out.append(to_np(u))
    assert rel(out[0], out[1]) <= 1e-9
