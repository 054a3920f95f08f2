"""The diagonal blocks formed in one pass over the 2D tangent coefficients against the oracle's dense
complex-step Jacobian, where strips are partly filled: one element more than a strip holds and a
single element, orders 1 to 4, with and without viscosity and source, several rows.

The coefficients and the point's tangent are FP32, at most some 16 roundings in a chain: velocity
diagonals to the 1e-5 of the FP32 actions, inverted blocks to 16 roundings times the block's condition
number where that is more."""
import numpy as np
import pytest

from gpu_common import close, make_pair, random_dir, random_state, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("prob,n,k,visc", [("tg2d", (33, 1), 1, "const"), ("triple", (17, 2), 2, None),
                                           ("tg2d", (11, 2), 3, "const"), ("triple", (3, 11), 3, "formula"),
                                           ("tg2d", (9, 1), 4, None), ("tg2d", (1, 1), 3, None)])
def test_blocks_of_partial_strips(prob, n, k, visc, mode):
    from oracle.krylov import dense_jacobian
    O, G = make_pair(prob, n, k, visc)
    u = random_state(O, 61)
    kk = 0.1 * random_dir(O, 62)
    tau = 0.004
    J = dense_jacobian(lambda q: O.residual(q, u, tau), kk)
    nh1, nl = O.nh1, k * k
    dv_ref = np.array([J[nh1 + i, nh1 + i] + (tau if mode == 1 else 0.0) * J[nh1 + i, i] for i in range(nh1)])
    blocks = [J[o:o + nl, o:o + nl] for o in range(2 * nh1, 2 * nh1 + O.nl2, nl)]
    einv_ref = np.stack([np.linalg.inv(b) for b in blocks])
    G.linearize(to_dev(kk), to_dev(u), tau)
    dv, einv = G.probe_blocks(mode)
    tol = max(1e-5, 16 * 2.0 ** -24 * max(np.linalg.cond(b) for b in blocks))
    assert close(to_np(dv), dv_ref, 1e-5), rel(to_np(dv), dv_ref)
    assert close(to_np(einv).ravel(), einv_ref.ravel(), tol), (rel(to_np(einv).ravel(), einv_ref.ravel()), tol)
