"""Order 4 in 2D around the sizes up to which single residuals and FP64 actions stay on the element
kernels (2,048 and 1,024 elements): both sides of each limit, and the strip kernels on small meshes
(one element, one less and one more than a strip of eight), which a set work split keeps, against the
oracle (1e-12, as at the other orders) and against the element kernels (1e-11 of each block: a
residual row of these states is a small difference of element terms)."""
import pytest
import torch

import paper_2609_16424_amd as ilh
from gpu_common import close, make_pair, random_dir, random_state, to_dev, to_np
from test_gpu_orders import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("problem,n,visc", [("tg2d", (1, 1), None), ("tg2d", (7, 2), None), ("triple", (8, 3), "formula"),
                                            ("tg2d", (9, 1), "const")])
@pytest.mark.parametrize("rows", [0, 1])
def test_small_meshes_match_oracle(problem, n, visc, rows):
    from oracle.krylov import jvp_cs
    O, G = make_pair(problem, n, 4, visc, width=0.1)
    G.set_apply_rows(rows)
    u, kk, dk = random_state(O, 1), 0.1 * random_dir(O, 2), random_dir(O, 3)
    tau = 0.01 / max(n)
    assert close(to_np(G.residual(to_dev(kk), to_dev(u), tau)), O.residual(kk, u, tau), 1e-12, O.nh1)
    jo = jvp_cs(lambda q: O.residual(q, u, tau), kk, dk)
    G.linearize(to_dev(kk), to_dev(u), tau)
    for _ in range(2):
        assert close(to_np(G.jvp_lin(to_dev(dk), 64)), jo, 1e-12, O.nh1)
        assert close(to_np(G.jvp_lin(to_dev(dk, torch.float32), 32)), jo, 1e-5, O.nh1)


@pytest.mark.parametrize("n", [(32, 32), (41, 25), (32, 64), (41, 50)])
def test_both_sides_of_the_limits(n):
    G = ilh.Hydro("tg2d", n, 4)
    u, kk, dk, tau = _inputs(G, 3)
    out = []
    for variant, rows in ((0, 0), (0, 1), (1, 0)):
        G.set_kernel_variant(variant)
        G.set_apply_rows(rows)
        out.append([to_np(G.residual(kk, u, tau)), to_np(G.jvp(kk, u, tau, to_dev(dk), 64))])
    for a in out[:2]:
        for x, y in zip(a, out[2]):
            assert close(x, y, 1e-11, G.nh1)
