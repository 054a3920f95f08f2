"""Residual, Jacobian action and transpose action write every entry of their output, whatever it held:
buffers full of NaN give the results of zeroed ones.  The meshes put the velocity rows, which are zeroed
in 16-byte stores ahead of the kernels that add to them, at every alignment (N mod 4 = 0 to 3), and
take the strip kernels of all orders, the 3D ones and the element kernels.  The two runs differ by the
order of atomic adds only: 1e-12 in FP64, 1e-5 in FP32 (the tolerances of the actions against the
oracle)."""
import pytest
import torch

import paper_2609_16424_amd as ilh
from gpu_common import make_pair, random_dir, random_state, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prob,n,k", [("tg2d", (3, 2), 1), ("tg2d", (2, 2), 2), ("tg2d", (4, 3), 2), ("tg2d", (3, 2), 3),
                                      ("tg2d", (11, 1), 3), ("tg2d", (1, 2), 4), ("tg3d", (5, 2, 1), 2),
                                      ("tg3d", (2, 1, 1), 3)])
def test_outputs_need_no_clearing(prob, n, k):
    O, G = make_pair(prob, n, k)
    u, kk, d = to_dev(random_state(O, 71)), to_dev(0.1 * random_dir(O, 72)), to_dev(random_dir(O, 73))
    tau = 0.004
    calls = [(lambda out: G.residual(kk, u, tau, out=out), torch.float64)]
    G.linearize(kk, u, tau)
    for prec, dt in ((64, torch.float64), (32, torch.float32)):
        x = d.to(dt)
        calls.append((lambda out, x=x, prec=prec: G.jvp_lin(x, prec, out=out), dt))
        if (len(n) == 2 and k in (2, 3)) or (len(n) == 3 and k == 2):
            calls.append((lambda out, x=x, prec=prec: G.vjp_lin(x, prec, out=out), dt))
    for f, dt in calls:
        a = f(torch.zeros(G.nblock, dtype=dt, device="cuda"))
        b = f(torch.full((G.nblock,), float("nan"), dtype=dt, device="cuda"))
        c = f(None)
        for v in (b, c):
            assert torch.isfinite(v).all()
            assert rel(to_np(v), to_np(a)) <= (1e-12 if dt == torch.float64 else 1e-5)
