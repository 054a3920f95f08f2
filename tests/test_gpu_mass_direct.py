"""The direct velocity-mass solve (one density: banded products with the 1D inverse masses) behind
the explicit rate and the explicit step, against the oracle's sparse LU on small meshes and against
the library's conjugate gradients (mass_v_solve) on wider ones: one element, node counts below and
above a tile of 64 nodes and 32 rows and above the band's reach, every order, 2D and 3D, freed faces,
and a mesh of two densities, which the conjugate gradients keep.  Bounds: 1e-12 against the LU (FP64
rounding times a condition number of at most 16^3); 1e-10 against conjugate gradients stopped at a
residual of 1e-13 (times that condition number)."""
import numpy as np
import pytest
import torch

import paper_2609_16424_amd as ilh
import seeded_inputs as si
from gpu_common import rel, to_dev, to_np

pytestmark = pytest.mark.gpu


def _state(H, seed):
    u = to_np(H.init_state())
    h = 1.0 / (H.k * max(H.n))
    return si.perturb_state(u, seed, H.nh1, 0.02 * h, 0.3, 0.1)


@pytest.mark.parametrize("n,k,free", [((1, 1), 1, 0), ((1, 1), 4, 0), ((2, 3), 2, 0), ((7, 5), 3, 0b0110),
                                      ((40, 3), 1, 0b1111), ((2, 1, 3), 2, 0), ((3, 2, 2), 1, 0b100001),
                                      ((1, 2, 1), 3, 0)])
def test_rate_matches_sparse_lu(n, k, free):
    from oracle.hydro import Hydro as OHydro
    O = OHydro("uniform", n, k, free_faces=free)
    G = ilh.Hydro("uniform", n, k, free_faces=free)
    u = _state(G, 3)
    f = to_np(G.rate(to_dev(u)))
    fo = O.rate(u)
    for sl in (slice(0, G.nh1), slice(G.nh1, 2 * G.nh1), slice(2 * G.nh1, None)):
        scale = max(np.abs(fo[sl]).max(), 1e-3 * np.abs(fo).max())
        assert np.abs(f[sl] - fo[sl]).max() <= 1e-12 * scale


@pytest.mark.parametrize("problem,n,k", [("tg2d", (150, 3), 2), ("tg2d", (3, 97), 3), ("tg2d", (64, 64), 1),
                                         ("tg2d", (33, 70), 4), ("tg3d", (30, 4, 5), 2), ("tg3d", (2, 21, 35), 2),
                                         ("triple", (21, 9), 3)])
def test_rate_matches_conjugate_gradients(problem, n, k):
    G = ilh.Hydro(problem, n, k)
    u = to_dev(_state(G, 5))
    f = G.rate(u)[G.nh1:2 * G.nh1]
    b = G.residual(torch.zeros_like(u), u, 0.0)[G.nh1:2 * G.nh1].clone()
    x, it, res = G.mass_v_solve(b, rtol=1e-13)
    assert rel(to_np(f), -to_np(x)) <= 1e-10, (it, res)


def test_explicit_steps_repeat_after_each_other():
    """The step clears its residual rows for the next one: a step repeated from the same state gives
    the same result, also after a step of another state."""
    G = ilh.Hydro("tg2d", (9, 6), 3)
    a, b = to_dev(_state(G, 1)), to_dev(_state(G, 2))
    first = to_np(G.rk2avg_step(a.clone(), 1e-3))
    G.rk2avg_step(b.clone(), 1e-3)
    assert rel(to_np(G.rk2avg_step(a.clone(), 1e-3)), first) <= 1e-14
