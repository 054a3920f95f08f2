"""Rounding of the direct velocity-mass solve behind the explicit rate, against the same tensor product in
extended precision (1D masses assembled from the library's FP64 tables, dense inverses refined to 64 bits
of mantissa) for the force vector that the library itself returns.  The strips are one group of elements
wide, so that no node sum has more than two terms and the force is the same in both calls.

Bound, 3.0e-16 of the 2-norm: a CPU model of the products gives 1.5e-16 to 2.4e-16 where the tile's own
columns are added one multiply at a time with the rounding carried along (conjugate gradients stopped
at 1e-14: 1.7e-16 to 2.9e-16 on smooth fields, more on rough ones), and 3.0e-16 to 5.1e-16 for a plain
sum over the band on meshes of more than a few elements."""
import math

import numpy as np
import pytest
import torch

import paper_2609_16424_amd as ilh
import seeded_inputs as si
from gpu_common import to_dev, to_np

pytestmark = pytest.mark.gpu

LD = np.longdouble


def _legendre(n, x):
    p0, p1 = 1.0, x
    for k in range(2, n + 1):
        p0, p1 = p1, ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k
    return p1, n * (x * p1 - p0) / (x * x - 1.0)


def _newton(z, step):
    for _ in range(100):
        dz = step(z)
        z -= dz
        if abs(dz) < 1e-16:
            break
    return z


def _tables(k):
    """The Gauss weights and the basis values at the points in FP64, formed as the library forms them: the
    mass that it defines is that of its rounded tables."""
    n = 2 * k
    xq, wq = [0.0] * n, [0.0] * n
    for i in range(n):
        z = _newton(math.cos(math.pi * (i + 0.75) / (n + 0.5)), lambda z: _legendre(n, z)[0] / _legendre(n, z)[1])
        dp = _legendre(n, z)[1]
        xq[n - 1 - i], wq[n - 1 - i] = 0.5 * (z + 1.0), 1.0 / ((1.0 - z * z) * dp * dp)

    def second(z):
        p, dp = _legendre(k, z)
        return dp / ((2.0 * z * dp - k * (k + 1.0) * p) / (1.0 - z * z))

    xn = [0.0] + [0.5 * (_newton(-math.cos(math.pi * i / k), second) + 1.0) for i in range(1, k)] + [1.0]
    B = np.empty((n, k + 1))
    for q in range(n):
        for a in range(k + 1):
            num = den = 1.0
            for b in range(k + 1):
                if b != a:
                    num *= xq[q] - xn[b]
                    den *= xn[a] - xn[b]
            B[q, a] = num / den
    return np.array(wq).astype(LD), B.astype(LD)


def _mass(n, k):
    w, B = _tables(k)
    m = (B * w[:, None]).T @ B
    A = np.zeros((n * k + 1, n * k + 1), LD)
    for e in range(n):
        A[e * k:e * k + k + 1, e * k:e * k + k + 1] += m
    return A


def _inverse(A, held):
    A = A.copy()
    for i in ((0, -1) if held else ()):
        A[i, :] = A[:, i] = 0
        A[i, i] = 1
    X = np.linalg.inv(A.astype(float)).astype(LD)
    for _ in range(4):
        X = X + X @ (np.eye(len(A), dtype=LD) - A @ X)
    return X


@pytest.mark.parametrize("n,k", [((1, 2), 3), ((10, 40), 3), ((16, 30), 2), ((8, 25), 4), ((32, 60), 1),
                                 ((2, 90), 3), ((4, 30, 1), 2)])
@pytest.mark.parametrize("seed", [1, 2])
def test_rate_error(n, k, seed):
    G = ilh.Hydro("uniform", n, k)
    G.set_apply_rows(1)  # the strip kernels at every order
    d = len(n)
    u = to_np(G.init_state())
    u = to_dev(si.perturb_state(u, seed, G.nh1, 0.02 / (k * max(n)), 0.3, 0.1))
    b = to_np(G.residual(torch.zeros_like(u), u, 0.0))[G.nh1:2 * G.nh1]
    f = to_np(G.rate(u))[G.nh1:2 * G.nh1]
    N = G.nh1 // d
    shape = [m * k + 1 for m in reversed(n)]
    err = ref = 0.0
    for c in range(d):
        x = b[c * N:(c + 1) * N].astype(LD).reshape(shape)
        for ax in range(d):  # axis d - 1 - ax holds direction ax
            X = _inverse(_mass(n[ax], k), ax == c)
            x = np.moveaxis(np.tensordot(X, np.moveaxis(x, d - 1 - ax, 0), axes=(1, 0)), 0, d - 1 - ax)
        x /= LD(float(np.prod([1.0 / m for m in n])))  # |J0|, as the library rounds it
        g = f[c * N:(c + 1) * N].reshape(shape)
        ends = [slice(None)] * d
        for end in (0, -1):
            ends[d - 1 - c] = end
            x[tuple(ends)] = 0
        err += float(((g + x) ** 2).sum())
        ref += float((x ** 2).sum())
    assert ref > 0 and np.sqrt(err / ref) <= 3.0e-16
