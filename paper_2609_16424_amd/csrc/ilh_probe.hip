// The diagonal blocks of the Jacobian that the probed preconditioner takes (eq. blockdiag_prec), in one
// pass over the stored tangent coefficients of a 2D mesh: the diagonal of the velocity block (with
// the position block eliminated: directions (ax e, e, 0), ax = tau; without: ax = 0) and every
// element's energy block.
//
// The tangent at a point is linear in the direction's gradients, so its action on the gradient g of one
// node's basis function, paired with g again, is a quadratic form: three numbers per point and
// component give every node's diagonal entry, and one number per point every entry of the energy
// block.  The same entries read off 2 (k + 1)^2 + k^2 coloured actions, each behind a kernel that forms its
// direction, took 440 us of the step on the 112 x 48 Q3Q2 triple point; the one pass takes 14 and a fill.
//
// Lane map as in the other 2D strip kernels: one wave = EPW elements of one element row, lane (z, qx) =
// quadrature column qx of element z.  Node entries are summed over the strip in LDS and take one
// atomic per node and strip (dv zero on entry); constrained rows of the Jacobian are the identity,
// their entry is set by the node's owner.  Energy blocks are element-owned.
#include <hip/hip_runtime.h>

#include "ilh_internal.h"
#include "ilh_lin.h"

namespace ilh {

template <int D1D, int Q1D, int VISC, int SRC>
__global__ void __launch_bounds__(64) k_probe2d(const KParams P, const Tab2<float, D1D, Q1D> tb,
                                                const float* __restrict__ qd, float ax, double* dv,
                                                double* __restrict__ einv) {
  constexpr int K = D1D - 1, L1D = K, NLD = L1D * L1D;
  constexpr int EPW = 64 / Q1D, NS = K * EPW + 1;
  constexpr int NQD = LinLayout<2, VISC, SRC>::NQD;
  constexpr int NT = L1D * (L1D + 1) / 2;     // pairs bl <= bm of energy rows
  constexpr int NP = 2 * 3 * D1D, NR = (NP > NT ? NP : NT) | 1;

  __shared__ double sP[64][NR];  // the lane's node sums (c, b, form), then its energy sums
  __shared__ double sB[3][Q1D][D1D];  // G G, G B, B B
  __shared__ double sL[Q1D][L1D];

  const int lane = threadIdx.x;
  const uint32_t tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int sx = tile % gridDim.x, ey = tile / gridDim.x, ex0 = sx * EPW;
  const int nx = P.n[0], E = min(EPW, nx - ex0), ns = K * E + 1;
  const uint32_t ng0 = P.ng[0], ng1 = P.ng[1], N = (uint32_t)P.N;
  const uint32_t ebase = (uint32_t)ey * nx + ex0;
  const int z0 = lane / Q1D, qx = lane - z0 * Q1D;
  const double rj = P.rj0[ebase + min(z0, E - 1)];
  for (int i = lane; i < Q1D * D1D; i += 64) {
    const double B = tb.B[i / D1D][i % D1D], G = tb.G[i / D1D][i % D1D];
    sB[0][i / D1D][i % D1D] = G * G;
    sB[1][i / D1D][i % D1D] = G * B;
    sB[2][i / D1D][i % D1D] = B * B;
  }
  for (int i = lane; i < Q1D * L1D; i += 64) sL[i / L1D][i % L1D] = tb.BL[i / L1D][i % L1D];

  double S[2][D1D][3] = {}, Q[NT] = {};
  const float* __restrict__ qb = qd + (int64_t)tile * (Q1D * NQD * 64);
#pragma unroll 1
  for (int qy = 0; qy < Q1D; ++qy) {
    const float* rb = sbase(qb + qy * (NQD * 64));
    float cf[NQD];
#pragma unroll
    for (int f = 0; f < NQD; ++f) cf[f] = ld32(rb, (uint32_t)(f * 64 + lane));
    const double mq = (double)tb.W[qx] * tb.W[qy] * rj;
    float ds;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      float t[2][2];  // t[d][e]: row c of dS, entry e, for a unit gradient along d of component c
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        float dJ[2][2] = {}, dG[2][2] = {}, dS[2][2];
        dJ[c][d] = ax;
        dG[c][d] = 1.f;
        lin_apply<2, float, VISC>(cf, dJ, dG, 0.f, dS, ds);
        t[d][0] = dS[c][0];
        t[d][1] = dS[c][1];
      }
      const double t00 = t[0][0], t01 = (double)t[0][1] + (double)t[1][0], t11 = t[1][1];
#pragma unroll
      for (int b = 0; b < D1D; ++b) {
        const double By = tb.B[qy][b], Gy = tb.G[qy][b];
        S[c][b][0] += t00 * (By * By);
        S[c][b][1] += t01 * (By * Gy);
        S[c][b][2] += t11 * (Gy * Gy) + mq * (By * By);
      }
    }
    const float zero[2][2] = {};
    float dS[2][2];
    lin_apply<2, float, VISC>(cf, zero, zero, 1.f, dS, ds);
    const double te = mq - (double)ds;
#pragma unroll
    for (int bl = 0; bl < L1D; ++bl)
#pragma unroll
      for (int bm = bl; bm < L1D; ++bm)
        Q[bl * L1D - bl * (bl - 1) / 2 + bm - bl] += te * ((double)tb.BL[qy][bl] * tb.BL[qy][bm]);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int b = 0; b < D1D; ++b)
#pragma unroll
      for (int f = 0; f < 3; ++f) sP[lane][(c * D1D + b) * 3 + f] = S[c][b][f];
  lds_barrier();
  const bool last_x = ex0 + E == nx, last_y = ey == P.n[1] - 1;
  for (int i = lane; i < 2 * D1D * NS; i += 64) {
    const int s = i % NS, t = i / NS, b = t % D1D, c = t / D1D;
    if (s >= ns) continue;
    const uint32_t I = K * ex0 + s, J = K * ey + b, g = c * N + J * ng0 + I;
    const uint32_t idx = c == 0 ? I : J, ngc = c == 0 ? ng0 : ng1;
    if (idx == 0 || idx == ngc - 1) {
      if ((s < K * E || last_x) && (b < K || last_y)) dv[g] = 1.0;
      continue;
    }
    const int zz = s / K, a = s - K * zz;
    double o = 0.0;
    auto add = [&](int ze, int an) {
#pragma unroll
      for (int q = 0; q < Q1D; ++q) {
        const double* p = &sP[ze * Q1D + q][(c * D1D + b) * 3];
        o += sB[0][q][an] * p[0] + sB[1][q][an] * p[1] + sB[2][q][an] * p[2];
      }
    };
    if (zz < E) add(zz, a);
    if (a == 0 && zz > 0) add(zz - 1, K);
    unsafeAtomicAdd(&dv[g], o);
  }
  lds_barrier();
#pragma unroll
  for (int i = 0; i < NT; ++i) sP[lane][i] = Q[i];
  lds_barrier();
  for (int i = lane; i < E * NLD * NLD; i += 64) {
    const int ze = i / (NLD * NLD), t = i - ze * (NLD * NLD), r = t / NLD, j = t - r * NLD;
    const int al = r % L1D, am = j % L1D, bl = min(r / L1D, j / L1D), bm = max(r / L1D, j / L1D);
    double o = 0.0;
#pragma unroll
    for (int q = 0; q < Q1D; ++q)
      o += sL[q][al] * sL[q][am] * sP[ze * Q1D + q][bl * L1D - bl * (bl - 1) / 2 + bm - bl];
    einv[(int64_t)(ebase + ze) * (NLD * NLD) + t] = o;
  }
}

template <int K, int VISC, int SRC>
static void probe_t(ilh_ctx* c, double ax) {
  constexpr int D1D = K + 1, Q1D = 2 * K, EPW = 64 / Q1D;
  Tab2<float, D1D, Q1D> tb;
  for (int q = 0; q < Q1D; ++q) {
    for (int d = 0; d < D1D; ++d) {
      tb.B[q][d] = (float)c->h_B[q * D1D + d];
      tb.G[q][d] = (float)c->h_G[q * D1D + d];
    }
    for (int d = 0; d < K; ++d) tb.BL[q][d] = (float)c->h_BL[q * K + d];
    tb.W[q] = (float)c->h_w1[q];
  }
  hipLaunchKernelGGL((k_probe2d<D1D, Q1D, VISC, SRC>), dim3((c->n[0] + EPW - 1) / EPW, c->n[1]), dim3(64), 0,
                     c->stream, c->kp, tb, (const float*)c->qd[0], (float)ax, c->pdv, c->peinv);
}

// c->pdv and c->peinv (the blocks themselves, not inverted) from the FP32 coefficients, which must be
// current; the 2D strip kernels' meshes only (lin2d_available).
int launch_probe2d(ilh_ctx* c, double ax) {
  if (!lin2d_available(c)) return ILH_EINVAL;
  if (!c->qd[0] || !c->qd_ok[0]) return fail(c, ILH_EINVAL, "diagonal blocks before the linearisation");
  int st = launch_fill(c, c->pdv, 0.0, c->nh1);
  if (st) return st;
  const int code = 4 * c->k + 2 * (c->kp.visc ? 1 : 0) + (c->kp.tg_source ? 1 : 0);
  switch (code) {
    case 4: probe_t<1, 0, 0>(c, ax); break;
    case 5: probe_t<1, 0, 1>(c, ax); break;
    case 6: probe_t<1, 1, 0>(c, ax); break;
    case 7: probe_t<1, 1, 1>(c, ax); break;
    case 8: probe_t<2, 0, 0>(c, ax); break;
    case 9: probe_t<2, 0, 1>(c, ax); break;
    case 10: probe_t<2, 1, 0>(c, ax); break;
    case 11: probe_t<2, 1, 1>(c, ax); break;
    case 12: probe_t<3, 0, 0>(c, ax); break;
    case 13: probe_t<3, 0, 1>(c, ax); break;
    case 14: probe_t<3, 1, 0>(c, ax); break;
    case 15: probe_t<3, 1, 1>(c, ax); break;
    case 16: probe_t<4, 0, 0>(c, ax); break;
    case 17: probe_t<4, 0, 1>(c, ax); break;
    case 18: probe_t<4, 1, 0>(c, ax); break;
    case 19: probe_t<4, 1, 1>(c, ax); break;
    default: return ILH_EINVAL;
  }
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}

}  // namespace ilh
