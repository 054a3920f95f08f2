// Device pieces shared by the lagged Gram-Schmidt kernels: the three-launch form (ilh_ops.hip) and
// the one-launch step (ilh_gs.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "ilh_internal.h"

namespace ilh {

// The value of another lane whose bit MASK (below 16) differs, through the vector unit: lane ^ 8,
// lane ^ 7 for MASK 4, lane ^ 2, lane ^ 1.
template <int MASK>
__device__ __forceinline__ double lane_other(double v) {
  static_assert(MASK == 8 || MASK == 4 || MASK == 2 || MASK == 1, "within a row of 16 lanes");
  // row_ror:8, row_half_mirror, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
  constexpr int C = MASK == 8 ? 0x128 : MASK == 4 ? 0x141 : MASK == 2 ? 0x4E : 0xB1;
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), C, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), C, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// a of the lane pair (l, l ^ MASK) summed in the lane whose bit MASK is clear, b in the other one
// (MASK 32 or 16): the swap hands each lane exactly the operand it lacks.
template <int MASK>
__device__ __forceinline__ double swap_sum(double a, double b) {
  static_assert(MASK == 32 || MASK == 16, "halves of the wave or rows of 16 lanes");
  const unsigned al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
  unsigned xl, xh, yl, yh;
  if constexpr (MASK == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    xl = l[0], yl = l[1], xh = h[0], yh = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    xl = l[0], yl = l[1], xh = h[0], yh = h[1];
  }
  return __hiloint2double((int)xh, (int)xl) + __hiloint2double((int)yh, (int)yl);
}

// Sums of K values (K a power of two, at most 64) over the 64 lanes of a wave.  Each exchange
// pairs the lanes whose bit MASK differs and halves the values a lane holds (it keeps one half, adds
// the partner's copy of that half): K - 1 + (6 - log2 K) exchanges instead of 6 K.  Afterwards every
// lane holds in acc[0] the complete sum of the value index returned (the lanes that differ only
// in their low 6 - log2 K bits hold the same one).  The exchanges are register swaps and lane permutes
// of the vector unit: through LDS (34 permutes a set of 16) eight waves queued behind one another,
// 1.3 us of a 10.5 us step with 19 sums.
template <int CNT, int MASK, int K>
__device__ __forceinline__ void wave_sums_r(double (&acc)[K], int lane, int& v) {
  if constexpr (MASK >= 1) {
    const bool hi = (lane & MASK) != 0;
    if constexpr (CNT > 1) {
      constexpr int HALF = CNT / 2;
#pragma unroll
      for (int i = 0; i < HALF; ++i) {
        if constexpr (MASK >= 16) {
          acc[i] = swap_sum<MASK>(acc[i], acc[i + HALF]);
        } else {
          const double send = hi ? acc[i] : acc[i + HALF];
          const double keep = hi ? acc[i + HALF] : acc[i];
          acc[i] = keep + lane_other<MASK>(send);
        }
      }
      if (hi) v += HALF;
      wave_sums_r<HALF, MASK / 2, K>(acc, lane, v);
    } else {
      if constexpr (MASK >= 16)
        acc[0] = swap_sum<MASK>(acc[0], acc[0]);
      else
        acc[0] += lane_other<MASK>(acc[0]);
      wave_sums_r<1, MASK / 2, K>(acc, lane, v);
    }
  }
}

template <int K>
__device__ __forceinline__ int wave_sums(double (&acc)[K]) {
  static_assert(K >= 1 && K <= 64 && (K & (K - 1)) == 0, "K: a power of two up to 64");
  int v = 0;
  wave_sums_r<K, 32, K>(acc, (int)(threadIdx.x & 63), v);
  return v;
}

// A partial sum as it is stored (never GS_EMPTY, which is one NaN among many)
__device__ __forceinline__ unsigned long long gs_bits(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  return u == GS_EMPTY ? 0x7FF8000000000000ull : u;
}

// The residual estimate and h_{j+1,j} of column j to host memory (mapped, coherent) as two 16-byte
// records {estimate, tag} and {h_{j+1,j}, tag}: each record is one store, so the host never pairs
// a new tag with an old value whatever order the two stores become visible in
__device__ __forceinline__ void publish_estimate(double* hest, int j, double est, double hn, double tag) {
  double2* rec = reinterpret_cast<double2*>(hest + 4 * j);
  rec[0] = make_double2(est, tag);
  rec[1] = make_double2(hn, tag);
  __threadfence_system();
}

// one row of the update from its loaded u_j and w: v_j (stored back when j > 0) and u_{j+1}
// (scaled by sg, stored over w); returns the stored u_{j+1}
template <typename TV>
__device__ __forceinline__ double lgs_row(TV* uj, TV* w, int64_t row, bool in, int j, double uv, double wv, double A,
                                          double B, double rinv, double d, double sg) {
  const TV vj = j > 0 ? (TV)((uv - A) * rinv) : (TV)uv;
  const TV un = (TV)(sg * (wv - B - d * (double)vj));
  if (in) {
    if (j > 0) uj[row] = vj;
    w[row] = un;
  }
  return (double)un;
}

// The serial part of step j, one thread, every operand in LDS: with the sums S (S[2k] = v_k . u_j,
// S[2k + 1] = v_k . w, k < j; S[2j] = |u_j|^2, S[2j + 1] = u_j . w, S[2j + 2] = |w|^2) it finishes
// column j - 1 of the Hessenberg matrix (the previous step's first-pass coefficients pl, the
// rotations csl, snl of the earlier columns; coll is scratch), sets the cycle-end flag
// h[HDEV_LGSE] = j + 1 when that column met the target or rho_j = 0, and leaves the coefficients
// of the update and of step j + 1 in h.  sc: g_{j-1}, |r|, the target, the cycle's tag, 1 / s_j.
// publish: hand the estimate to the host from here.  has_w = false: the closing step.
__device__ __forceinline__ void lgs_column(const double* S, int j, int m, int has_w, const double* csl,
                                           const double* snl, double* coll, const double* pl, const double* sc,
                                           double* h, double* G, double* hest, bool publish) {
  double* cs = G + 64 * 64;
  double* g = cs + 128;
  double aa = 0.0, ab = 0.0;
  for (int k = 0; k < j; ++k) {
    aa += S[2 * k] * S[2 * k];
    ab += S[2 * k] * S[2 * k + 1];
  }
  double rho = 1.0, flag = 0.0;
  if (j > 0) {
    const double r2 = S[2 * j] - aa;
    rho = (r2 == r2) ? sqrt(fmax(r2, 0.0)) : r2;
    const double gs = sc[4];  // 1 / s_j
    for (int k = 0; k < j; ++k) coll[k] = pl[k] + S[2 * k] * gs;
    const double hn = rho * gs;
    // Givens update of column jc = j - 1 (as givens_col, every operand from LDS)
    const int jc = j - 1;
    double* Hm = G;
    double cur = coll[0];
    for (int i = 0; i < jc; ++i) {
      const double nx = coll[i + 1];
      Hm[i * 64 + jc] = csl[i] * cur + snl[i] * nx;
      cur = -snl[i] * cur + csl[i] * nx;
    }
    const double den = hypot(cur, hn);
    const double c_ = den > 0 ? cur / den : 1.0, s_ = den > 0 ? hn / den : 0.0;
    cs[jc] = c_;
    cs[64 + jc] = s_;
    Hm[jc * 64 + jc] = den;
    const double gj = jc == 0 ? sc[1] : sc[0];
    if (jc == 0)
      for (int i = 2; i <= m; ++i) g[i] = 0.0;
    g[jc] = c_ * gj;
    g[jc + 1] = -s_ * gj;
    const double est = fabs(s_ * gj);
    h[352 + 2 * jc] = est;
    h[353 + 2 * jc] = hn;
    flag = (est <= sc[2] || hn == 0.0) ? 1.0 : 0.0;
    if (hest && publish) publish_estimate(hest, jc, est, hn, sc[3]);
  }
  if (flag != 0.0) h[HDEV_LGSE] = j + 1;
  if (!has_w) return;
  const double rinv = (rho > 0.0 && rho <= 1.7e308) ? 1.0 / rho : 0.0;
  const double d = j > 0 ? (S[2 * j + 1] - ab) * rinv : S[1];
  double* p = h + HDEV_LGSP;
  for (int k = 0; k < j; ++k) {
    h[k] = S[2 * k];
    h[72 + k] = S[2 * k + 1];
    p[k] = S[2 * k + 1];
  }
  p[j] = d;
  const double wn = sqrt(fmax(S[2 * j + 2], 0.0));
  const bool ok = wn > 0.0 && wn <= 1.7e308;
  p[65] = ok ? wn : 1.0;
  h[144] = j > 0 ? rinv : 1.0;
  h[145] = d;
  h[146] = ok ? 1.0 / wn : 1.0;
}

}  // namespace ilh
