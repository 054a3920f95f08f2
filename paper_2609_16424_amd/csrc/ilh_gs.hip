// One launch for the Gram-Schmidt part of a lagged Arnoldi step: the dot sweep, the final block and
// the update sweep with the block preconditioner of ilh_ops.hip (scheme and formulas there), the
// work-groups meeting once inside the launch.
//
// What bounds it: three launches read the basis twice and pay three ramps and drains plus the final
// block's own round trip to memory.  Here every thread keeps its rows of V, u_j and w in registers
// from the products to the update, so the basis is read once, and the work-groups' partial sums
// cross the chip once.  Register rows per thread (2 NP) times 512 threads times one work-group per
// compute unit is the capacity; larger vectors take the three launches.
//
// Measured (rocprofv3, us per Arnoldi step; three launches -> one): 11.8 -> 5.0 to 7.6 on 8 x 8 Q2Q1
// (FP64 basis, 3 work-groups), 19.3 -> 9.2 on the 112 x 48 Q3Q2 triple point (240 groups).  Implicit
// steps: 1.09 -> 0.67 and 6.8 -> 5.2 ms; 128 x 128 Q3Q2 (243 groups) 0.480 -> 0.437 ms: there the
// launch, the loads and the 10 MB of stores remain.
//
// The meeting.  Each data work-group stores its partial sums with agent-scope atomic stores (they go
// past the XCD's L2) into words that hold GS_EMPTY until then; every group reads the words of all
// groups (agent-scope loads) until none is empty, and adds them in one fixed order, so that all hold
// the same bits.  No cache is written back or invalidated and nothing is counted: the data are their own
// arrival mark.  Arrivals counted in 16 words 256 bytes apart, behind a wait for the stores, took two
// round trips more (1.8 us of 11.8 a step on the triple point), with a single word 4 to 8 us more.  Steps alternate between two areas;
// each step empties the words that the next one fills, the cycle's start those of step 0.
//
// The wait ends whatever else runs on the device: a work-group that has waited for `limit` ticks of
// the 100 MHz clock marks the cycle as ended (every launch behind this one returns at once), tells the
// host and returns.  Other groups may have seen all sums and stored their rows: the host repeats the
// cycle, which forms every vector anew, with the three launches.  A residual estimate that the
// control group published is one of complete sums and holds in either case.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "ilh_internal.h"
#include "ilh_lgs.h"
#include "ilh_lin.h"

namespace ilh {

static constexpr int GS_T = 512;          // threads of a work-group
static constexpr int GS_MAXB = 256;       // work-groups: the control group and up to 255 data groups
static constexpr int GS_AREA = 64 * GS_MAXB;      // partial sums of one step
// Largest basis count: the rows of the vectors fit 256 registers (two wavefronts per SIMD)
template <typename TV, int NP>
constexpr int gs_max_j() {
  return NP == 1 ? 22 : sizeof(TV) == 8 ? 16 : 20;
}

// The cycle-end flag as the waves of a group read it: a group that gives a step up may set it while
// another still starts, so a group goes on only if none of its waves saw it.
__device__ __forceinline__ bool gs_ended(const double* endw) {
  bool e = false;
#pragma unroll
  for (int i = 0; i < GS_T / 64; ++i) e = e || endw[i] != 0.0;
  return e;
}

// Work-group 0 is the control group: it holds no rows, waits for the sums and runs the serial part
// (lgs_column).  Groups [1, 1 + nbx) hold NP node pairs (i, nh1 + i) per thread, the rest 2 NP sets of
// GS_T / Nl whole elements.  The update does not wait for the serial part: when column j - 1 ends
// the cycle, the vectors stored here are ones that the solution over j columns does not read.
// close: the closing step, which has no w (its sums are zero): it ends with the serial part.
template <typename TV, int J, int NP>
__global__ void __launch_bounds__(GS_T) k_lgs_step(TV* __restrict__ V, int64_t ldv, int m, double* h, double* G,
                                                   int64_t nh1, int64_t Ne, int Nl, int nbx, int nbd,
                                                   TV* __restrict__ z, float* __restrict__ z32,
                                                   TV* __restrict__ zero_v, const double* __restrict__ dv,
                                                   const double* __restrict__ me, int64_t estride,
                                                   const double* __restrict__ escale, int coupled,
                                                   unsigned long long* part, int never, uint64_t limit, double* hest,
                                                   int close) {
  constexpr int R = 2 * NP;
  constexpr int NA = 2 * J + 3;
  constexpr int NS = (NA + 15) / 16 * 16;  // sums, padded
  constexpr int NW = GS_T / 64;
  __shared__ double S[NS];
  __shared__ double sh[NW][NS];
  __shared__ double csl[64], snl[64], coll[65], pl[65], sc[6];
  __shared__ int late_s;
  __shared__ double endw[NW];
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const bool control = blockIdx.x == 0;
  unsigned long long* mine = part + (J & 1) * GS_AREA;         // this step's partial sums
  unsigned long long* next = part + ((J + 1) & 1) * GS_AREA;  // the next step's
  if (t == 0) late_s = 0;
  const int b = (int)blockIdx.x - 1;
  const bool h1 = b < nbx;
  TV* uj = V + (int64_t)J * ldv;
  TV* w = uj + ldv;
  uint32_t row[R];
  bool in[R];
  const int epb = GS_T / Nl, le = t / Nl, rr = t - le * Nl;  // (L2 groups)
  TV vr[J > 0 ? J : 1][R], ur[R], wr[R];
  double dd[R];  // dv of the node pairs, or the element scales
  const double ended = h[HDEV_LGSE];
  const double tau = h[250];
  if (!control) {
    if (h1) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int64_t i = ((int64_t)b * NP + q) * GS_T + t;
        in[2 * q] = in[2 * q + 1] = i < nh1;
        row[2 * q] = i < nh1 ? (uint32_t)i : 0u;
        row[2 * q + 1] = (uint32_t)nh1 + row[2 * q];
      }
    } else {
#pragma unroll
      for (int s = 0; s < R; ++s) {
        const int64_t e = ((int64_t)(b - nbx) * R + s) * epb + le;
        in[s] = le < epb && e < Ne;
        row[s] = (uint32_t)(2 * nh1 + (in[s] ? e * Nl + rr : 0));
      }
    }
    // 32-bit offsets from wave-uniform bases (n sizeof(TV) < 4 GiB: the capacity is far below), all
    // loads of the thread in flight before the first product
#pragma unroll
    for (int k = 0; k < J; ++k) {
      const TV* vk = sbase(V + (int64_t)k * ldv);
#pragma unroll
      for (int r = 0; r < R; ++r) vr[k][r] = ld32(vk, row[r]);
    }
    const TV* ub = sbase(uj);
    const TV* wb = sbase(w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ur[r] = ld32(ub, row[r]);
      wr[r] = close ? TV(0) : ld32(wb, row[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ur[r] = in[r] ? ur[r] : TV(0);
      wr[r] = in[r] ? wr[r] : TV(0);
    }
    // the sums q = 2k: v_k . u_j, 2k + 1: v_k . w, then |u_j|^2, u_j . w, |w|^2, reduced across the
    // wave 16 at a time (all of the up to 47 at once spilled the widest instances)
#pragma unroll
    for (int q0 = 0; q0 < NA; q0 += 16) {
      if (ended != 0.0) break;  // behind the loads: one round trip for both
      double acc[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[q] = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double u = (double)ur[r], x = (double)wr[r];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int s = q0 + q;
          if (s < 2 * J)
            acc[q] += (double)vr[s / 2][r] * (s % 2 == 0 ? u : x);
          else if (s < NA)
            acc[q] += (s == 2 * J + 2 ? x : u) * (s == 2 * J ? u : x);
        }
      }
      const int v = wave_sums<16>(acc);
      if ((lane & 3) == 0) sh[wid][q0 + v] = acc[0];
    }
    // (read in the update; requested here so that they arrive during the meeting)
    if (h1) {
#pragma unroll
      for (int q = 0; q < NP; ++q) dd[2 * q] = z ? dv[row[2 * q]] : 1.0;
    } else {
#pragma unroll
      for (int s = 0; s < R; ++s)
        dd[s] = (z && escale && in[s]) ? escale[(row[s] - (uint32_t)(2 * nh1)) / (uint32_t)Nl] : 1.0;
    }
    if (lane == 0) endw[wid] = ended;
    __syncthreads();
    if (gs_ended(endw)) return;
    if (t < NA) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < NW; ++i) s += sh[i][t];
      __hip_atomic_store(&mine[t * nbd + b], gs_bits(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (J < gs_max_j<TV, NP>() && t >= 64 && t < 64 + NA + 2)
      __hip_atomic_store(&next[(t - 64) * nbd + b], GS_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    // the operands of the serial part, staged while the data groups work
    const double* cs = G + 64 * 64;
    if (t < J - 1) {
      csl[t] = cs[t];
      snl[t] = cs[64 + t];
    }
    if (t >= 128 && t < 128 + J) pl[t - 128] = h[HDEV_LGSP + t - 128];
    if (t == 192) {
      sc[0] = J >= 1 ? cs[128 + (J >= 1 ? J - 1 : 0)] : 0.0;
      sc[1] = h[240];
      sc[2] = h[252];
      sc[3] = h[255];
      sc[4] = h[HDEV_LGSP + 65];
    }
    if (lane == 0) endw[wid] = ended;
    __syncthreads();
    if (gs_ended(endw)) return;
  }
#pragma unroll
  for (int s0 = 0; s0 < NA; s0 += GS_T / 16) {
    // 16 lanes per sum, 16 partials per lane (nbd <= 255), all loads of a round in flight together; a
    // wave asks again for the words that were empty
    const int s = s0 + (t >> 4), l16 = t & 15;
    const unsigned long long* p = mine + s * nbd;
    unsigned long long x[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = s < NA && l16 + 16 * q < nbd ? GS_EMPTY : 0ull;
    const uint64_t t0 = wall_clock64();
    bool late = false;
    while (!late) {
      bool wait = never && s < NA;
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (x[q] == GS_EMPTY) x[q] = __hip_atomic_load(&p[l16 + 16 * q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int q = 0; q < 16; ++q) wait = wait || x[q] == GS_EMPTY;
      if (__ballot(wait) == 0) break;
      late = wall_clock64() - t0 > limit;
    }
    if (late && lane == 0) {  // the step is given up: the cycle ends here, and the host repeats it
      late_s = 1;
      h[HDEV_LGSE] = -1.0;
      if (hest) {
        *reinterpret_cast<double2*>(hest + HEST_ABORT) = make_double2((double)J, h[255]);
        __threadfence_system();
      }
    }
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) a += __longlong_as_double((long long)x[q]);
    a += lane_other<8>(a);
    a += lane_other<4>(a);
    a += lane_other<2>(a);
    a += lane_other<1>(a);
    if (l16 == 0 && s < NA) S[s] = a;
  }
  __syncthreads();
  if (late_s) return;
  if (control) {
    if (t == 0) {
      lgs_column(S, J, m, close ? 0 : 1, csl, snl, coll, pl, sc, h, G, hest, false);
      if (J > 0 && hest) publish_estimate(hest, J - 1, h[352 + 2 * (J - 1)], h[353 + 2 * (J - 1)], sc[3]);
    }
    return;
  }
  if (close) return;
  // the update's coefficients, as lgs_column forms them
  double rinv = 1.0, d = S[2 * J + 1];
  if constexpr (J > 0) {
    double aa = 0.0, ab = 0.0;
#pragma unroll
    for (int k = 0; k < J; ++k) {
      aa += S[2 * k] * S[2 * k];
      ab += S[2 * k] * S[2 * k + 1];
    }
    const double r2 = S[2 * J] - aa;
    const double rho = (r2 == r2) ? sqrt(fmax(r2, 0.0)) : r2;
    rinv = (rho > 0.0 && rho <= 1.7e308) ? 1.0 / rho : 0.0;
    d = (S[2 * J + 1] - ab) * rinv;
  }
  const double wn = sqrt(fmax(S[2 * J + 2], 0.0));
  const double sg = (wn > 0.0 && wn <= 1.7e308) ? 1.0 / wn : 1.0;
  double un[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double A = 0.0, B = 0.0;
#pragma unroll
    for (int k = 0; k < J; ++k) {
      A += S[2 * k] * (double)vr[k][r];
      B += S[2 * k + 1] * (double)vr[k][r];
    }
    un[r] = lgs_row(uj, w, row[r], in[r], J, (double)ur[r], (double)wr[r], A, B, rinv, d, sg);
  }
  if (!z) return;
  if (h1) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      if (!in[2 * q]) continue;
      const uint32_t i = row[2 * q], iv = row[2 * q + 1];
      const double zv = un[2 * q + 1] / dd[2 * q];
      const double zx = coupled ? tau * zv + un[2 * q] : un[2 * q];
      z[i] = (TV)zx;
      z[iv] = (TV)zv;
      if (z32) {
        z32[i] = (float)zx;
        z32[iv] = (float)zv;
      }
      if (zero_v) zero_v[iv] = TV(0);
    }
  } else {
    __shared__ double shu[R][GS_T];
#pragma unroll
    for (int s = 0; s < R; ++s) shu[s][t] = un[s];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < R; ++s) {
      if (!in[s]) continue;
      const int64_t e = (int64_t)((row[s] - (uint32_t)(2 * nh1)) / (uint32_t)Nl);
      const double* Me = me + e * estride + (int64_t)rr * Nl;
      const double* ue = &shu[s][le * Nl];
      double a = 0.0;
      for (int l = 0; l < Nl; ++l) a += Me[l] * ue[l];
      a *= dd[s];
      z[row[s]] = (TV)a;
      if (z32) z32[row[s]] = (float)a;
    }
  }
}

// ---- host side ---------------------------------------------------------------------------
template <typename TV, int NP, int... I>
static auto gs_table(std::integer_sequence<int, I...>) {
  using F = decltype(&k_lgs_step<TV, 0, NP>);
  static const F t[] = {k_lgs_step<TV, I, NP>...};
  return t;
}
template <typename TV, int NP>
static auto gs_kernel(int j) {
  return gs_table<TV, NP>(std::make_integer_sequence<int, gs_max_j<TV, NP>() + 1>())[j];
}

// work-groups for NP node pairs per thread
static void gs_groups(const ilh_ctx* c, int np, int* nbx, int* nbe) {
  const int64_t pairs = (int64_t)GS_T * np, els = (int64_t)(GS_T / c->Nl) * 2 * np;
  *nbx = (int)std::min<int64_t>(1 << 20, (c->nh1 + pairs - 1) / pairs);
  *nbe = (int)std::min<int64_t>(1 << 20, (c->Ne + els - 1) / els);
}

// Node pairs per thread of the one-launch step (0: the three launches).  One pair per thread while
// the data groups fit one per compute unit beside the control group, else the largest count whose
// rows fit the registers (three pairs of an FP32 basis, two of FP64).  Wider vectors would need
// several work-groups per compute unit or spill.
int lgs_step_pairs(const ilh_ctx* c, bool f32) {
  if (c->gs_wait_us < 0.0 || c->Nl > 64 || c->gs_cus < 2) return 0;
  const int most = std::min(GS_MAXB, c->gs_cus) - 1;
  for (int np : {1, f32 ? 3 : 2}) {
    int nbx, nbe;
    gs_groups(c, np, &nbx, &nbe);
    if (nbx + nbe <= most) return np;
  }
  return 0;
}

// largest j of the one-launch step with np node pairs per thread
int lgs_step_max_j(int np, bool f32) {
  return f32 ? (np == 1 ? gs_max_j<float, 1>() : gs_max_j<float, 3>())
             : (np == 1 ? gs_max_j<double, 1>() : gs_max_j<double, 2>());
}

template <typename TV>
int lgs_step(ilh_ctx* c, int np, TV* V, int64_t ldv, int j, int m, double* h, double* G, TV* z, float* z32,
             TV* zero_v, int probe, int coupled, double* part, double* hest, bool close) {
  if (j < 0 || j > lgs_step_max_j(np, sizeof(TV) == 4)) return fail(c, ILH_EINVAL, "one-launch Arnoldi step: basis count out of range");
  int nbx, nbe;
  gs_groups(c, np, &nbx, &nbe);
  const double* dv = probe ? c->pdv : c->Mdiag;
  const double* me = probe ? c->peinv : c->MEinv;
  const int64_t estride = probe ? (int64_t)c->Nl * c->Nl : c->me_stride;
  const double* escale = probe ? nullptr : c->me_scale;
  const int never = c->gs_wait_us == 0.0 ? 1 : 0;  // a zero wait: the step is always given up
  const uint64_t limit = (uint64_t)(c->gs_wait_us * 100.0);
  auto f = np == 1 ? gs_kernel<TV, 1>(j) : gs_kernel<TV, sizeof(TV) == 4 ? 3 : 2>(j);
  hipLaunchKernelGGL(f, dim3(1 + nbx + nbe), dim3(GS_T), 0, c->stream, V, ldv, m, h, G, c->nh1, c->Ne, c->Nl, nbx,
                     nbx + nbe, z, z32, zero_v, dv, me, estride, escale, coupled,
                     reinterpret_cast<unsigned long long*>(part), never, limit, hest,
                     close ? 1 : 0);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}
template int lgs_step<double>(ilh_ctx*, int, double*, int64_t, int, int, double*, double*, double*, float*, double*,
                              int, int, double*, double*, bool);
template int lgs_step<float>(ilh_ctx*, int, float*, int64_t, int, int, double*, double*, float*, float*, float*, int,
                             int, double*, double*, bool);


// words (from the start of the partial sums) that the cycle's start sets to GS_EMPTY for step 0
int lgs_step_first(const ilh_ctx* c, int np) {
  int nbx, nbe;
  gs_groups(c, np, &nbx, &nbe);
  return 3 * (nbx + nbe);
}

}  // namespace ilh
