// Linearised 3D Jacobian action of the stage residual (eq. pa_jac_action at a fixed Newton
// iterate): the 3D counterpart of ilh_jvplin2d.hip, with the stress-tangent coefficients of
// ilh_lin.h (20 values per point without viscosity, 29 with it; no TG source in 3D).
//
// Lane map (both kernels): one wave = EPW consecutive elements of one element row (fixed y and
// z index); lane (z, qy, qx) owns the quadrature column (qx, qy) of element z and walks its Q1D
// points in the third direction.  The wave's node strip (D1D z-layers x D1D y-rows x NS nodes
// per field) is gathered once into LDS; each lane forms the x and y contractions of every field
// for its column; the third direction is unrolled with the 1D tables in kernel arguments.  The
// outputs are summed over the strip's columns by lane permutes (node_sums3), one velocity component at
// a time, and take one atomic per node and strip.
//
// Stored data: field f of lane l at step qz of strip b sits at qd[((b Q1D + qz) NQD + f) 64 + l]
// (the NQD fields of one wave's step form one contiguous block).  Strips are dealt to the XCDs
// in contiguous bands (xcd_tile).
#include <hip/hip_runtime.h>

#include "ilh_internal.h"
#include "ilh_lin.h"
#include "ilh_pointwise.h"

namespace ilh {

// ---- linearisation: state w (FP64) -> stored coefficients (T) ----------------------------
template <int D1D, int Q1D, typename T, int VISC>
__global__ void __launch_bounds__(64) k_lin3d(const KParams P, const Tab2<double, D1D, Q1D> tb,
                                              const double* __restrict__ w, double tau, T* __restrict__ qd) {
  constexpr int K = D1D - 1, L1D = K, NLD = L1D * L1D * L1D;
  constexpr int LPE = Q1D * Q1D, EPW = 64 / LPE;
  constexpr int NS = K * EPW + 1;
  constexpr int NQD = LinLayout<3, VISC, 0>::NQD;
  constexpr int NPRE = 2 * 3 * 3;  // J^-1 and gv are not scaled by tau
  constexpr int NF = 6;            // x0 x1 x2 v0 v1 v2

  __shared__ double sS[NF][D1D][D1D][NS];
  __shared__ double sE[EPW * NLD];
  __shared__ double sBG[2][Q1D][D1D];
  __shared__ double sBL[Q1D][L1D];

  const int lane = threadIdx.x;
  const uint32_t tile = xcd_tile((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x,
                                 gridDim.x * gridDim.y * gridDim.z);
  const int ex0 = (tile % gridDim.x) * EPW, ey = (tile / gridDim.x) % gridDim.y, ez = tile / (gridDim.x * gridDim.y);
  const int nx = P.n[0], ny = P.n[1];
  const int E = min(EPW, nx - ex0);
  const int ns = K * E + 1;
  const uint32_t ng0 = P.ng[0], ng01 = ng0 * P.ng[1], N = (uint32_t)P.N, nh1 = 3 * N;
  const uint32_t ebase = ((uint32_t)ez * ny + ey) * nx + ex0;
  const uint32_t row0 = (uint32_t)(K * ez) * ng01 + (uint32_t)(K * ey) * ng0 + (uint32_t)(K * ex0);

  constexpr int NTS = NF * D1D * D1D * NS, RT = (NTS + 63) / 64;
  double tr[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    // branch-free: lanes past the strip re-read its last node
    const int i = lane + 64 * r, s = min(i % NS, ns - 1), t = min(i / NS, NF * D1D * D1D - 1), b = t % D1D,
              cz = (t / D1D) % D1D, f = t / (D1D * D1D);
    tr[r] = ld32(w, (f < 3 ? f * N : nh1 + (f - 3) * N) + row0 + cz * ng01 + b * ng0 + s);
  }
  constexpr int NLS = EPW * NLD, RL = (NLS + 63) / 64;
  double lr[RL];
#pragma unroll
  for (int r = 0; r < RL; ++r) lr[r] = ld32(w, 2 * nh1 + ebase * NLD + min(lane + 64 * r, E * NLD - 1));
  // the lanes past the strip repeat points of its last element: with every lane storing, the rows of
  // coefficients are whole cache lines
  const int z0 = lane / LPE, z = min(z0, E - 1), rr = lane - z0 * LPE, qy = rr / Q1D, qx = rr - qy * Q1D;
  const double gam = P.gamma[ebase + z], dJ0 = P.j0e[ebase + z], rj = P.rj0[ebase + z];
  for (int i = lane; i < Q1D * D1D; i += 64) {
    sBG[0][i / D1D][i % D1D] = tb.B[i / D1D][i % D1D];
    sBG[1][i / D1D][i % D1D] = tb.G[i / D1D][i % D1D];
  }
  for (int i = lane; i < Q1D * L1D; i += 64) sBL[i / L1D][i % L1D] = tb.BL[i / L1D][i % L1D];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int i = lane + 64 * r;
    if (i < NTS) (&sS[0][0][0][0])[i] = tr[r];
  }
#pragma unroll
  for (int r = 0; r < RL; ++r) {
    const int i = lane + 64 * r;
    if (i < NLS) sE[i] = lr[r];
  }
  lds_barrier();

  const int s0 = K * z;
  double Bx[D1D], Gx[D1D], By[D1D], Gy[D1D], BLx[L1D], BLy[L1D];
#pragma unroll
  for (int a = 0; a < D1D; ++a) {
    Bx[a] = sBG[0][qx][a];
    Gx[a] = sBG[1][qx][a];
    By[a] = sBG[0][qy][a];
    Gy[a] = sBG[1][qy][a];
  }
#pragma unroll
  for (int a = 0; a < L1D; ++a) {
    BLx[a] = sBL[qx][a];
    BLy[a] = sBL[qy][a];
  }
  // x-y contractions per z-layer: BB (values), GB (d/dx), BG (d/dy)
  double BB[NF][D1D], GB[NF][D1D], BG[NF][D1D];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int cz = 0; cz < D1D; ++cz) {
      double bb = 0, gb = 0, bg = 0;
#pragma unroll
      for (int b = 0; b < D1D; ++b) {
        double ab = 0, ag = 0;
#pragma unroll
        for (int a = 0; a < D1D; ++a) {
          const double xv = sS[f][cz][b][s0 + a];
          ab += Bx[a] * xv;
          ag += Gx[a] * xv;
        }
        bb += By[b] * ab;
        gb += By[b] * ag;
        bg += Gy[b] * ab;
      }
      BB[f][cz] = bb;
      GB[f][cz] = gb;
      BG[f][cz] = bg;
    }
  double EL[L1D];
#pragma unroll
  for (int cl = 0; cl < L1D; ++cl) {
    double acc = 0;
#pragma unroll
    for (int bl = 0; bl < L1D; ++bl)
#pragma unroll
      for (int al = 0; al < L1D; ++al) acc += BLy[bl] * BLx[al] * sE[z * NLD + al + L1D * (bl + L1D * cl)];
    EL[cl] = acc;
  }
  const double wxy = tb.W[qx] * tb.W[qy] * rj;
  const int64_t blk = tile;
#pragma unroll 1
  for (int qz = 0; qz < Q1D; ++qz) {
    double J[3][3], Gv[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      double j0 = 0, j1 = 0, j2 = 0, g0 = 0, g1 = 0, g2 = 0;
#pragma unroll
      for (int c = 0; c < D1D; ++c) {
        const double Bz = tb.B[qz][c], Gz = tb.G[qz][c];
        j0 += Bz * GB[r][c];
        j1 += Bz * BG[r][c];
        j2 += Gz * BB[r][c];
        g0 += Bz * GB[3 + r][c];
        g1 += Bz * BG[3 + r][c];
        g2 += Gz * BB[3 + r][c];
      }
      J[r][0] = j0;
      J[r][1] = j1;
      J[r][2] = j2;
      Gv[r][0] = g0;
      Gv[r][1] = g1;
      Gv[r][2] = g2;
    }
    double eq = 0;
#pragma unroll
    for (int cl = 0; cl < L1D; ++cl) eq += tb.BL[qz][cl] * EL[cl];
    const double mq = wxy * tb.W[qz];
    double cf[NQD];
    lin_coefs<3, VISC>(P, gam, mq, dJ0, J, Gv, eq, cf);
#pragma unroll
    for (int f = NPRE; f < NQD; ++f) cf[f] *= tau;
    T* q = qd + (blk * Q1D + qz) * (NQD * 64) + lane;
#pragma unroll
    for (int f = 0; f < NQD; ++f) q[f * 64] = T(cf[f]);
  }
}

// ---- apply: direction dk (T) -> J dk (T) --------------------------------------------------
// Bound by the coefficient stream (8 or 4 bytes x 20 or 29 a point) once enough wavefronts keep it
// full, which registers decide.  Two per SIMD in FP64 and four in FP32 fit because the position
// contractions (27 values a lane) wait in LDS, and because the
// next step's coefficients are asked for when the point's tangent is formed, into the registers it
// leaves.  57x44x39 Q2Q1 with viscosity, fill included: FP64 766 us with one wavefront per SIMD, which
// waited 70 % of its cycles, field-major rows and one atomic per node and element, 410 us with two,
// 373 us with the node sums in the vector unit (1.53 GB of coefficients: 320 us at the rate of a large
// copy); FP32 204 and 178 us (160); without viscosity 380 and 277, 161 and 134 us.  FP32 with the
// coefficients copied to LDS directly measured 218 us against 204, with two steps' coefficients and
// the contractions in registers at three wavefronts 183 against 178.
template <int D1D, int Q1D, typename T, int VISC>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4)))
k_jvp3d_q(const KParams P, const Tab2<T, D1D, Q1D> tb, const T* __restrict__ dk, const T* __restrict__ qd,
          double tau_, T* __restrict__ out) {
  constexpr int K = D1D - 1, L1D = K, NLD = L1D * L1D * L1D;
  constexpr int LPE = Q1D * Q1D, EPW = 64 / LPE;
  constexpr int NS = K * EPW + 1;
  constexpr int NQD = LinLayout<3, VISC, 0>::NQD;
  constexpr int NF = 6;                      // dkx0 dkx1 dkx2 dkv0 dkv1 dkv2

  __shared__ T sS[NF][D1D][D1D][NS];
  __shared__ T sE[EPW * NLD];
  constexpr int NPC = 9 * D1D;
  __shared__ T sU[64 * NPC];  // (lane, position contraction)
  __shared__ T sBG[2][Q1D][D1D];
  __shared__ T sBL[Q1D][L1D];

  const int lane = threadIdx.x;
  const uint32_t tile = xcd_tile((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x,
                                 gridDim.x * gridDim.y * gridDim.z);
  const int ex0 = (tile % gridDim.x) * EPW, ey = (tile / gridDim.x) % gridDim.y, ez = tile / (gridDim.x * gridDim.y);
  const int nx = P.n[0], ny = P.n[1];
  const int E = min(EPW, nx - ex0);
  const int ns = K * E + 1;
  const uint32_t ng0 = P.ng[0], ng1 = P.ng[1], ng2 = P.ng[2], ng01 = ng0 * ng1;
  const uint32_t N = (uint32_t)P.N, nh1 = 3 * N;
  const uint32_t ebase = ((uint32_t)ez * ny + ey) * nx + ex0;
  const uint32_t row0 = (uint32_t)(K * ez) * ng01 + (uint32_t)(K * ey) * ng0 + (uint32_t)(K * ex0);

  constexpr int NNE = 3 * D1D * D1D * NS, RG = (NNE + 63) / 64;  // node entries (c, cz, b, s)
  constexpr int NLS = EPW * NLD, RL = (NLS + 63) / 64;
  T gx[RG], gv[RG], lr[RL];
  // branch-free gathers: lanes past the strip re-read its last node (their LDS slots feed no
  // output), so every load is in flight before the first LDS store
#pragma unroll
  for (int q = 0; q < RG; ++q) {
    const int i = min(lane + 64 * q, NNE - 1), s = min(i % NS, ns - 1), t = i / NS, b = t % D1D,
              cz = (t / D1D) % D1D, c = t / (D1D * D1D);
    const uint32_t gi = c * N + row0 + (uint32_t)cz * ng01 + (uint32_t)b * ng0 + s;
    gx[q] = ld32(dk, gi);
    gv[q] = ld32(dk, nh1 + gi);
  }
#pragma unroll
  for (int r = 0; r < RL; ++r) lr[r] = ld32(dk, 2 * nh1 + ebase * NLD + min(lane + 64 * r, E * NLD - 1));
  const T* __restrict__ qb = sbase(qd + (int64_t)tile * (Q1D * NQD * 64));
  T cf[NQD];
  auto ldstep = [&](const int qz) {
    const T* rb = sbase(qb + qz * (NQD * 64));
#pragma unroll
    for (int f = 0; f < NQD; ++f) cf[f] = ld32(rb, (uint32_t)(f * 64 + lane));
  };
  ldstep(0);
  const int zl = lane / LPE;
  const double rj_l = P.rj0[ebase + (zl < E ? zl : 0)];
  for (int i = lane; i < Q1D * D1D; i += 64) {
    sBG[0][i / D1D][i % D1D] = tb.B[i / D1D][i % D1D];
    sBG[1][i / D1D][i % D1D] = tb.G[i / D1D][i % D1D];
  }
  for (int i = lane; i < Q1D * L1D; i += 64) sBL[i / L1D][i % L1D] = tb.BL[i / L1D][i % L1D];
  const T tau = T(tau_);
  const bool last_x = (ex0 + E == nx), last_y = (ey == ny - 1), last_z = (ez == P.n[2] - 1);
#pragma unroll
  for (int q = 0; q < RG; ++q) {
    const int i = lane + 64 * q;
    if (i >= NNE) continue;
    const int s = i % NS, t = i / NS, b = t % D1D, cz = (t / D1D) % D1D, c = t / (D1D * D1D);
    sS[c][cz][b][s] = gx[q];
    sS[3 + c][cz][b][s] = gv[q];
    // position rows (dk_x - tau dk_v) and constrained velocity rows (dk_v): the node's single owner
    if (s >= ns || !((s < K * E || last_x) && (b < K || last_y) && (cz < K || last_z))) continue;
    const uint32_t gi = c * N + row0 + (uint32_t)cz * ng01 + (uint32_t)b * ng0 + s;
    st32(out, gi, gx[q] - tau * gv[q]);
    const uint32_t I = K * ex0 + s, J = K * ey + b, Kz = K * ez + cz;
    const uint32_t idx = c == 0 ? I : (c == 1 ? J : Kz), ngc = c == 0 ? ng0 : (c == 1 ? ng1 : ng2);
    if (idx == 0 || idx == ngc - 1) st32(out, nh1 + gi, gv[q]);
  }
#pragma unroll
  for (int r = 0; r < RL; ++r) {
    const int i = lane + 64 * r;
    if (i < NLS) sE[i] = lr[r];
  }
  lds_barrier();

  const int z = lane / LPE, rr = lane - z * LPE, qy = rr / Q1D, qx = rr - qy * Q1D;
  T Bx[D1D], Gx[D1D], By[D1D], Gy[D1D], BLx[L1D], BLy[L1D];
#pragma unroll
  for (int a = 0; a < D1D; ++a) {
    Bx[a] = sBG[0][qx][a];
    Gx[a] = sBG[1][qx][a];
    By[a] = sBG[0][qy][a];
    Gy[a] = sBG[1][qy][a];
  }
#pragma unroll
  for (int a = 0; a < L1D; ++a) {
    BLx[a] = sBL[qx][a];
    BLy[a] = sBL[qy][a];
  }
  // per-lane sums over the column: Tx (coefficient of Gx By), Ty (Bx Gy), Tz (Bx By) per
  // velocity component and z-layer, TL per energy layer
  T Tx[3][D1D], Ty[3][D1D], Tz[3][D1D], TL[L1D];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < D1D; ++c) Tx[r][c] = Ty[r][c] = Tz[r][c] = T(0);
#pragma unroll
  for (int cl = 0; cl < L1D; ++cl) TL[cl] = T(0);
  {  // lanes past the strip walk along: their columns feed no output
    const int s0 = K * z;
    T BB[NF][D1D], GB[NF][D1D], BG[NF][D1D];  // (the velocity fields')
    T* const pc = sU + lane * NPC;
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int cz = 0; cz < D1D; ++cz) {
        T bb = 0, gb = 0, bg = 0;
#pragma unroll
        for (int b = 0; b < D1D; ++b) {
          T ab = 0, ag = 0;
#pragma unroll
          for (int a = 0; a < D1D; ++a) {
            const T xv = sS[f][cz][b][s0 + a];
            ab += Bx[a] * xv;
            ag += Gx[a] * xv;
          }
          bb += By[b] * ab;
          gb += By[b] * ag;
          bg += Gy[b] * ab;
        }
        if (f < 3) {
          pc[(f * D1D + cz) * 3] = gb;
          pc[(f * D1D + cz) * 3 + 1] = bg;
          pc[(f * D1D + cz) * 3 + 2] = bb;
        } else {
          BB[f][cz] = bb;
          GB[f][cz] = gb;
          BG[f][cz] = bg;
        }
      }

    T EL[L1D];
#pragma unroll
    for (int cl = 0; cl < L1D; ++cl) {
      T acc = 0;
#pragma unroll
      for (int bl = 0; bl < L1D; ++bl)
#pragma unroll
        for (int al = 0; al < L1D; ++al) acc += BLy[bl] * BLx[al] * sE[z * NLD + al + L1D * (bl + L1D * cl)];
      EL[cl] = acc;
    }
    const T wxy = tb.W[qx] * tb.W[qy] * T(rj_l);
    auto step = [&](const int qz) {
      // tau is folded into the coefficients: the contractions enter unscaled
      T dJ[3][3], dGv[3][3], dkv[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        T j0 = 0, j1 = 0, j2 = 0, g0 = 0, g1 = 0, g2 = 0, mv = 0;
#pragma unroll
        for (int c = 0; c < D1D; ++c) {
          const T Bz = tb.B[qz][c], Gz = tb.G[qz][c];
          j0 += Bz * pc[(r * D1D + c) * 3];
          j1 += Bz * pc[(r * D1D + c) * 3 + 1];
          j2 += Gz * pc[(r * D1D + c) * 3 + 2];
          g0 += Bz * GB[3 + r][c];
          g1 += Bz * BG[3 + r][c];
          g2 += Gz * BB[3 + r][c];
          mv += Bz * BB[3 + r][c];
        }
        dJ[r][0] = j0;
        dJ[r][1] = j1;
        dJ[r][2] = j2;
        dGv[r][0] = g0;
        dGv[r][1] = g1;
        dGv[r][2] = g2;
        dkv[r] = mv;
      }
      T dke = 0;
#pragma unroll
      for (int cl = 0; cl < L1D; ++cl) dke += tb.BL[qz][cl] * EL[cl];
      const T mq = wxy * tb.W[qz];
      T dS[3][3], ds;
      lin_apply<3, T, VISC>(cf, dJ, dGv, dke, dS, ds);
      // the point's results are formed before the next coefficients are asked for: both sets in
      // registers at once would not fit
      asm volatile(""
                   : "+v"(dS[0][0]), "+v"(dS[0][1]), "+v"(dS[0][2]), "+v"(dS[1][0]), "+v"(dS[1][1]),
                     "+v"(dS[1][2]), "+v"(dS[2][0]), "+v"(dS[2][1]), "+v"(dS[2][2]), "+v"(ds)
                   :
                   : "memory");
      if (qz + 1 < Q1D) ldstep(qz + 1);
      const T cl_ = mq * dke - ds;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const T mv = mq * dkv[r];
#pragma unroll
        for (int c = 0; c < D1D; ++c) {
          const T Bz = tb.B[qz][c], Gz = tb.G[qz][c];
          Tx[r][c] += Bz * dS[r][0];
          Ty[r][c] += Bz * dS[r][1];
          Tz[r][c] += Gz * dS[r][2] + Bz * mv;
        }
      }
#pragma unroll
      for (int cl = 0; cl < L1D; ++cl) TL[cl] += tb.BL[qz][cl] * cl_;
    };
#pragma unroll 1
    for (int qz = 0; qz < Q1D; ++qz) {
      asm volatile("" ::: "memory");  // the contractions in LDS are read again each step
      step(qz);
    }
  }
  // the lane's indices once more, from a value the compiler does not connect with the first: what the
  // gather and the column walk derived from them is not kept in registers up to here
  int ln = threadIdx.x;
  asm volatile("" : "+v"(ln));
  const int pz = ln / LPE, pr = ln - pz * LPE, py = pr / Q1D, px = pr - py * Q1D;
  // velocity rows: node sums (node_sums3), one atomic per node and strip (constrained rows were written
  // by their owner above)
  static_assert(D1D == 3 && Q1D == 4, "one row of 16 lanes per element");
#pragma unroll
  for (int a = 0; a < D1D; ++a) {  // reloaded: not kept live through the column loop
    Bx[a] = sBG[0][px][a];
    Gx[a] = sBG[1][px][a];
    By[a] = sBG[0][py][a];
    Gy[a] = sBG[1][py][a];
  }
  const uint32_t I = K * (ex0 + pz) + px, J = K * ey + py;
  const bool cI = I == 0 || I == ng0 - 1, cJ = J == 0 || J == ng1 - 1;
  const bool node = px < D1D && py < D1D && pz < E && !(px == K && pz + 1 < E);
  const uint32_t off = row0 + (uint32_t)(K * pz + px) + (uint32_t)py * ng0;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    T v[D1D];
    node_sums3<T>(Tx[r], Ty[r], Tz[r], Bx, Gx, By, Gy, px, py, 4 * (ln - (LPE - K)), px == 0 && pz > 0, v);
#pragma unroll
    for (int cz = 0; cz < D1D; ++cz) {
      const uint32_t Kz = K * ez + cz;
      const bool cons = r == 0 ? cI : (r == 1 ? cJ : Kz == 0 || Kz == ng2 - 1);
      if (node && !cons) atomic_add32(out, nh1 + r * N + cz * ng01 + off, v[cz]);
    }
  }
  // energy rows (element-owned)
  const T o = energy_sums3<T>(TL, sBL[px], sBL[py], px, py);
  if (py < 2 && pz < E) st32(out, 2 * nh1 + (ebase + pz) * NLD + (px & 1) + 2 * (py + 2 * (px >> 1)), o);
}

// ---- host side ---------------------------------------------------------------------------
template <typename T, int D1D, int Q1D>
static Tab2<T, D1D, Q1D> make_tab3(const ilh_ctx* c) {
  Tab2<T, D1D, Q1D> tb;
  for (int q = 0; q < Q1D; ++q) {
    for (int d = 0; d < D1D; ++d) {
      tb.B[q][d] = T(c->h_B[q * D1D + d]);
      tb.G[q][d] = T(c->h_G[q * D1D + d]);
    }
    for (int d = 0; d < D1D - 1; ++d) tb.BL[q][d] = T(c->h_BL[q * (D1D - 1) + d]);
    tb.W[q] = T(c->h_w1[q]);
  }
  return tb;
}

// 3D, Q2Q1 (4 elements per wave), no TG source; 32-bit element offsets into the block vectors
bool lin3d_available(const ilh_ctx* c) {
  return c->dim == 3 && c->k == 2 && !c->kp.tg_source && c->nblock < (int64_t(1) << 29) && !c->general;
}

static dim3 lin3d_grid(const ilh_ctx* c) {
  const int Q1D = 2 * c->k, EPW = 64 / (Q1D * Q1D);
  return dim3((c->n[0] + EPW - 1) / EPW, c->n[1], c->n[2]);
}

static int lin3d_nqd(const ilh_ctx* c) { return c->kp.visc ? LinLayout<3, 1, 0>::NQD : LinLayout<3, 0, 0>::NQD; }

static int64_t lin3d_stride(const ilh_ctx* c) {
  const dim3 g = lin3d_grid(c);
  return (int64_t)g.x * g.y * g.z * (2 * c->k) * 64;
}

template <typename T>
static int lin3d_t(ilh_ctx* c, T* qd) {
  if (c->kp.visc)
    klaunch(c, k_lin3d<3, 4, T, 1>, lin3d_grid(c), dim3(64), 0, c->kp, make_tab3<double, 3, 4>(c),
            (const double*)c->w64, c->lin_tau, qd);
  else
    klaunch(c, k_lin3d<3, 4, T, 0>, lin3d_grid(c), dim3(64), 0, c->kp, make_tab3<double, 3, 4>(c),
            (const double*)c->w64, c->lin_tau, qd);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}

template <typename T>
static int apply3d_t(ilh_ctx* c, const T* dk, const T* qd, T* out) {
  if (c->kp.visc)
    klaunch(c, k_jvp3d_q<3, 4, T, 1>, lin3d_grid(c), dim3(64), 0, c->kp, make_tab3<T, 3, 4>(c), dk, qd,
            c->lin_tau, out);
  else
    klaunch(c, k_jvp3d_q<3, 4, T, 0>, lin3d_grid(c), dim3(64), 0, c->kp, make_tab3<T, 3, 4>(c), dk, qd,
            c->lin_tau, out);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}

int launch_lin3d(ilh_ctx* c, int prec) {
  if (!lin3d_available(c)) return ILH_EINVAL;
  const int p = prec == 64 ? 1 : 0;
  const int64_t len = (int64_t)lin3d_nqd(c) * lin3d_stride(c) * (p ? 8 : 4);
  if (!c->qd[p]) ILH_HIP(c, hipMalloc(&c->qd[p], len));
  return p ? lin3d_t<double>(c, (double*)c->qd[p]) : lin3d_t<float>(c, (float*)c->qd[p]);
}

int64_t lin3d_coef_bytes(const ilh_ctx* c, int prec) {
  return (int64_t)lin3d_nqd(c) * lin3d_stride(c) * (prec == 64 ? 8 : 4);
}

int launch_jvp3d_q(ilh_ctx* c, int prec, const void* dk, void* out) {
  if (!lin3d_available(c)) return ILH_EINVAL;
  const int p = prec == 64 ? 1 : 0;
  if (!c->qd[p]) return fail(c, ILH_EINVAL, "linearised Jacobian action before its linearisation");
  return p ? apply3d_t<double>(c, (const double*)dk, (const double*)c->qd[p], (double*)out)
           : apply3d_t<float>(c, (const float*)dk, (const float*)c->qd[p], (float*)out);
}

}  // namespace ilh
