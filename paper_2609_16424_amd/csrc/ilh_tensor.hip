// Direct velocity-mass solve on an affine initial mesh with one density.
//
// With rho0 |J0| the same in every element, M_V is (rho0 |J0|) times the tensor product of the 1D mass
// matrices of the directions, and the eliminated operator Mhat = P_u M_V P_u + P_c keeps that form per
// component: component c is held on wall faces normal to direction c, whole lines of its nodes, so
// the 1D matrix of direction c loses those end rows and the others none.  Its inverse is the tensor
// product of the 1D inverses.  A 1D inverse is dense, but its entries fall off exponentially (the 1D
// condition number is 4 to 16): beyond 29 to 68 nodes (k = 1 to 4) they are below 1e-17 of the largest,
// less than the rounding of the result.  So the solve is one banded product along each direction, where
// conjugate gradients took some 20 iterations of nine launches.
//
// Rounding.  A plain sum over the band rounds some 60 times next to its largest terms (4e-16 to 5e-16 of
// the solution, twice what conjugate gradients leave).  So the columns left and right of a tile's
// own ones are summed from the ends of the band inwards, each of the four or five multiplies over its own
// columns starts from zero, and those sums are added with their rounding errors carried along.
//
// The product along a direction is a band matrix times the matrix of all lines, so it runs on the FP64
// matrix instructions: a wave makes a tile of 16 nodes by 16 lines from (16 + 2 bw) / 4 multiplies of
// 16x16x4, its weights packed in the operand's lane order.  What bounds it: on small meshes the
// launches and the round trips to memory (the operands of TM_U multiplies are in flight together;
// a first form with one lane per node, weights and lines through the caches and LDS, took 13 us a pass at
// 49 x 49 nodes against 5 and 8 now), on large ones the multiplies, about 2 (16 + 2 bw) flop per node and
// direction against 16 bytes moved.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "ilh_internal.h"

namespace ilh {

static constexpr int TM_W = 4;   // waves per work-group
static constexpr int TM_U = 24;  // multiplies whose operands are in flight together (half from each end): 16 x 16 Q3Q2
                                 // steps 68.5 us with 24, 72.2 with 16, 73.1 with 32; 96 x 90 133, 126 and 130
static constexpr int TM_M = 5;   // multiplies that hold a column of the tile's own rows: 4, or 5 where the
                                 // band starts between two multiples of 4

// The 1D inverse mass matrix on the n k + 1 nodes of a direction as rows of 2 bw + 1 band entries (row
// i, offset o: column i + o - bw); with lo / hi, the end node is held (its row and column zero).
// Banded Cholesky (half bandwidth k) in extended precision, and the entries kept so, for weights that are
// rounded once; the rows of the inverse from the last one up, over a window wide enough that what it
// leaves out is below 1e-25, the middle rows repeated.  (The low end is not the mirror of the high one:
// the rounded quadrature points are not symmetric, which put 4e-16 into the solution at k = 4.)
static std::vector<long double> inverse_band(const ilh_ctx* c, int n, bool lo, bool hi, int* bw_out) {
  const int k = c->k, n1 = n * k + 1, D1D = k + 1, Q1D = 2 * k;
  std::vector<long double> m(D1D * D1D, 0.0L), A((size_t)n1 * D1D, 0.0L);  // A[i][k + j - i], j <= i
  for (int a = 0; a < D1D; ++a)
    for (int b = 0; b < D1D; ++b)
      for (int q = 0; q < Q1D; ++q) m[a * D1D + b] += (long double)c->h_w1[q] * c->h_B[q * D1D + a] * c->h_B[q * D1D + b];
  for (int e = 0; e < n; ++e)
    for (int a = 0; a < D1D; ++a)
      for (int b = 0; b <= a; ++b) A[(size_t)(e * k + a) * D1D + k + b - a] += m[a * D1D + b];
  auto hold = [&](int i) {
    for (int o = 0; o < k; ++o) A[(size_t)i * D1D + o] = 0.0;
    A[(size_t)i * D1D + k] = 1.0;
    for (int j = i + 1; j <= std::min(n1 - 1, i + k); ++j) A[(size_t)j * D1D + k + i - j] = 0.0;
  };
  if (lo) hold(0);
  if (hi) hold(n1 - 1);
  for (int i = 0; i < n1; ++i)  // A = L L^T in place
    for (int j = std::max(0, i - k); j <= i; ++j) {
      long double s = A[(size_t)i * D1D + k + j - i];
      for (int p = std::max(0, i - k); p < j; ++p)
        if (j - p <= k) s -= A[(size_t)i * D1D + k + p - i] * A[(size_t)j * D1D + k + p - j];
      A[(size_t)i * D1D + k + j - i] = j == i ? std::sqrt(s) : s / A[(size_t)j * D1D + k];
    }
  // Rows of the inverse Z from the last one up, right of the diagonal (it is symmetric): with A = L L^T,
  // L_ii Z_ij = [i = j] / L_ii - sum_{i < p <= i + k} L_pi Z_pj.  U[i][d] = Z_{i, i + d}.
  const int win = 100, far = win;  // beyond `far` from both ends the rows repeat with the elements' period k
  std::vector<long double> U((size_t)n1 * (win + 1), 0.0L);
  long double top = 0.0L;
  for (int i = n1 - 1; i >= 0; --i) {
    long double* u = &U[(size_t)i * (win + 1)];
    if (i >= far && i <= n1 - 1 - far - k) {
      std::copy(u + (size_t)k * (win + 1), u + (size_t)(k + 1) * (win + 1), u);
      continue;
    }
    const int m = std::min(win, n1 - 1 - i), np = std::min(k, n1 - 1 - i);
    const long double r = 1.0L / A[(size_t)i * D1D + k];
    for (int q = 1; q <= np; ++q) {
      const long double l = A[(size_t)(i + q) * D1D + k - q];
      const long double* z = u + (size_t)q * (win + 1);  // row i + q
      for (int d = q; d <= m; ++d) u[d] -= l * z[d - q];
      for (int d = 1; d < q; ++d) u[d] -= l * U[(size_t)(i + d) * (win + 1) + q - d];
    }
    for (int d = 1; d <= m; ++d) u[d] *= r;
    long double s = r;
    for (int q = 1; q <= np; ++q) s -= A[(size_t)(i + q) * D1D + k - q] * u[q];
    u[0] = (lo && i == 0) || (hi && i == n1 - 1) ? 0.0L : s * r;
    for (int d = 0; d <= m; ++d) top = std::max(top, std::fabs(u[d]));
  }
  int bw = 0;
  for (int i = 0; i < n1; ++i)
    for (int d = win; d > bw; --d)
      if (std::fabs(U[(size_t)i * (win + 1) + d]) > 1e-18L * top) bw = d;
  std::vector<long double> W((size_t)n1 * (2 * bw + 1), 0.0L);
  for (int i = 0; i < n1; ++i)
    for (int d = 0; d <= std::min(bw, n1 - 1 - i); ++d)
      W[(size_t)i * (2 * bw + 1) + bw + d] = W[(size_t)(i + d) * (2 * bw + 1) + bw - d] = U[(size_t)i * (win + 1) + d];
  *bw_out = bw;
  return W;
}

// (the extent keeps the weights' set-up small and the grids within their limits)
bool tensor_mass_available(const ilh_ctx* c) {
  if (!(c->rj0_one > 0.0)) return false;
  for (int d = 0; d < c->dim; ++d)
    if (c->ng[d] > 16384) return false;
  return c->dim == 2 || (int64_t)((c->ng[1] + 15) / 16) * c->ng[2] <= 65535;
}

// The weights on the device, on first use: per direction, without and with held ends, row tile by row
// tile in the order of the multiplies' first operand: lane l of multiply t of tile i0 / 16 holds row
// i0 + l mod 16, column i0 - bw + 4 t + l / 16 (zero outside the band and the matrix).
// 1 / (rho0 |J0|) is folded into direction 0.
static int tensor_setup(ilh_ctx* c) {
  if (c->tm_ok) return ILH_OK;
  struct Inv {
    int n, ends, bw;
    std::vector<long double> w;
  };
  std::vector<Inv> invs;  // directions of one extent and the same held ends share theirs
  std::vector<double> P;  // all weights: one allocation and one copy (each of them costs tenths of a millisecond)
  size_t at_d[3][2] = {};
  for (int d = 0; d < c->dim; ++d)
    for (int held = 0; held < 2; ++held) {
      const int ends = held ? (c->kp.walls >> (2 * d)) & 3 : 0;
      const long double scale = d == 0 ? 1.0L / c->rj0_one : 1.0L;
      size_t at = 0;
      while (at < invs.size() && (invs[at].n != c->n[d] || invs[at].ends != ends)) ++at;
      if (at == invs.size()) {
        Inv v{c->n[d], ends, 0, {}};
        v.w = inverse_band(c, c->n[d], (ends & 1) != 0, (ends & 2) != 0, &v.bw);
        invs.push_back(std::move(v));
      }
      const std::vector<long double>& Wl = invs[at].w;
      std::vector<double> W(Wl.size());  // the weights: scaled, then rounded once
      for (size_t i = 0; i < W.size(); ++i) W[i] = (double)(scale * Wl[i]);
      const int bw = invs[at].bw;
      const int n1 = c->ng[d], nb = 2 * bw + 1, tiles = (n1 + 15) / 16, nt = (16 + 2 * bw + 3) / 4;
      const size_t p0 = P.size();
      at_d[d][held] = p0;
      P.resize(p0 + (size_t)tiles * nt * 64, 0.0);
      for (int i = 0; i < n1; ++i) {
        double* row = &P[p0 + (size_t)(i / 16) * nt * 64 + i % 16];
        const int c0 = 16 * (i / 16) - bw;  // first column of the tile's first multiply
        for (int col = std::max(0, i - bw); col <= std::min(n1 - 1, i + bw); ++col)
          row[((col - c0) / 4) * 64 + 16 * ((col - c0) % 4)] = W[(size_t)i * nb + col - i + bw];
      }
      c->tm_bw[d][held] = bw;
    }
  if (!c->tm_all) ILH_HIP(c, hipMalloc((void**)&c->tm_all, (P.size() + 2 * (size_t)c->nh1) * sizeof(double)));
  ILH_HIP(c, hipMemcpy(c->tm_all, P.data(), P.size() * sizeof(double), hipMemcpyHostToDevice));
  for (int d = 0; d < c->dim; ++d)
    for (int held = 0; held < 2; ++held) c->tm_w[d][held] = c->tm_all + at_d[d][held];
  c->tm_tmp = c->tm_all + P.size();
  c->tm_ok = true;
  return ILH_OK;
}

struct TensorW {
  const double* w[3];  // per component
  int bw[3];
};

typedef double d4 __attribute__((ext_vector_type(4)));

// One direction (n1 nodes at stride sn) of every component (grid.z): lines at stride 1 within
// `inner` of them (direction d >= 1, outer blocks of n1 * inner entries), or at stride n1 (FIRST:
// direction 0).  A wave takes 16 nodes (row tile) of 16 lines; the waves of a group take
// neighbouring row tiles of the same lines (FIRST: a line's entries are read by all of them) or
// neighbouring lines of one row tile (the weights are).  LAST: the solution's entries go through the
// epilogue of MassOut instead of to out.
template <bool FIRST, bool LAST>
__global__ void __launch_bounds__(64 * TM_W) k_tensor(const double* __restrict__ in, double* __restrict__ out,
                                                      const TensorW tw, int n1, int64_t lines, int64_t N,
                                                      const KParams P, const MassOut mo) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int tiles = (n1 + 15) / 16, c = blockIdx.z, bw = tw.bw[c], nt = (16 + 2 * bw + 3) / 4;
  int tile, ot = 0;
  int64_t l0;
  if constexpr (FIRST) {
    tile = blockIdx.y * TM_W + wid;
    l0 = (int64_t)blockIdx.x * 16;
  } else {
    ot = blockIdx.y / tiles;
    tile = blockIdx.y - ot * tiles;
    l0 = ((int64_t)blockIdx.x * TM_W + wid) * 16;
  }
  if (tile >= tiles || l0 >= lines) return;
  const int i0 = 16 * tile, ln = lane & 15, lk = lane >> 4;
  const bool have = l0 + ln < lines;
  const int64_t line = have ? l0 + ln : lines - 1;
  const int64_t sn = FIRST ? 1 : lines;
  const int64_t base = c * N + (FIRST ? line * n1 : (int64_t)ot * n1 * lines + line);
  const double* w = tw.w[c] + (int64_t)tile * nt * 64 + lane;
  const int r0 = i0 - bw + lk;
  auto wt = [&](int t) { return w[t * 64]; };
  auto xt = [&](int t) { return in[base + (int64_t)min(max(r0 + 4 * t, 0), n1 - 1) * sn]; };
  // the multiplies over the tile's own columns, then those left of them (nl) and right of them (nr)
  const int nl = bw / 4, mid = (bw + 15) / 4 - nl + 1, nr = nt - nl - mid;
  double am[TM_M], bm[TM_M];
#pragma unroll
  for (int q = 0; q < TM_M; ++q) {
    const int t = nl + min(q, mid - 1);
    am[q] = wt(t);
    bm[q] = xt(t);
  }
  d4 lo = {0.0, 0.0, 0.0, 0.0}, hi = lo, acc, err;
  for (int t0 = 0; t0 < max(nl, nr); t0 += TM_U / 2) {
    double a[TM_U], b[TM_U];
#pragma unroll
    for (int q = 0; q < TM_U; ++q) {
      const int t = t0 + q / 2, tt = q % 2 == 0 ? min(t, nt - 1) : max(nt - 1 - t, 0);
      a[q] = wt(tt);
      b[q] = xt(tt);
    }
#pragma unroll
    for (int q = 0; q < TM_U; ++q) {
      const int t = t0 + q / 2;
      if (q % 2 == 0)
        lo = __builtin_amdgcn_mfma_f64_16x16x4f64(t < nl ? a[q] : 0.0, b[q], lo, 0, 0, 0);
      else
        hi = __builtin_amdgcn_mfma_f64_16x16x4f64(t < nr ? a[q] : 0.0, b[q], hi, 0, 0, 0);
    }
  }
  // s + e += x, the rounding error of the sum kept in e
  auto add = [](double& s, double& e, double x) {
    const double n = s + x, t = n - s;
    e += (s - (n - t)) + (x - t);
    s = n;
  };
  acc = lo;
  err = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double v = acc[r], e = 0.0;
    add(v, e, hi[r]);
    acc[r] = v;
    err[r] = e;
  }
#pragma unroll
  for (int q = 0; q < TM_M; ++q) {
    if (q >= mid) break;
    const d4 zero = {0.0, 0.0, 0.0, 0.0}, x = __builtin_amdgcn_mfma_f64_16x16x4f64(am[q], bm[q], zero, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double v = acc[r], e = err[r];
      add(v, e, x[r]);
      acc[r] = v;
      err[r] = e;
    }
  }
  // (an infinite sum has no rounding error: inf - inf)
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] += err[r] == err[r] ? err[r] : 0.0;
  if (!have) return;
  // grid index of the line along direction c of the last pass (c below the pass's direction)
  const uint32_t l32 = (uint32_t)line, ng0 = P.ng[0];
  const int gl = P.dim == 2 ? (int)l32 : c == 0 ? (int)(l32 % ng0) : (int)(l32 / ng0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // lane l holds rows l / 16 + 4 q of line l mod 16
    const int j = i0 + lk + 4 * q;
    if (j >= n1) break;
    const int64_t g = base + (int64_t)j * sn;
    if constexpr (!LAST) {
      out[g] = acc[q];
    } else {
      const bool cons = on_wall(P.walls, c, c == P.dim - 1 ? j : gl, P.ng[c]);
      const double s = !cons ? mo.sign * acc[q] : mo.cons != 0.0 ? mo.cons * mo.b[g] : 0.0;
      if (mo.a) mo.a[g] = s;
      if (mo.zero) mo.zero[g] = 0.0;
      if (mo.v) {
        const double v = mo.v[g], vm = v + mo.dv * s;
        mo.vm[g] = vm;
        mo.xo[g] = mo.x[g] + mo.dx * vm;
        if (mo.vo) mo.vo[g] = v + mo.dvo * s;
      }
    }
  }
}

int tensor_mass_solve(ilh_ctx* c, const MassOut& mo) {
  int st = tensor_setup(c);
  if (st) return st;
  const int D = c->dim;
  const double* src = mo.b;
  for (int d = 0; d < D; ++d) {
    TensorW tw{};
    for (int k = 0; k < D; ++k) {
      tw.w[k] = c->tm_w[d][k == d ? 1 : 0];
      tw.bw[k] = c->tm_bw[d][k == d ? 1 : 0];
    }
    const int n1 = c->ng[d];
    const unsigned tiles = (n1 + 15) / 16;
    double* dst = c->tm_tmp + (int64_t)(d & 1) * c->nh1;
    if (d == 0) {
      const int64_t lines = c->N / n1;
      hipLaunchKernelGGL((k_tensor<true, false>), dim3((unsigned)((lines + 15) / 16), (tiles + TM_W - 1) / TM_W, D),
                         dim3(64 * TM_W), 0, c->stream, src, dst, tw, n1, lines, c->N, c->kp, mo);
    } else {
      const int64_t inner = d == 1 ? c->ng[0] : (int64_t)c->ng[0] * c->ng[1], outer = c->N / (inner * n1);
      const dim3 grid((unsigned)((inner + 16 * TM_W - 1) / (16 * TM_W)), (unsigned)(tiles * outer), D);
      auto f = d == D - 1 ? k_tensor<false, true> : k_tensor<false, false>;
      hipLaunchKernelGGL(f, grid, dim3(64 * TM_W), 0, c->stream, src, dst, tw, n1, inner, c->N, c->kp, mo);
    }
    src = dst;
  }
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}

}  // namespace ilh
