// Learned Newton initial guess: per-element features, a BF16/FP32 MLP on MFMA, and the
// assembly of the predicted element-local stage rates into a block vector.
//
// MLP tensors: every width w is padded to P(w) = 32 ceil(w / 32); padding entries are zero.
//   W_l  [P(w_{l+1})][P(w_l)]  BF16 (uint16 storage), WT_l = transpose of W_l
//   b_l  [P(w_{l+1})]          FP32
//   activations [batch][P(w)]  FP32 (rounded to BF16 where they enter an MFMA)
// Dense products use v_mfma_f32_16x16x32_bf16: BF16 operands, FP32 accumulation.
// Hidden layers use GELU in its erf form; the last layer is linear.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "ilh_internal.h"

namespace ilh {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

static inline int pad32(int w) { return (w + 31) / 32 * 32; }

// round-to-nearest-even FP32 -> BF16 bits (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_d(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// ---------------------------------------------------------------------------------------
// Training: three launches for a whole network, instead of one per layer and product.
//
// A row of the batch goes through every layer by itself, forward and (for the data gradients)
// backward, so a work-group takes 16 rows through all layers: eight waves, each with one 16-column
// output tile of a layer (widths are at most 128), the activations passing between layers through two
// alternating LDS tiles in the MFMA operand layout, the next layer's weights requested from L2 while
// this layer's are used.  What bounds it is that chain (a barrier, four MFMAs, the erf and the stores
// per layer), not bytes or flops: batch 4,096 of the 90-128-128-128-41 network is 1.3 GFLOP and 30 MB.
// The weight gradients reduce over the batch, so they come in a third launch over (256 rows, 64 x 64
// output) blocks of all layers at once, from the BF16 data gradients that the second left behind.
// Layer by layer the forward took 55 us, the data gradients 58 and the weight gradients 132 (one wave
// read its operands element by element down a column, and one work-group row summed the bias gradients
// in a serial loop), now 10, 15 and 10; a training step of 4,096 rows 310 -> 60 us.  Operand rounding,
// accumulation order and epilogues are those of the layer-by-layer form, so zs, acts and the data
// gradients are bit for bit the same.
//
// MFMA 16x16x32 operand layout: lane l holds row/col (l % 16) and the 8 consecutive k of
// block (l / 16); the accumulator holds column (l % 16), rows 4 (l / 16) + 0..3.
constexpr int ML_MAXL = 8;
constexpr int FZ_WMAX = 57344;   // BF16 weights (rows counted padded by 8) that the fused inference call takes: the
                                 // limit of its first form, which held them in LDS; larger models go layer by layer
constexpr int ML_T = 512;        // threads of the row kernels: one wave per 16-column tile
constexpr int ML_LD = 128 + 8;   // LDS row of an activation tile (BF16, padded)
constexpr int ML_MAXB = 512;     // work-groups of the data-gradient launch (each walks 16-row tiles)
constexpr int MW_ROWS = 256;     // batch rows of a weight-gradient block
constexpr int MW_LD = MW_ROWS + 8;

struct MlpNet {
  int nl;
  int kp[ML_MAXL], np[ML_MAXL];  // padded widths
  int wo[ML_MAXL], bo[ML_MAXL];  // weight and bias offsets
  int64_t ao[ML_MAXL];           // offset of the layer's [batch][np] block in zs, acts and the data gradients
  int qo[ML_MAXL + 1];           // first 64 x 64 block of the layer in the weight-gradient grid
  int wtot, btot;
  // (gradients, not WHOLE) the layers l0 .. l1 of one pair of launches, the offsets of their data
  // gradients in dzb, and the columns of their bias sums
  int l0, l1;
  int64_t zo[ML_MAXL];
  int bcols;
};

// 16-byte loads that assume the alignment of one element only (global memory takes them)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 ldbf8(const uint16_t* p) {
  const u32x4 v = *reinterpret_cast<const u32x4u*>(p);
  return __builtin_bit_cast(bf16x8, v);
}

// a wave's operand of layer l: column n = 16 wave + ln of the output (clamped), its weights and bias
__device__ __forceinline__ void load_weights(const MlpNet& F, const uint16_t* W, const float* bias, int l, int wave,
                                             int ln, int kb, bf16x8 (&w)[4], float& b) {
  const int n = min(wave * 16 + ln, F.np[l] - 1), ns = F.kp[l] / 32;
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = ldbf8(W + F.wo[l] + n * F.kp[l] + min(q, ns - 1) * 32 + kb);
  b = bias[F.bo[l] + n];
}
// 16 rows (a: this lane's row of the LDS tile) times 16 columns over ns blocks of 32
__device__ __forceinline__ f32x4 row_product(const uint16_t* a, int ns, const bf16x8 (&w)[4]) {
  f32x4 acc = {0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q < ns)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(a + q * 32), w[q], acc, 0, 0, 0);
  return acc;
}

// Z_l = bf(A_{l-1}) W_l^T + b_l and A_l = gelu(Z_l) (last layer: Z_l) for 16 rows per work-group.
__global__ void __launch_bounds__(ML_T) k_mlp_fwd(const MlpNet F, const uint16_t* __restrict__ W,
                                                  const float* __restrict__ bias, const float* __restrict__ x,
                                                  int batch, float* __restrict__ zs, float* __restrict__ acts) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][16][ML_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, kb = (lane >> 4) * 8;
  const int row0 = blockIdx.x * 16;
  bf16x8 wc[4], wn[4];
  float bc = 0.0f, bn = 0.0f;
  load_weights(F, W, bias, 0, wave, ln, kb, wc, bc);
  {
    const int q = F.kp[0] / 4, r = tid / q, c4 = tid - r * q;
    if (r < 16) {
      f32x4u v = {0, 0, 0, 0};
      if (row0 + r < batch) v = *reinterpret_cast<const f32x4u*>(x + (int64_t)(row0 + r) * F.kp[0] + c4 * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) sA[0][r][c4 * 4 + j] = f2bf(v[j]);
    }
  }
  for (int l = 0; l < F.nl; ++l) {
    const int NP = F.np[l], cur = l & 1;
    const bool last = l == F.nl - 1;
    __syncthreads();  // this layer's input is complete, the other tile is no longer read
    if (!last) load_weights(F, W, bias, l + 1, wave, ln, kb, wn, bn);
    if (wave < NP / 16) {
      const f32x4 acc = row_product(&sA[cur][ln][kb], F.kp[l] / 32, wc);
      const int n = wave * 16 + ln;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rl = (lane >> 4) * 4 + j;
        const float z = acc[j] + bc, a = last ? z : gelu(z);
        if (!last) sA[cur ^ 1][rl][n] = f2bf(a);
        if (row0 + rl < batch) {
          const int64_t o = F.ao[l] + (int64_t)(row0 + rl) * NP + n;
          zs[o] = z;
          acts[o] = a;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) wc[q] = wn[q];
    bc = bn;
  }
}

// Loss gradient dZ_last = (Y - T) mask / batch, then dZ_{l-1} = (bf(dZ_l) W_l) gelu'(Z_{l-1}) down to
// layer l0, 16 rows at a time: to dzb in BF16 (the operand the weight gradients take), the column sums
// of the FP32 values over the work-group's rows to db (the first work-group's) and dbp[work-group -
// 1][bcols], the loss sum to part (nullable).  Also clears dW for the launch that follows.  A group of layers
// below the last one starts from the data gradients of layer l1 + 1 that an earlier launch left in dzb.
// WHOLE: all layers, with the offsets of the activations (4,096 rows: 14.8 us, with a group's offsets 15.2;
// the weight gradients 10.1 and 11.3).
template <bool WHOLE>
__global__ void __launch_bounds__(ML_T) k_mlp_bwd(const MlpNet F, const uint16_t* __restrict__ WT,
                                                  const float* __restrict__ zs, const float* __restrict__ acts,
                                                  const float* __restrict__ target, int batch, int nvalid,
                                                  uint16_t* __restrict__ dzb, float* __restrict__ dbp,
                                                  float* __restrict__ dW, float* __restrict__ db,
                                                  double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint16_t sD[2][16][ML_LD];
  __shared__ float sB[ML_MAXL * 128];
  __shared__ double sL[ML_T / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, kb = (lane >> 4) * 8;
  const int rl0 = (lane >> 4) * 4, n = wave * 16 + ln;
  const int l0 = WHOLE ? 0 : F.l0, b0 = WHOLE ? 0 : F.bo[F.l0], bcols = WHOLE ? F.btot : F.bcols;
  const bool from_loss = WHOLE || F.l1 == F.nl - 1;
  if (from_loss)
    for (int i = blockIdx.x * ML_T + tid; i < F.wtot; i += gridDim.x * ML_T) dW[i] = 0.0f;
  for (int i = tid; i < bcols; i += ML_T) sB[i] = 0.0f;
  __syncthreads();
  double loss = 0.0;
  const int ntiles = (batch + 15) / 16;
  // one column's four rows: to LDS (operand of the next product), to dzb, and its sum to sB
  auto put = [&](int l, int buf, int row0, const float (&v)[4]) {
    const int NP = F.np[l];
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint16_t h = f2bf(v[j]);
      sD[buf][rl0 + j][n] = h;
      if (row0 + rl0 + j < batch) dzb[(WHOLE ? F.ao[l] : F.zo[l]) + (int64_t)(row0 + rl0 + j) * NP + n] = h;
      s += v[j];
    }
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < 16) sB[F.bo[l] - b0 + n] += s;  // (the column belongs to this wave alone)
  };
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int row0 = tile * 16;
    int cur = 0;
    if (!from_loss) {
      const int l = F.l1 + 1, NP = F.np[l], r = tid / 32, c = 4 * (tid % 32);
      if (c < NP) {
        const uint16_t* p = dzb + F.zo[l] + (int64_t)min(row0 + r, batch - 1) * NP + c;
#pragma unroll
        for (int j = 0; j < 4; ++j) sD[0][r][c + j] = row0 + r < batch ? p[j] : (uint16_t)0;
      }
    } else {
      const int l = F.nl - 1, NP = F.np[l];
      if (wave < NP / 16) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int rr = row0 + rl0 + j;
          const int64_t o = (int64_t)rr * NP + n;
          const float d = (n < nvalid && rr < batch) ? acts[F.ao[l] + o] - target[o] : 0.0f;
          v[j] = d / batch;
          loss += 0.5 * (double)d * d / batch;
        }
        put(l, 0, row0, v);
      }
    }
    for (int l = WHOLE ? F.nl - 1 : min(F.l1 + 1, F.nl - 1); l > l0; --l) {
      const int KP = F.kp[l], NP = F.np[l], ns = NP / 32;
      bf16x8 w[4];
      float gz[4];
      const bool on = wave < KP / 16;
      const int k = min(n, KP - 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = ldbf8(WT + F.wo[l] + k * NP + min(q, ns - 1) * 32 + kb);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        gz[j] = zs[F.ao[l - 1] + (int64_t)min(row0 + rl0 + j, batch - 1) * KP + k];
      __syncthreads();  // dZ_l is complete, the other tile is no longer read
      if (on) {
        const f32x4 acc = row_product(&sD[cur][ln][kb], ns, w);
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = row0 + rl0 + j < batch ? acc[j] * gelu_d(gz[j]) : 0.0f;
        put(l - 1, cur ^ 1, row0, v);
      }
      cur ^= 1;
    }
    __syncthreads();  // the next tile writes the first LDS tile again
  }
  float* bp = blockIdx.x == 0 ? db + b0 : dbp + (int64_t)(blockIdx.x - 1) * bcols;
  for (int i = tid; i < bcols; i += ML_T) bp[i] = sB[i];
  if (!from_loss || !part) return;
  for (int o = 32; o > 0; o >>= 1) loss += __shfl_down(loss, o, 64);
  if (lane == 0) sL[wave] = loss;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int i = 0; i < ML_T / 64; ++i) s += sL[i];
    part[blockIdx.x] = s;
  }
}

// 8 x 8 BF16 values (v[i]: row i, eight columns) as eight columns of eight rows
__device__ __forceinline__ void transpose8(const u32x4 (&v)[8], u32x4 (&t)[8]) {
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t a = v[2 * i][c / 2], b = v[2 * i + 1][c / 2];
      t[c][i] = (c & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
    }
}

// dW_l[n][k] += sum_b bf(dZ_l[b][n]) bf(A_{l-1}[b][k]) over 256 batch rows (grid.x) for one 64 x 64 block
// of one layer's weights (grid.y).  Both operands run along the batch, so the rows are staged in LDS
// transposed (a thread loads 8 rows x 8 columns in 16-byte pieces and stores 8 columns), from where a
// lane reads its 8 consecutive rows in one piece.  The first row of groups also sums the bias gradients
// and the loss from the parts of the launch before.
template <bool WHOLE>
__global__ void __launch_bounds__(256) k_mlp_wgrad(const MlpNet F, const uint16_t* __restrict__ dzb,
                                                   const float* __restrict__ x, const float* __restrict__ acts,
                                                   int batch, float* __restrict__ dW, const float* __restrict__ dbp,
                                                   const double* __restrict__ part, int nparts, float* db,
                                                   double* loss) {
  __shared__ __attribute__((aligned(16))) uint16_t sZ[64][MW_LD], sX[64][MW_LD];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, ln = lane & 15, kb = (lane >> 4) * 8;
  const int l0 = WHOLE ? 0 : F.l0, l1 = WHOLE ? F.nl - 1 : F.l1, bcols = WHOLE ? F.btot : F.bcols;
  int l = l0;
  while (l < l1 && (int)blockIdx.y >= F.qo[l + 1]) ++l;
  const int KP = F.kp[l], NP = F.np[l], qk = (KP + 63) / 64, qi = blockIdx.y - F.qo[l];
  const int n0 = 64 * (qi / qk), k0 = 64 * (qi % qk), nn = min(64, NP - n0), kk = min(64, KP - k0);
  const int b0 = blockIdx.x * MW_ROWS, rb = (t / 8) * 8, cb = (t % 8) * 8;
  const float* X = l == 0 ? x : acts + F.ao[l - 1];
  if (cb < nn) {
    u32x4 v[8], o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = b0 + rb + i;
      v[i] = u32x4{0, 0, 0, 0};
      if (row < batch) v[i] = *reinterpret_cast<const u32x4u*>(dzb + (WHOLE ? F.ao[l] : F.zo[l]) + (int64_t)row * NP + n0 + cb);
    }
    transpose8(v, o);
#pragma unroll
    for (int c = 0; c < 8; ++c) *reinterpret_cast<u32x4*>(&sZ[cb + c][rb]) = o[c];
  }
  if (cb < kk) {
    u32x4 v[8], o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = b0 + rb + i;
      f32x4u a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
      if (row < batch) {
        const float* p = X + (int64_t)row * KP + k0 + cb;
        a = *reinterpret_cast<const f32x4u*>(p);
        b = *reinterpret_cast<const f32x4u*>(p + 4);
      }
      v[i] = u32x4{f2bf(a[0]) | (uint32_t)f2bf(a[1]) << 16, f2bf(a[2]) | (uint32_t)f2bf(a[3]) << 16,
                   f2bf(b[0]) | (uint32_t)f2bf(b[1]) << 16, f2bf(b[2]) | (uint32_t)f2bf(b[3]) << 16};
    }
    transpose8(v, o);
#pragma unroll
    for (int c = 0; c < 8; ++c) *reinterpret_cast<u32x4*>(&sX[cb + c][rb]) = o[c];
  }
  __syncthreads();
  const int wn = (wave & 1) * 32, wk = (wave >> 1) * 32;  // the wave's 32 x 32 outputs
  if (wn < nn && wk < kk) {
    f32x4 acc[2][2] = {};
#pragma unroll
    for (int s = 0; s < MW_ROWS / 32; ++s) {
      bf16x8 a[2], b[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        a[q] = *reinterpret_cast<const bf16x8*>(&sZ[wn + 16 * q + ln][s * 32 + kb]);
        b[q] = *reinterpret_cast<const bf16x8*>(&sX[wk + 16 * q + ln][s * 32 + kb]);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int p = 0; p < 2; ++p) acc[q][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q], b[p], acc[q][p], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          unsafeAtomicAdd(&dW[F.wo[l] + (n0 + wn + 16 * q + (lane >> 4) * 4 + j) * KP + k0 + wk + 16 * p + ln],
                          acc[q][p][j]);
  }
  if (blockIdx.x != 0) return;
  __syncthreads();  // the LDS tiles are no longer read
  if (k0 == 0) {
    float* sF = reinterpret_cast<float*>(&sZ[0][0]);
    const int col = t & 63;
    float s = 0.0f;
    if (col < nn) {
      // part 0 waits in db itself: these columns of it are read here only, before the sums replace them
      if (wave == 0) s = db[F.bo[l] + n0 + col];
      const float* p = dbp + F.bo[l] - (WHOLE ? 0 : F.bo[l0]) + n0 + col;
      for (int b = wave; b < nparts - 1; b += 4 * 16) {  // 16 loads in flight
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = p[(int64_t)min(b + 4 * q, nparts - 2) * bcols];
#pragma unroll
        for (int q = 0; q < 16; ++q) s += b + 4 * q < nparts - 1 ? v[q] : 0.0f;
      }
    }
    sF[t] = s;
    __syncthreads();
    if (t < nn) db[F.bo[l] + n0 + t] = sF[t] + sF[64 + t] + sF[128 + t] + sF[192 + t];
  }
  if (loss && blockIdx.y == 0) {
    double* sP = reinterpret_cast<double*>(&sX[0][0]);
    double s = 0.0;
    for (int b = t; b < nparts; b += 256) s += part[b];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (lane == 0) sP[wave] = s;
    __syncthreads();
    if (t == 0) *loss = sP[0] + sP[1] + sP[2] + sP[3];
  }
}

// Adam on FP32 master parameters; the weight part is rounded to BF16 into W and WT.
__global__ void k_adam(int64_t n, float* p, const float* g, float* m1, float* m2, float b1, float b2, float lr,
                       float bc1, float bc2, float eps) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.0f - b1) * gi;
    const float b = b2 * m2[i] + (1.0f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    p[i] -= lr * (a * bc1) / (sqrtf(b * bc2) + eps);
  }
}
// every layer's FP32 weights to BF16, W and its transpose
__global__ void k_pack(const MlpNet F, const float* __restrict__ Wm, uint16_t* __restrict__ W,
                       uint16_t* __restrict__ WT) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < F.wtot; i += gridDim.x * blockDim.x) {
    int l = 0;
    while (l + 1 < F.nl && i >= F.wo[l + 1]) ++l;
    const int o = i - F.wo[l], r = o / F.kp[l], c = o - r * F.kp[l];
    const uint16_t h = f2bf(Wm[i]);
    W[i] = h;
    WT[F.wo[l] + c * F.np[l] + r] = h;
  }
}

// ---------------------------------------------------------------------------------------
// Learned-guess features and targets (2D).  Per element e with local H1 node (a, b) and
// L2 dof j:  features = [v_c(a,b)/vs (c = 0, 1) | e_j/es | corner_c - centre_c)/xs (4 corners)
//                        | optionally base_v/kvs | base_e/kes],  row stride ld, zero padded.
struct FeatArgs {
  const double* u;
  const double* base;  // nullable: no base block
  double vs, es, xs, kvs, kes;
  const float* mu;  // nullable: no normalisation
  const float* sd;
};

// feature i of element e (0 past the feature count)
__device__ __forceinline__ float feature_value(const KParams& P, const FeatArgs& A, int64_t e, int i) {
  const int k = P.k, D1D = k + 1, ND = D1D * D1D, NL = k * k;
  const int ex = (int)(e % P.n[0]), ey = (int)(e / P.n[0]);
  const int64_t N = P.N, nh1 = 2 * N, ng0 = P.ng[0];
  const double* u = A.u;
  const int nbase = A.base ? 2 * ND + NL : 0;
  const int nin = 2 * ND + NL + 8 + nbase;
  double val = 0.0;
  if (i < 2 * ND) {
    const int c = i / ND, li = i % ND, a = li % D1D, b = li / D1D;
    val = u[nh1 + c * N + (int64_t)(k * ey + b) * ng0 + k * ex + a] / A.vs;
  } else if (i < 2 * ND + NL) {
    val = u[2 * nh1 + e * NL + (i - 2 * ND)] / A.es;
  } else if (i < 2 * ND + NL + 8) {
    const int j = i - 2 * ND - NL, corner = j / 2, c = j % 2;
    const int a = (corner & 1) ? k : 0, b = (corner & 2) ? k : 0;
    double cen = 0;
    for (int q = 0; q < 4; ++q)
      cen += u[c * N + (int64_t)(k * ey + ((q & 2) ? k : 0)) * ng0 + k * ex + ((q & 1) ? k : 0)];
    val = (u[c * N + (int64_t)(k * ey + b) * ng0 + k * ex + a] - 0.25 * cen) / A.xs;
  } else if (i < nin) {
    const int j = i - 2 * ND - NL - 8;
    if (j < 2 * ND) {
      const int c = j / ND, li = j % ND, a = li % D1D, b = li / D1D;
      val = A.base[nh1 + c * N + (int64_t)(k * ey + b) * ng0 + k * ex + a] / A.kvs;
    } else {
      val = A.base[2 * nh1 + e * NL + (j - 2 * ND)] / A.kes;
    }
  }
  if (A.mu && i < nin) val = (val - (double)A.mu[i]) / (double)A.sd[i];
  return (float)val;
}

__global__ void k_features(const KParams P, const FeatArgs A, float* feat, int ld) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.y + threadIdx.y;
  if (e >= P.Ne) return;
  float* f = feat + e * ld;
  for (int i = threadIdx.x; i < ld; i += blockDim.x) f[i] = feature_value(P, A, e, i);
}

// ---------------------------------------------------------------------------------------
// Fused inference: the features of 16 elements, every layer and the store of the network output in
// one launch, on the row scheme of k_mlp_fwd (a wave per 16-column tile, weights from L2 one layer ahead).
// The operand rounding (BF16), the accumulation order and the epilogue are those of k_mlp_fwd, so the
// output is the layered forward's.  Copying all weights to LDS first (111 KB a work-group, 336 tiles on
// 256 compute units) took 27 us at 5,376 elements, this form 17.7 (half of it the features).
__global__ void __launch_bounds__(ML_T) k_guess_fused(const KParams P, const FeatArgs FA, const MlpNet F,
                                                     const uint16_t* __restrict__ W, const float* __restrict__ bias,
                                                     float* __restrict__ pred, int ld_out) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][16][ML_LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ln = lane & 15, kb = (lane >> 4) * 8;
  const int64_t row0 = (int64_t)blockIdx.x * 16;
  bf16x8 wc[4], wn[4];
  float bc = 0.0f, bn = 0.0f;
  load_weights(F, W, bias, 0, wave, ln, kb, wc, bc);
  const int KP0 = F.kp[0];
  for (int i = tid; i < 16 * KP0; i += ML_T) {
    const int r = i / KP0, f = i - r * KP0;
    const int64_t e = row0 + r;
    sA[0][r][f] = f2bf(e < P.Ne ? feature_value(P, FA, e, f) : 0.0f);
  }
  for (int l = 0; l < F.nl; ++l) {
    const int cur = l & 1;
    const bool last = l == F.nl - 1;
    __syncthreads();  // this layer's input is complete, the other tile is no longer read
    if (!last) load_weights(F, W, bias, l + 1, wave, ln, kb, wn, bn);
    if (wave < F.np[l] / 16) {
      const f32x4 acc = row_product(&sA[cur][ln][kb], F.kp[l] / 32, wc);
      const int n = wave * 16 + ln;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int rl = (lane >> 4) * 4 + j;
        const float z = acc[j] + bc;
        if (last) {
          if (row0 + rl < P.Ne && n < ld_out) pred[(row0 + rl) * ld_out + n] = z;
        } else {
          sA[cur ^ 1][rl][n] = f2bf(gelu(z));
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) wc[q] = wn[q];
    bc = bn;
  }
}

// targets: element-local [(k_v - base_v)/kvs | (k_e - base_e)/kes], row stride ld
__global__ void k_targets(const KParams P, const double* kk, const double* base, double kvs, double kes,
                          const float* osc, float* t, int ld) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.y + threadIdx.y;
  if (e >= P.Ne) return;
  const int k = P.k, D1D = k + 1, ND = D1D * D1D, NL = k * k;
  const int ex = (int)(e % P.n[0]), ey = (int)(e / P.n[0]);
  const int64_t N = P.N, nh1 = 2 * N, ng0 = P.ng[0];
  for (int i = threadIdx.x; i < ld; i += blockDim.x) {
    double val = 0.0;
    if (i < 2 * ND) {
      const int c = i / ND, li = i % ND, a = li % D1D, b = li / D1D;
      const int64_t g = nh1 + c * N + (int64_t)(k * ey + b) * ng0 + k * ex + a;
      val = (kk[g] - (base ? base[g] : 0.0)) / kvs;
    } else if (i < 2 * ND + NL) {
      const int64_t g = 2 * nh1 + e * NL + (i - 2 * ND);
      val = (kk[g] - (base ? base[g] : 0.0)) / kes;
    }
    if (osc && i < 2 * ND + NL) val /= (double)osc[i];
    t[e * ld + i] = (float)val;
  }
}

// Assembly, one thread per H1 velocity entry or energy entry: k_v = base_v plus the mean over the (up
// to four) elements that hold the node of kvs pred_v (0 on constrained rows), k_x = u_v + tau k_v, k_e =
// base_e + kes pred_e.  Each node gathers its elements' predictions: no zero fill and no atomics in
// front of it.  zero (nullable): 2 N entries cleared by the same launch.
__global__ void k_assemble(const KParams P, const float* __restrict__ pred, int ld, double kvs, double kes,
                           const float* __restrict__ osc, const double* __restrict__ base,
                           const double* __restrict__ u, double tau, double* __restrict__ kout, double* zero,
                           double* zero2) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t N = P.N, nh1 = 2 * N;
  const int k = P.k, D1D = k + 1, ND = D1D * D1D, NL = k * k;
  if (i < nh1) {
    const int c = i < N ? 0 : 1;
    const int64_t node = i - c * N;
    const int ng0 = P.ng[0], I = (int)(node % ng0), J = (int)(node / ng0);
    // the last element with the node at its start or inside, and the one before when it is on the edge
    const int ex1 = min(I / k, P.n[0] - 1), ex0 = (I % k == 0 && I > 0 && I < ng0 - 1) ? ex1 - 1 : ex1;
    const int ey1 = min(J / k, P.n[1] - 1), ey0 = (J % k == 0 && J > 0 && J < P.ng[1] - 1) ? ey1 - 1 : ey1;
    double acc = 0.0;
    for (int ey = ey0; ey <= ey1; ++ey)
      for (int ex = ex0; ex <= ex1; ++ex) {
        const int li = c * ND + (J - k * ey) * D1D + I - k * ex;
        const double sc = osc ? (double)osc[li] : 1.0;
        acc += kvs * sc * (double)pred[((int64_t)ey * P.n[0] + ex) * ld + li];
      }
    const bool cons = on_wall(P.walls, c, c == 0 ? I : J, P.ng[c]);
    const double kv = cons ? 0.0 : base[nh1 + i] + acc / ((ex1 - ex0 + 1) * (ey1 - ey0 + 1));
    kout[nh1 + i] = kv;
    kout[i] = u[nh1 + i] + tau * kv;
    if (zero) zero[i] = 0.0;
    if (zero2) zero2[i] = 0.0;
  } else if (i < nh1 + (int64_t)P.Ne * NL) {
    const int64_t q = i - nh1, e = q / NL, j = q - e * NL;
    const double sc = osc ? (double)osc[2 * ND + j] : 1.0;
    kout[2 * nh1 + q] = base[2 * nh1 + q] + kes * sc * (double)pred[e * ld + 2 * ND + j];
  }
}

// ---------------------------------------------------------------------------------------
static int check_widths(ilh_ctx* c, int nl, const int* w) {
  if (nl < 1 || nl > 8) return fail(c, ILH_EINVAL, "1..8 layers");
  for (int l = 0; l <= nl; ++l)
    if (w[l] < 1 || w[l] > 128) return fail(c, ILH_EINVAL, "MLP widths must be in 1..128");
  return ILH_OK;
}

// the layer shapes (padded input, padded output) that forward and backward take
static bool layer_shape(int k, int n) {
  return k == 128 || n == 128 || ((k == 32 || k == 64) && (n == 32 || n == 64));
}

static MlpNet make_net(int nl, const int* widths, int batch) {
  MlpNet F{};
  F.nl = nl;
  int64_t ao = 0;
  for (int l = 0; l < nl; ++l) {
    F.kp[l] = pad32(widths[l]);
    F.np[l] = pad32(widths[l + 1]);
    F.wo[l] = F.wtot;
    F.bo[l] = F.btot;
    F.ao[l] = ao;
    F.qo[l + 1] = F.qo[l] + ((F.np[l] + 63) / 64) * ((F.kp[l] + 63) / 64);
    F.wtot += F.kp[l] * F.np[l];
    F.btot += F.np[l];
    ao += (int64_t)batch * F.np[l];
  }
  return F;
}

int guess_assemble(ilh_ctx* c, const float* pred, int ld, double kvs, double kes, const float* osc,
                   const double* base, const double* u, double tau, double* kout, double* zero, double* zero2) {
  const int64_t n = c->nh1 + c->nl2;
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->kp, pred, ld, kvs, kes,
                     osc, base, u, tau, kout, zero, zero2);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
}

}  // namespace ilh

using namespace ilh;

extern "C" {

int ilh_guess_features(ilh_ctx* c, const double* u, const double* base, double vs, double es, double xs,
                       double kvs, double kes, const float* mu, const float* sd, float* feat, int ld) {
  ILH_TRY
  if (!c || !u || !feat || c->dim != 2) return fail(c, ILH_EINVAL, "guess features: 2D only, non-null u/feat");
  const int ND = (c->k + 1) * (c->k + 1), NL = c->k * c->k;
  const int nin = 2 * ND + NL + 8 + (base ? 2 * ND + NL : 0);
  if (ld < nin) return fail(c, ILH_EINVAL, "feature row stride too small");
  if (!(vs > 0 && es > 0 && xs > 0 && kvs > 0 && kes > 0)) return fail(c, ILH_EINVAL, "scales must be > 0");
  const FeatArgs fa{u, base, vs, es, xs, kvs, kes, mu, sd};
  hipLaunchKernelGGL(k_features, dim3((unsigned)((c->Ne + 3) / 4)), dim3(64, 4), 0, c->stream, c->kp, fa, feat, ld);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_guess_targets(ilh_ctx* c, const double* kk, const double* base, double kvs, double kes, const float* osc,
                      float* t, int ld) {
  ILH_TRY
  if (!c || !kk || !t || c->dim != 2) return fail(c, ILH_EINVAL, "guess targets: 2D only");
  const int ND = (c->k + 1) * (c->k + 1), NL = c->k * c->k;
  if (ld < 2 * ND + NL || !(kvs > 0 && kes > 0)) return fail(c, ILH_EINVAL, "target stride/scales");
  hipLaunchKernelGGL(k_targets, dim3((unsigned)((c->Ne + 3) / 4)), dim3(64, 4), 0, c->stream, c->kp, kk, base, kvs, kes,
                     osc, t, ld);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_guess_assemble(ilh_ctx* c, const float* pred, int ld, double kvs, double kes, const float* osc,
                       const double* base, const double* u, double tau, double* kout) {
  ILH_TRY
  if (!c || !pred || !base || !u || !kout || c->dim != 2) return fail(c, ILH_EINVAL, "guess assemble: 2D only");
  const int ND = (c->k + 1) * (c->k + 1), NL = c->k * c->k;
  if (ld < 2 * ND + NL) return fail(c, ILH_EINVAL, "prediction stride too small");
  return guess_assemble(c, pred, ld, kvs, kes, osc, base, u, tau, kout, nullptr, nullptr);
  ILH_CATCH(c)
}

int ilh_mlp_forward(ilh_ctx* c, int nl, const int* widths, const uint16_t* W, const float* b, const float* x,
                    int batch, float* zs, float* acts) {
  ILH_TRY
  if (!c || !widths || !W || !b || !x || !zs || !acts || batch < 0) return ILH_EINVAL;
  int st = check_widths(c, nl, widths);
  if (st) return st;
  if (batch == 0) return ILH_OK;
  const MlpNet F = make_net(nl, widths, batch);
  for (int l = 0; l < nl; ++l)
    if (!layer_shape(F.kp[l], F.np[l]))
      return fail(c, ILH_EINVAL, "unsupported MLP layer width (padded widths 32..128)");
  hipLaunchKernelGGL(k_mlp_fwd, dim3((batch + 15) / 16), dim3(ML_T), 0, c->stream, F, W, b, x, batch, zs, acts);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_guess_mlp_fused(ilh_ctx* c, const ilh_guess_model* m, const double* u, const double* base, float* pred,
                        int ld) {
  ILH_TRY
  if (!c || !m || !u || !pred || !m->W || !m->b || c->dim != 2) return fail(c, ILH_EINVAL, "fused guess MLP: 2D, non-null");
  int st = check_widths(c, m->nl, m->widths);
  if (st) return st;
  const int ND = (c->k + 1) * (c->k + 1), NL = c->k * c->k;
  const int nin = 2 * ND + NL + 8 + (m->with_base ? 2 * ND + NL : 0);
  if (m->widths[0] != nin || m->widths[m->nl] != 2 * ND + NL)
    return fail(c, ILH_EINVAL, "fused guess MLP: widths do not match the features and outputs of this mesh");
  if (m->with_base && !base) return fail(c, ILH_EINVAL, "fused guess MLP: the model takes the base iterate");
  const MlpNet F = make_net(m->nl, m->widths, 0);
  int64_t padded = 0;
  for (int l = 0; l < m->nl; ++l) padded += (int64_t)F.np[l] * (F.kp[l] + 8);
  if (padded > FZ_WMAX) return fail(c, ILH_EINVAL, "fused guess MLP: the weights exceed 112 KiB");
  if (ld < F.np[m->nl - 1]) return fail(c, ILH_EINVAL, "prediction stride below the padded output width");
  if ((reinterpret_cast<uintptr_t>(m->W) & 15) != 0) return fail(c, ILH_EINVAL, "fused guess MLP: W not 16-byte aligned");
  const FeatArgs fa{u, m->with_base ? base : nullptr, m->vscale, m->escale, m->xscale, m->kvscale, m->kescale,
                    m->mu, m->sd};
  hipLaunchKernelGGL(k_guess_fused, dim3((unsigned)((c->Ne + 15) / 16)), dim3(ML_T), 0, c->stream, c->kp, fa, F, m->W, m->b,
                     pred, ld);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_mlp_backward(ilh_ctx* c, int nl, const int* widths, const uint16_t* WT, const float* x, const float* zs,
                     const float* acts, const float* target, int batch, float* dW, float* db, float* work,
                     double* loss) {
  ILH_TRY
  if (!c || !widths || !WT || !x || !zs || !acts || !target || !dW || !db || !work || batch <= 0) return ILH_EINVAL;
  int st = check_widths(c, nl, widths);
  if (st) return st;
  MlpNet F = make_net(nl, widths, batch);
  for (int l = 0; l < nl; ++l)
    if (!layer_shape(F.kp[l], F.np[l]))
      return fail(c, ILH_EINVAL, "unsupported MLP layer width (padded widths 32..128)");
  // The caller's work holds 1,024 bytes a row: the BF16 data gradients and the bias sums of all layers (a
  // part for every 16 rows, the first one in db) where the padded outputs are some 450 or fewer, else of
  // two layers at a time, the lower one's gradients left for the next pair in one of two slots.
  const int nparts = std::min((batch + 15) / 16, ML_MAXB);
  const int64_t room = (int64_t)batch * 1024;
  uint16_t* dzb = reinterpret_cast<uint16_t*>(work);
  const bool whole = 2 * (int64_t)batch * F.btot + 4 * (int64_t)(nparts - 1) * F.btot <= room;
  int slot = 0;
  for (int hi = nl - 1; hi >= 0; hi = F.l0 - 1) {
    F.l1 = hi;
    F.l0 = whole ? 0 : std::max(hi - 1, 0);
    float* dbp;
    if (whole) {
      dbp = reinterpret_cast<float*>(dzb + (int64_t)batch * F.btot);
    } else {
      F.zo[hi] = 256 * (int64_t)batch;
      F.zo[F.l0] = 128 * (int64_t)slot * batch;
      slot ^= 1;
      dbp = reinterpret_cast<float*>(dzb + 384 * (int64_t)batch);
    }
    F.bcols = 0;
    F.qo[F.l0] = 0;
    for (int l = F.l0; l <= hi; ++l) {
      F.bcols += F.np[l];
      F.qo[l + 1] = F.qo[l] + ((F.np[l] + 63) / 64) * ((F.kp[l] + 63) / 64);
    }
    double* out = loss && hi == nl - 1 ? c->red_host + 2 : nullptr;
    auto bwd = whole ? k_mlp_bwd<true> : k_mlp_bwd<false>;
    auto wgrad = whole ? k_mlp_wgrad<true> : k_mlp_wgrad<false>;
    hipLaunchKernelGGL(bwd, dim3(nparts), dim3(ML_T), 0, c->stream, F, WT, zs, acts, target, batch, widths[nl], dzb,
                       dbp, dW, db, loss ? c->red : nullptr);
    hipLaunchKernelGGL(wgrad, dim3((batch + MW_ROWS - 1) / MW_ROWS, F.qo[hi + 1]), dim3(256), 0, c->stream, F, dzb, x,
                       acts, batch, dW, dbp, c->red, nparts, db, out);
  }
  ILH_HIP(c, hipGetLastError());
  if (loss) {  // (the last launch writes it to the pinned host buffer)
    ILH_HIP(c, hipStreamSynchronize(c->stream));
    *loss = c->red_host[2];
  }
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_mlp_adam(ilh_ctx* c, int64_t n, float* p, const float* g, float* m1, float* m2, int step, double lr,
                 double beta1, double beta2, double eps) {
  ILH_TRY
  if (!c || !p || !g || !m1 || !m2 || n < 0 || step < 1) return ILH_EINVAL;
  const double bc1 = 1.0 / (1.0 - std::pow(beta1, step)), bc2 = 1.0 / (1.0 - std::pow(beta2, step));
  hipLaunchKernelGGL(k_adam, dim3(1024), dim3(256), 0, c->stream, n, p, g, m1, m2, (float)beta1, (float)beta2,
                     (float)lr, (float)bc1, (float)bc2, (float)eps);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

int ilh_mlp_pack(ilh_ctx* c, int nl, const int* widths, const float* Wmaster, uint16_t* W, uint16_t* WT) {
  ILH_TRY
  if (!c || !widths || !Wmaster || !W || !WT) return ILH_EINVAL;
  int st = check_widths(c, nl, widths);
  if (st) return st;
  const MlpNet F = make_net(nl, widths, 0);
  hipLaunchKernelGGL(k_pack, dim3((F.wtot + 255) / 256), dim3(256), 0, c->stream, F, Wmaster, W, WT);
  ILH_HIP(c, hipGetLastError());
  return ILH_OK;
  ILH_CATCH(c)
}

}  // extern "C"
