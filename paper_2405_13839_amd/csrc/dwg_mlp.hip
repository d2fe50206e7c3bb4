// Learned initial normals: MLP 48 -> 128 -> 128 -> 3 (ReLU, normalised output) on the
// gfx950 matrix cores (v_mfma_f32_16x16x32_bf16: BF16 operands, FP32 accumulation),
// its backward pass and Adam, all in this file. Not in the paper: it replaces the random /
// PCA / Gauss-map initial normals of Sec. 5.1 ("Normal Initialization").
//
// MFMA operand layout (16x16x32): lane l holds A[l % 16][8 (l / 16) + j] and
// B[8 (l / 16) + j][l % 16], j = 0..7; the FP32 result holds D[4 (l / 16) + i][l % 16]. A and B
// are laid out alike (16 vectors of 32 consecutive products' operands), so an operand
// "fragment" (8 BF16 values per lane, 1 KB per wavefront) serves as either: with the weights as A
// and the rows as B a layer's result is transposed, four consecutive neurons of one row per lane.
// Two such result tiles (neurons 0-15 and 16-31) hold, in the four lanes l % 16, + 16, + 32, + 48 of
// a row, exactly the 32 values that the next layer's fragment wants in them; two register
// swaps per 32-bit word (v_permlane32_swap, v_permlane16_swap) put them in order (to_frag). So
// activations never leave the registers, in the same order of products as before. Weights are
// kept as fragments in LDS, read without bank conflicts.
//
// Parameter blob (FP32): W1[128][48] b1[128] W2[128][128] b2[128] W3[3][128] b3[3].
#include <cmath>

#include "dwg_internal.h"

namespace dwg {
namespace {

constexpr int IN = DWG_MLP_IN, HID = DWG_MLP_HID, OUT = DWG_MLP_OUT;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + HID * IN, OFF_W2 = OFF_B1 + HID,
              OFF_B2 = OFF_W2 + HID * HID, OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + OUT * HID,
              NPAR = OFF_B3 + OUT;
constexpr int NPART = NPAR + 1;  // per-block partial gradient + loss

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16;

// Fragments of the weights: W1 as [8 neuron tiles][2 steps of 32 inputs] (inputs 48-63 zero), W2 as
// [8][4], W3 as [4] (neurons 3-15 zero), and W2 transposed as [8 input tiles][4 steps of 32
// outputs] for the backward pass.
constexpr int F_W1 = 0, F_W2 = F_W1 + 16, F_W3 = F_W2 + 32, F_FWD = F_W3 + 4, F_W2T = F_FWD, F_ALL = F_W2T + 32;

// Four floats that are only known to be aligned as floats (one 16-byte load all the same).
struct __attribute__((packed, aligned(4))) float4u {
  float x, y, z, w;
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {  // BF16, round to nearest even
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

__device__ __forceinline__ uint4 pack8(const float* f) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

__device__ __forceinline__ f32x4 mfma(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// a = rows of 16 lanes (a0 a1 a2 a3), b = (b0 b1 b2 b3) -> a = (a0 a2 b0 b2), b = (a1 a3 b1 b3).
__device__ __forceinline__ void interleave(uint32_t& a, uint32_t& b) {
  const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  const auto t = __builtin_amdgcn_permlane16_swap(s[0], s[1], false, false);
  a = t[0];
  b = t[1];
}

// Fragment of the 32 values whose results lie in two tiles: lane l holds the values 4 (l / 16) + 0..3
// of tile 0 in (p0, p1), of tile 1 in (q0, q1), as BF16 pairs.
__device__ __forceinline__ uint4 to_frag(uint32_t p0, uint32_t p1, uint32_t q0, uint32_t q1) {
  interleave(p0, q0);
  interleave(p1, q1);
  return make_uint4(p0, p1, q0, q1);
}

// Fragment f of the weights for lane l, from the FP32 blob.
__device__ __forceinline__ uint4 weight_frag(const float* __restrict__ prm, int f, int l) {
  const int lr = l & 15, lg = l >> 4;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = 0.0f;
  if (f < F_W2) {
    const int n = 16 * ((f - F_W1) >> 1) + lr, k = 32 * (f & 1) + 8 * lg;
    if (k < IN)
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = prm[OFF_W1 + n * IN + k + j];
  } else if (f < F_W3) {
    const int n = 16 * ((f - F_W2) >> 2) + lr, k = 32 * (f & 3) + 8 * lg;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = prm[OFF_W2 + n * HID + k + j];
  } else if (f < F_FWD) {
    if (lr < OUT)
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = prm[OFF_W3 + lr * HID + 32 * (f & 3) + 8 * lg + j];
  } else {
    const int n = 16 * ((f - F_W2T) >> 2) + lr, k = 32 * (f & 3) + 8 * lg;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = prm[OFF_W2 + (k + j) * HID + n];
  }
  return pack8(v);
}
static_assert(F_W2 % 4 == 0 && F_W3 % 4 == 0 && F_W2T % 4 == 0, "the low bits of a fragment number are its step");

// Eight consecutive features of a row from k on (zero from IN on).
__device__ __forceinline__ uint4 row_frag(const float* __restrict__ row, int k) {
  if (k >= IN) return make_uint4(0, 0, 0, 0);
  const float4u a = *reinterpret_cast<const float4u*>(row + k), b = *reinterpret_cast<const float4u*>(row + k + 4);
  return make_uint4(pack2(a.x, a.y), pack2(a.z, a.w), pack2(b.x, b.y), pack2(b.z, b.w));
}

// ReLU(acc + bias) of four consecutive neurons as two BF16 pairs.
__device__ __forceinline__ uint2 relu4(const f32x4& acc, const float4& b) {
  return make_uint2(pack2(fmaxf(acc[0] + b.x, 0.0f), fmaxf(acc[1] + b.y, 0.0f)),
                    pack2(fmaxf(acc[2] + b.z, 0.0f), fmaxf(acc[3] + b.w, 0.0f)));
}

// One layer of NT tiles of 16 rows with 128 neurons: h = ReLU(W x + b) as fragments.
template <int NT, int KK>
__device__ __forceinline__ void layer(const uint4* __restrict__ w, const float* __restrict__ bias, const uint4 (*x)[KK],
                                      uint4 (*h)[4]) {
  const int l = threadIdx.x & 63, lg = l >> 4;
#pragma unroll
  for (int tp = 0; tp < 4; ++tp) {
    uint2 d[2][NT];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int t = 2 * tp + s;
      f32x4 acc[NT];
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const uint4 a = w[(t * KK + kk) * 64 + l];
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[n] = mfma(a, x[n][kk], acc[n]);
      }
      const float4 b = *reinterpret_cast<const float4*>(bias + 16 * t + 4 * lg);
#pragma unroll
      for (int n = 0; n < NT; ++n) d[s][n] = relu4(acc[n], b);
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) h[n][tp] = to_frag(d[0][n].x, d[0][n].y, d[1][n].x, d[1][n].y);
    // keeps the compiler from loading the next tiles' weights ahead of time, which spills at 128 VGPRs
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Orders the LDS accesses of a wavefront that shares data between its own lanes only.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- Inference ----
// A wavefront takes 32 rows at a time through the whole network; 16 wavefronts share the weights (52 KB
// of LDS, staged once per block). Per 32 rows it reads 52 KB of fragments (416 cycles of the CU's
// LDS) for 104 MFMAs (1,664 cycles of one of its four SIMDs), so neither waits for the other; the
// rows' 6 KB come from memory. 1M rows in the kernel that kept activations in LDS (64 rows per
// block of 4 wavefronts, 93 KB: one wavefront per SIMD, a barrier per layer): 800 us, and 137 us
// to write the features; this one forms them itself and takes 87 us in all.
constexpr int kFwdBlock = 1024;
constexpr int kFwdWaves = kFwdBlock / 64;
constexpr int kFwdRows = 32;
constexpr int kXStride = 72;  // u16 per LDS feature row: 64 and a pad that spreads the rows over the banks

// Rows given as features (X) or, ANCHORS, as the neighbour lists of dwg_features (the same
// arithmetic, formed row tile by row tile in LDS instead of 192 bytes per row through memory).
template <bool ANCHORS>
__global__ __launch_bounds__(kFwdBlock) void k_mlp_fwd(const float* __restrict__ prm, const float* __restrict__ X,
                                                       AnchorRows ar, int64_t B, float* __restrict__ Y, int64_t sr,
                                                       int64_t sc) {
  __shared__ uint4 wf[F_FWD * 64];
  __shared__ __align__(16) float bias[2 * HID + 4];
  __shared__ __align__(16) u16 xt_all[ANCHORS ? kFwdWaves * kFwdRows * kXStride : 8];
  const int t = threadIdx.x, l = t & 63, wv = t >> 6, lr = l & 15, lg = l >> 4;
  for (int i = t; i < F_FWD * 64; i += kFwdBlock) wf[i] = weight_frag(prm, i >> 6, i & 63);
  for (int i = t; i < 2 * HID + OUT; i += kFwdBlock)
    bias[i] = i < HID ? prm[OFF_B1 + i] : (i < 2 * HID ? prm[OFF_B2 + i - HID] : prm[OFF_B3 + i - 2 * HID]);
  u16* const xt = xt_all + (ANCHORS ? wv * kFwdRows * kXStride : 0);
  if (ANCHORS)  // inputs 48-63 stay zero
    for (int i = l; i < kFwdRows * 8; i += 64) *reinterpret_cast<uint32_t*>(xt + (i >> 3) * kXStride + IN + 2 * (i & 7)) = 0u;
  __syncthreads();
  const int64_t tiles = (B + kFwdRows - 1) / kFwdRows;
  for (int64_t tile = (int64_t)wv * gridDim.x + blockIdx.x; tile < tiles; tile += (int64_t)gridDim.x * kFwdWaves) {
    const int64_t row0 = tile * kFwdRows;
    uint4 x[2][2];
    if (ANCHORS) {
#pragma unroll
      for (int u = 0; u < kFwdRows * DWG_FEAT_K / 64; ++u) {  // one (row, neighbour) pair per lane
        const int r = u * 4 + lg;
        const int64_t row = min(row0 + r, B - 1), o = ar.q0 + row;
        const float4 a = ar.A4[ar.idx[row * DWG_FEAT_K + lr]];
        const float is = ar.inv[row];
        const float f0 = (a.x - ar.P[o]) * is, f1 = (a.y - ar.P[ar.n + o]) * is, f2 = (a.z - ar.P[2 * ar.n + o]) * is;
        u16* const to = xt + r * kXStride + 3 * lr;
        const uint32_t p01 = pack2(f0, f1), p2 = pack2(f2, 0.0f);
        to[0] = (u16)p01;
        to[1] = (u16)(p01 >> 16);
        to[2] = (u16)p2;
      }
      wave_lds_fence();
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
          x[n][kk] = *reinterpret_cast<const uint4*>(xt + (16 * n + lr) * kXStride + 32 * kk + 8 * lg);
      wave_lds_fence();
    } else {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const float* row = X + min(row0 + 16 * n + lr, B - 1) * IN;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) x[n][kk] = row_frag(row, 32 * kk + 8 * lg);
      }
    }
    uint4 h1[2][4], h2[2][4];
    layer<2, 2>(wf + F_W1 * 64, bias, x, h1);
    layer<2, 4>(wf + F_W2 * 64, bias + HID, h1, h2);
    f32x4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint4 a = wf[(F_W3 + kk) * 64 + l];
#pragma unroll
      for (int n = 0; n < 2; ++n) y[n] = mfma(a, h2[n][kk], y[n]);
    }
    if (lg == 0) {  // the three outputs of row lr
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int64_t g = row0 + 16 * n + lr;
        if (g >= B) continue;
        const float y0 = y[n][0] + bias[2 * HID], y1 = y[n][1] + bias[2 * HID + 1], y2 = y[n][2] + bias[2 * HID + 2];
        const float nr = sqrtf(y0 * y0 + y1 * y1 + y2 * y2);
        const float inv = 1.0f / fmaxf(nr, 1e-30f);
        Y[g * sr] = y0 * inv;
        Y[g * sr + sc] = y1 * inv;
        Y[g * sr + 2 * sc] = y2 * inv;
      }
    }
  }
}

// ---- Training ----
constexpr int kTrainRows = 128;  // rows per block: 4 wavefronts of 32
constexpr int kPrepFragBlocks = F_ALL * 64 / 256;
constexpr int kMaskBlocks = 64;  // most blocks counting the mask
constexpr int64_t kMaskTile = 8192;
static_assert(F_ALL * 64 % 256 == 0, "whole blocks of fragments");

// Weight fragments for the step's blocks and the number of kept rows, as one count per block.
__global__ __launch_bounds__(256) void k_train_prep(const float* __restrict__ prm, const uint8_t* __restrict__ mask,
                                                    int64_t B, uint4* __restrict__ frags, int* __restrict__ cnt) {
  __shared__ int red[4];
  const int t = threadIdx.x;
  if (blockIdx.x < kPrepFragBlocks) {
    const int i = blockIdx.x * 256 + t;
    frags[i] = weight_frag(prm, i >> 6, i & 63);
    return;
  }
  const int b = blockIdx.x - kPrepFragBlocks, nb = gridDim.x - kPrepFragBlocks;
  int c = 0;
  for (int64_t i = (int64_t)b * 256 + t; i < B; i += (int64_t)nb * 256) c += mask[i] != 0;
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((t & 63) == 0) red[t >> 6] = c;
  __syncthreads();
  if (t == 0) cnt[b] = red[0] + red[1] + red[2] + red[3];
}

struct TrainLds {
  uint4 w1[16 * 64], w2[32 * 64], w2t[32 * 64];  // 80 KB
  uint4 ex[4][16][64];                           // 64 KB: fragments that the wavefronts share
  float db2[4][HID], db1[4][HID], dw3[4][OUT][HID], db3[4][OUT];
  __align__(16) float b1[HID], b2[HID], w3[OUT][HID];
  double loss[4];
};
static_assert(sizeof(TrainLds) <= 160 * 1024, "LDS budget");

// Sum over the four lanes l % 16 + 16 g.
__device__ __forceinline__ float sum_groups(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// Forward + backward of 128 rows; writes the block's partial gradient (FP32) and partial loss sum
// (as float) to part[block][NPART]. A wavefront takes its 32 rows through both passes in
// registers. The products over rows (dW1, dW2) need fragments of 32 consecutive rows per neuron:
// those come, by the same register swaps, from each layer computed once more with the rows as
// operand A (D then holds four consecutive rows of one neuron), which costs fewer cycles than
// reading strided 16-bit values from LDS. The four wavefronts exchange these fragments through
// LDS, and each accumulates a quarter of the gradient tiles over the block's 128 rows.
// One wavefront per SIMD (160 KB of LDS per block): bound by the chain of the passes and the staging of
// 80 KB of weights. 8,192 rows (64 blocks): 27 us, against 108 us with the activations in LDS and
// db1 summed by 4,096 scalar products per thread; the whole step 146 -> 36 us.
__global__ __launch_bounds__(256) void k_mlp_train(const float* __restrict__ prm, const uint4* __restrict__ frags,
                                                   const int* __restrict__ cnt, int ncnt,
                                                   const float* __restrict__ X, const float* __restrict__ T,
                                                   const uint8_t* __restrict__ mask, int64_t B,
                                                   float* __restrict__ part) {
  __shared__ TrainLds s;
  const int t = threadIdx.x, l = t & 63, w = t >> 6, lr = l & 15, lg = l >> 4;
  for (int i = t; i < 16 * 64; i += 256) s.w1[i] = frags[F_W1 * 64 + i];
  for (int i = t; i < 32 * 64; i += 256) s.w2[i] = frags[F_W2 * 64 + i];
  for (int i = t; i < 32 * 64; i += 256) s.w2t[i] = frags[F_W2T * 64 + i];
  if (t < HID) {
    s.b1[t] = prm[OFF_B1 + t];
    s.b2[t] = prm[OFF_B2 + t];
  }
  for (int i = t; i < OUT * HID; i += 256) (&s.w3[0][0])[i] = bf16_lo(pack2(prm[OFF_W3 + i], 0.0f));
  int nk = 0;
  if (mask) {
    nk = l < ncnt ? cnt[l] : 0;
    for (int o = 32; o > 0; o >>= 1) nk += __shfl_xor(nk, o, 64);
  } else {
    nk = (int)B;
  }
  const float inv_nk = 1.0f / (float)max(nk, 1);
  const int64_t row0 = (int64_t)blockIdx.x * kTrainRows + 32 * w;
  const uint4 zero = make_uint4(0, 0, 0, 0);
  uint4 x[2][2], xb[3];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int64_t g = row0 + 16 * n + lr;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) x[n][kk] = g < B ? row_frag(X + g * IN, 32 * kk + 8 * lg) : zero;
  }
#pragma unroll
  for (int f = 0; f < 3; ++f) {  // feature 16 f + lr of the rows 8 lg + j
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t g = row0 + 8 * lg + j;
      v[j] = g < B ? X[g * IN + 16 * f + lr] : 0.0f;
    }
    xb[f] = pack8(v);
  }
  __syncthreads();

  // forward
  uint4 h1[2][4], h2[2][4];
  layer<2, 2>(s.w1, s.b1, x, h1);
  layer<2, 4>(s.w2, s.b2, h1, h2);
  f32x4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const uint4 a = frags[(F_W3 + kk) * 64 + l];
#pragma unroll
    for (int n = 0; n < 2; ++n) y[n] = mfma(a, h2[n][kk], y[n]);
  }

  // d loss / d y = -(t - <yhat,t> yhat) / |y| / nk for kept rows (row lr, in the lanes lg == 0)
  float dy[2][3];
  double lossv = 0.0;
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int64_t g = row0 + 16 * n + lr;
    const bool keep = lg == 0 && g < B && (!mask || mask[g] != 0);
    float d0 = 0.f, d1 = 0.f, d2 = 0.f;
    if (keep) {
      const float y0 = y[n][0] + prm[OFF_B3], y1 = y[n][1] + prm[OFF_B3 + 1], y2 = y[n][2] + prm[OFF_B3 + 2];
      const float nr = fmaxf(sqrtf(y0 * y0 + y1 * y1 + y2 * y2), 1e-30f);
      const float e0 = y0 / nr, e1 = y1 / nr, e2 = y2 / nr;
      const float t0 = T[g * 3], t1 = T[g * 3 + 1], t2 = T[g * 3 + 2];
      const float cs = e0 * t0 + e1 * t1 + e2 * t2;
      lossv += 1.0 - (double)cs;
      const float f = -inv_nk / nr;
      d0 = f * (t0 - cs * e0);
      d1 = f * (t1 - cs * e1);
      d2 = f * (t2 - cs * e2);
    }
    dy[n][0] = __shfl(d0, lr, 64);
    dy[n][1] = __shfl(d1, lr, 64);
    dy[n][2] = __shfl(d2, lr, 64);
  }
  for (int o = 8; o > 0; o >>= 1) lossv += __shfl_xor(lossv, o, 64);
  if (l == 0) s.loss[w] = lossv;
#pragma unroll
  for (int c = 0; c < OUT; ++c) {
    float v = dy[0][c] + dy[1][c];
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (l == 0) s.db3[w][c] = v;
  }
  float dr[2][4][3];  // dy of the rows 4 lg + i
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < OUT; ++c) dr[n][i][c] = __shfl(dy[n][c], 4 * lg + i, 64);

  // dz2 = (dy W3) * [h2 > 0] as fragments of 32 neurons per row
  uint4 z2[2][4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    float w3[3][8];
#pragma unroll
    for (int c = 0; c < OUT; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) w3[c][j] = s.w3[c][32 * kk + 8 * lg + j];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const uint32_t m[4] = {h2[n][kk].x, h2[n][kk].y, h2[n][kk].z, h2[n][kk].w};
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = dy[n][0] * w3[0][j] + dy[n][1] * w3[1][j] + dy[n][2] * w3[2][j];
        const bool on = (j & 1) ? (m[j >> 1] >> 16) != 0u : (m[j >> 1] & 0xffffu) != 0u;
        v[j] = on ? v[j] : 0.0f;
      }
      z2[n][kk] = pack8(v);
    }
  }

  // layer 1 with the rows as A: h1 as fragments of 32 rows per neuron, and its signs
  uint64_t on1 = 0;
#pragma unroll
  for (int tn = 0; tn < 8; ++tn) {
    const float b = s.b1[16 * tn + lr];
    uint2 d[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) acc = mfma(x[n][kk], s.w1[(tn * 2 + kk) * 64 + l], acc);
      d[n] = relu4(acc, make_float4(b, b, b, b));
      const uint32_t bits = ((d[n].x & 0xffffu) ? 1u : 0u) | ((d[n].x >> 16) ? 2u : 0u) | ((d[n].y & 0xffffu) ? 4u : 0u) |
                            ((d[n].y >> 16) ? 8u : 0u);
      on1 |= (uint64_t)bits << (8 * tn + 4 * n);
    }
    s.ex[w][8 + tn][l] = to_frag(d[0].x, d[0].y, d[1].x, d[1].y);
  }

  // layer 2 with the rows as A: dW3 and db2 sums (FP32), dz2 as fragments of 32 rows per neuron
#pragma unroll
  for (int tn = 0; tn < 8; ++tn) {
    const int k = 16 * tn + lr;
    const float b = s.b2[k], w30 = s.w3[0][k], w31 = s.w3[1][k], w32 = s.w3[2][k];
    float g0 = 0.f, g1 = 0.f, g2 = 0.f, bsum = 0.f;
    uint2 d[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc = mfma(h1[n][kk], s.w2[(tn * 4 + kk) * 64 + l], acc);
      const uint2 hp = relu4(acc, make_float4(b, b, b, b));
      const float h[4] = {bf16_lo(hp.x), bf16_hi(hp.x), bf16_lo(hp.y), bf16_hi(hp.y)};
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        g0 = fmaf(dr[n][i][0], h[i], g0);
        g1 = fmaf(dr[n][i][1], h[i], g1);
        g2 = fmaf(dr[n][i][2], h[i], g2);
        v[i] = dr[n][i][0] * w30 + dr[n][i][1] * w31 + dr[n][i][2] * w32;
        v[i] = h[i] != 0.0f ? v[i] : 0.0f;
        bsum += v[i];
      }
      d[n] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
    }
    s.ex[w][tn][l] = to_frag(d[0].x, d[0].y, d[1].x, d[1].y);
    g0 = sum_groups(g0);
    g1 = sum_groups(g1);
    g2 = sum_groups(g2);
    bsum = sum_groups(bsum);
    if (lg == 0) {
      s.dw3[w][0][k] = g0;
      s.dw3[w][1][k] = g1;
      s.dw3[w][2][k] = g2;
      s.db2[w][k] = bsum;
    }
  }

  // dz1 = (dz2 W2) * [h1 > 0]: db1 sums (FP32) and fragments of 32 rows per neuron
  uint4 z1[8];
#pragma unroll
  for (int tn = 0; tn < 8; ++tn) {
    float bsum = 0.f;
    uint2 d[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc = mfma(z2[n][kk], s.w2t[(tn * 4 + kk) * 64 + l], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[i] = (on1 >> (8 * tn + 4 * n + i)) & 1u ? acc[i] : 0.0f;
        bsum += acc[i];
      }
      d[n] = make_uint2(pack2(acc[0], acc[1]), pack2(acc[2], acc[3]));
    }
    z1[tn] = to_frag(d[0].x, d[0].y, d[1].x, d[1].y);
    bsum = sum_groups(bsum);
    if (lg == 0) s.db1[w][16 * tn + lr] = bsum;
  }
  __syncthreads();

  float* out = part + (int64_t)blockIdx.x * NPART;
  // dW2[m][n] = sum_r dz2[r][m] h1[r][n]: 8 x 8 tiles, 16 per wavefront, 128 rows
#pragma unroll
  for (int mt = 2 * w; mt < 2 * w + 2; ++mt) {
    uint4 a[4];
#pragma unroll
    for (int kw = 0; kw < 4; ++kw) a[kw] = s.ex[kw][mt][l];
#pragma unroll
    for (int tn = 0; tn < 8; ++tn) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kw = 0; kw < 4; ++kw) acc = mfma(a[kw], s.ex[kw][8 + tn][l], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) out[OFF_W2 + (16 * mt + 4 * lg + i) * HID + 16 * tn + lr] = acc[i];
    }
  }
  for (int i = t; i < OUT * HID; i += 256) {
    const int c = i / HID, k = i % HID;
    out[OFF_W3 + i] = (s.dw3[0][c][k] + s.dw3[1][c][k]) + (s.dw3[2][c][k] + s.dw3[3][c][k]);
  }
  if (t < HID) {
    out[OFF_B2 + t] = (s.db2[0][t] + s.db2[1][t]) + (s.db2[2][t] + s.db2[3][t]);
    out[OFF_B1 + t] = (s.db1[0][t] + s.db1[1][t]) + (s.db1[2][t] + s.db1[3][t]);
  } else if (t < HID + OUT) {
    const int c = t - HID;
    out[OFF_B3 + c] = (s.db3[0][c] + s.db3[1][c]) + (s.db3[2][c] + s.db3[3][c]);
  } else if (t == HID + OUT) {
    out[NPAR] = (float)((s.loss[0] + s.loss[1]) + (s.loss[2] + s.loss[3]));
  }
  __syncthreads();  // every wavefront has read the shared fragments
#pragma unroll
  for (int tn = 0; tn < 8; ++tn) s.ex[w][tn][l] = z1[tn];
#pragma unroll
  for (int f = 0; f < 3; ++f) s.ex[w][8 + f][l] = xb[f];
  __syncthreads();
  // dW1[m][n] = sum_r dz1[r][m] x[r][n], n < 48: 8 x 3 tiles, 6 per wavefront
#pragma unroll
  for (int mt = 2 * w; mt < 2 * w + 2; ++mt)
#pragma unroll
    for (int f = 0; f < 3; ++f) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kw = 0; kw < 4; ++kw) acc = mfma(s.ex[kw][mt][l], s.ex[kw][8 + f][l], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) out[OFF_W1 + (16 * mt + 4 * lg + i) * IN + 16 * f + lr] = acc[i];
    }
}

// Fixed-order sum of the per-block partials (four Kahan sums over every fourth block, eight loads in
// flight each, then their sum): grad[p] = sum_b part[b][p], loss = sum / nk; then Adam with bias
// correction (beta1 0.9, beta2 0.999, eps 1e-8) on the FP32 master weights.
__global__ __launch_bounds__(256) void k_reduce_adam(const float* __restrict__ part, int nblk,
                                                     const int* __restrict__ cnt, int ncnt, int64_t B,
                                                     float* __restrict__ prm, float* __restrict__ m1,
                                                     float* __restrict__ m2, float lr, float bc1, float bc2,
                                                     float* __restrict__ gout, float* __restrict__ loss) {
  __shared__ float red[4][64];
  const int p = blockIdx.x * 64 + (threadIdx.x & 63), seg = threadIdx.x >> 6;
  float s = 0.f, c = 0.f;
  if (p <= NPAR) {
    for (int b0 = seg; b0 < nblk; b0 += 32) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = b0 + 4 * u < nblk ? part[(int64_t)(b0 + 4 * u) * NPART + p] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float y = x[u] - c;
        const float tt = s + y;
        c = (tt - s) - y;
        s = tt;
      }
    }
  }
  red[seg][threadIdx.x & 63] = s - c;
  __syncthreads();
  if (seg != 0 || p > NPAR) return;
  const int q = threadIdx.x & 63;
  const float gi = (red[0][q] + red[1][q]) + (red[2][q] + red[3][q]);
  if (p == NPAR) {
    if (!loss) return;
    int nk = 0;
    for (int i = 0; i < ncnt; ++i) nk += cnt[i];
    if (ncnt == 0) nk = (int)B;
    *loss = gi / (float)max(nk, 1);
    return;
  }
  const float a = 0.9f * m1[p] + 0.1f * gi;
  const float b = 0.999f * m2[p] + 0.001f * gi * gi;
  m1[p] = a;
  m2[p] = b;
  prm[p] -= lr * (a / bc1) / (sqrtf(b / bc2) + 1e-8f);
  if (gout) gout[p] = gi;
}

// Blocks of the inference kernel: one per CU (its LDS leaves room for one), fewer when there are
// fewer tiles of 32 rows.
constexpr int64_t kFwdBlocks = 256;

}  // namespace

size_t mlp_ws_bytes(int64_t B) {
  Carver c(nullptr);
  c.take<float>((size_t)cdiv(B, kTrainRows) * NPART);
  c.take<uint4>((size_t)F_ALL * 64);
  c.take<int>(kMaskBlocks);
  return c.used;
}

dwg_status mlp_infer_run(const float* params, const float* X, int64_t B, float* Y, hipStream_t stream) {
  hipLaunchKernelGGL((k_mlp_fwd<false>), dim3((unsigned)std::min<int64_t>(cdiv(B, kFwdRows), kFwdBlocks)),
                     dim3(kFwdBlock), 0, stream, params, X, AnchorRows{}, B, Y, (int64_t)3, (int64_t)1);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mlp_anchor_normals(const float* params, const AnchorRows& rows, int64_t B, float* N, int64_t n,
                              hipStream_t stream) {
  hipLaunchKernelGGL((k_mlp_fwd<true>), dim3((unsigned)std::min<int64_t>(cdiv(B, kFwdRows), kFwdBlocks)),
                     dim3(kFwdBlock), 0, stream, params, static_cast<const float*>(nullptr), rows, B, N, (int64_t)1, n);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mlp_train_run(float* params, float* m1, float* m2, int64_t step, float lr, const float* X,
                         const float* T, const uint8_t* mask, int64_t B, float* grad_out, float* loss_out,
                         void* ws, hipStream_t stream) {
  const int nblk = (int)cdiv(B, kTrainRows);
  Carver c(ws);
  float* part = c.take<float>((size_t)nblk * NPART);
  uint4* frags = c.take<uint4>((size_t)F_ALL * 64);
  int* cnt = c.take<int>(kMaskBlocks);
  const int ncnt = mask ? (int)std::min<int64_t>(cdiv(B, kMaskTile), kMaskBlocks) : 0;
  hipLaunchKernelGGL(k_train_prep, dim3(kPrepFragBlocks + ncnt), dim3(256), 0, stream, params, mask, B, frags, cnt);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_mlp_train, dim3(nblk), dim3(256), 0, stream, params, frags, cnt, ncnt, X, T, mask, B, part);
  DWG_TRY_LAUNCH();
  const float bc1 = 1.0f - powf(0.9f, (float)step);
  const float bc2 = 1.0f - powf(0.999f, (float)step);
  hipLaunchKernelGGL(k_reduce_adam, dim3((unsigned)cdiv(NPAR + 1, 64)), dim3(256), 0, stream, part, nblk, cnt, ncnt, B,
                     params, m1, m2, lr, bc1, bc2, grad_out, loss_out);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

}  // namespace dwg
