// Radix sort of (key, value) pairs, and the spatial order of the points for the all-pairs kernel.
//
// Spatial order: sort key = (radius class, Morton code of the point's cell in a 128^3 grid over the
// bounding box). Radius class 1 holds points whose kernel radius max(delta, eps) exceeds 4 x the
// mean radius (outliers, sparse regions): grouped at the end, their large radii do not spoil the
// near/far test of the tiles of dense surface points. The (key, index) pairs go through the
// stable LSD radix sort (3 passes of 8 bits over the 22-bit key): equal keys keep ascending
// indices, so the permutation is deterministic, and the cost is linear in n whatever the
// distribution (every point in one cell included). Up to kSortTile points, one block does all of it.
#include <cfloat>
#include <cmath>

#include "dwg_internal.h"

namespace dwg {
namespace {

// ---- LSD radix sort, 8 bits per pass ----
// One launch per pass instead of five (digit counts, a three-launch scan, scatter): the digit
// totals of every pass are counted up front in one sweep over the keys (a pass only permutes
// them), and within a pass each block publishes its tile's digit counts and adds up those of the
// tiles before it (chained scan with look-back after Merrill and Garland, 2016, one thread per digit). A pass over few tiles is a
// chain of device-scope round trips (ticket, counts, look-back): 24 -> 14 us for 20,011 64-bit
// keys; 1M keys 35 -> 25 us.
constexpr int kRsThreads = 512;
constexpr int kRsWaves = kRsThreads / 64;
constexpr int kRsItems = 8;                        // per thread
constexpr int kRsTile = kRsThreads * kRsItems;     // a wavefront holds 512 consecutive elements
constexpr int kRsMaxPasses = 8;
constexpr int kRsHistBlocks = 256;
constexpr int kSortTile = kRsTile;

// Work area (ints): totals [kRsMaxPasses][256], tickets [kRsMaxPasses], then two buffers of tile states
// [tiles][256] (64-bit words: flag << 32 | count), used in turn: each pass clears the next one's.
constexpr int kRsHead = kRsMaxPasses * 256 + kRsMaxPasses;
static_assert(kRsHead % 2 == 0, "tile states are 64-bit words");

constexpr unsigned long long kCount = 1ull << 32, kPrefix = 2ull << 32;

__global__ void k_rs_clear(int32_t* __restrict__ work, int64_t words) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x)
    work[i] = 0;
}

template <class K>
__global__ __launch_bounds__(kRsThreads) void k_rs_totals(const K* __restrict__ key, int64_t n, int passes,
                                                          int32_t* __restrict__ total) {
  __shared__ int32_t h[kRsMaxPasses * 256];
  for (int i = threadIdx.x; i < passes * 256; i += kRsThreads) h[i] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * kRsThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRsThreads) {
    const K k = key[i];
    for (int p = 0; p < passes; ++p) atomicAdd(&h[p * 256 + (int)((k >> (8 * p)) & 255u)], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < passes * 256; i += kRsThreads)
    if (const int32_t c = h[i]) atomicAdd(&total[i], c);
}

// Lanes of the wavefront (valid ones) whose digit equals this lane's.
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const bool on = (d >> bit) & 1u;
    const uint64_t b = __ballot(valid && on);
    peers &= on ? b : ~b;
  }
  return peers;
}

// Ranks of a wavefront's elements among those with the same digit in its earlier elements (item
// major, then lane), counted in its 256 LDS counters (zero before).
template <int ITEMS>
__device__ __forceinline__ void rank_items(const uint32_t* digit, int count, volatile int32_t* cnt, int* rank) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const bool valid = j * 64 + lane < count;
    const uint64_t peers = same_digit(digit[j], valid);
    if (valid) {
      const int before = cnt[digit[j]];
      rank[j] = before + __popcll(peers & lt);
      if ((peers & lt) == 0ull) cnt[digit[j]] = before + __popcll(peers);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Exclusive scan of 256 values by threads 0..255 of the block (others pass 0 and ignore the result).
__device__ __forceinline__ int32_t scan256(int32_t v, int32_t* lds4) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int32_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  __syncthreads();
  if (wv < 4 && lane == 63) lds4[wv] = inc;
  __syncthreads();
  int32_t before = 0;
  for (int w = 0; w < 4; ++w) before += w < wv ? lds4[w] : 0;
  return before + inc - v;
}

// Where a pass reads an element's value: its position (kValIota) or the value array; kValNone
// sorts keys only.
enum ValMode { kValNone = 0, kValIota = 1, kValArray = 2 };

// One pass. Every wait ends: a block takes the next tile from a ticket counter and waits only for
// tiles with smaller tickets, whose blocks are running and publish their counts before they wait.
template <class K>
__global__ __launch_bounds__(kRsThreads) void k_rs_pass(const K* __restrict__ kin, const int32_t* __restrict__ vin,
                                                        int64_t n, int shift, int mode,
                                                        const int32_t* __restrict__ total, int32_t* __restrict__ ticket,
                                                        unsigned long long* __restrict__ state,
                                                        unsigned long long* __restrict__ next_state,
                                                        K* __restrict__ kout, int32_t* __restrict__ vout) {
  __shared__ int32_t cnt[kRsWaves][256];
  __shared__ int32_t lds4[4];
  __shared__ int32_t s_tile;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (t == 0) s_tile = atomicAdd(ticket, 1);
  for (int i = t; i < kRsWaves * 256; i += kRsThreads) (&cnt[0][0])[i] = 0;
  const int32_t base = scan256(t < 256 ? total[t] : 0, lds4);  // the barriers inside publish s_tile and cnt
  const int64_t tile = s_tile;
  const int64_t w0 = tile * kRsTile + (int64_t)wv * (64 * kRsItems);
  const int count = (int)(n - w0 < 64 * kRsItems ? (n > w0 ? n - w0 : 0) : 64 * kRsItems);
  K key[kRsItems];
  uint32_t digit[kRsItems];
  int rank[kRsItems];
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = j * 64 + lane;
    key[j] = i < count ? kin[w0 + i] : K(0);
    digit[j] = (uint32_t)(key[j] >> shift) & 255u;
  }
  rank_items<kRsItems>(digit, count, cnt[wv], rank);
  __syncthreads();
  if (t < 256) {
    int32_t c[kRsWaves], sum = 0;
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) {
      c[w] = cnt[w][t];
      sum += c[w];
    }
    unsigned long long* const mine = state + tile * 256 + t;
    next_state[tile * 256 + t] = 0ull;
    int32_t before = 0;
    if (tile > 0) {
      __hip_atomic_store(mine, kCount | (uint32_t)sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      constexpr int kBatch = 16;  // predecessors asked at once
      for (int64_t at = tile - 1;;) {
        unsigned long long v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          v[u] = at - u >= 0 ? __hip_atomic_load(state + (at - u) * 256 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                             : kPrefix;
        bool open = true, done = false;  // open: every earlier answer of the batch was known
        int used = 0;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const uint32_t flag = (uint32_t)(v[u] >> 32);
          open = open && flag != 0u && !done;
          if (open) {
            before += (int32_t)(uint32_t)v[u];
            ++used;
            done = flag == 2u;
          }
        }
        if (done) break;
        if (used == 0) __builtin_amdgcn_s_sleep(1);
        at -= used;
      }
    }
    __hip_atomic_store(mine, kPrefix | (uint32_t)(before + sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int32_t run = base + before;
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) {
      cnt[w][t] = run;
      run += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = j * 64 + lane;
    if (i >= count) continue;
    const int64_t pos = cnt[wv][digit[j]] + rank[j];
    kout[pos] = key[j];
    if (mode == kValIota) vout[pos] = (int32_t)(w0 + i);
    if (mode == kValArray) vout[pos] = vin[w0 + i];
  }
}

// All passes over at most kSortTile elements held by one block of kRsThreads: key[j], val[j] are
// elements wave * 512 + j * 64 + lane, in order on return. xk, xv: kSortTile LDS slots.
template <class K>
__device__ void block_sort(K* key, int32_t* val, int n, int bits, int32_t (*cnt)[256], int32_t* lds4, K* xk,
                           int32_t* xv) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int w0 = wv * (64 * kRsItems);
  const int count = n - w0 < 64 * kRsItems ? (n > w0 ? n - w0 : 0) : 64 * kRsItems;
  for (int shift = 0; shift < bits; shift += 8) {
    uint32_t digit[kRsItems];
    int rank[kRsItems];
    __syncthreads();
    for (int i = t; i < kRsWaves * 256; i += kRsThreads) (&cnt[0][0])[i] = 0;
#pragma unroll
    for (int j = 0; j < kRsItems; ++j) digit[j] = (uint32_t)(key[j] >> shift) & 255u;
    __syncthreads();
    rank_items<kRsItems>(digit, count, cnt[wv], rank);
    __syncthreads();
    int32_t sum = 0;
    if (t < 256)
      for (int w = 0; w < kRsWaves; ++w) sum += cnt[w][t];
    int32_t run = scan256(sum, lds4);
    if (t < 256)
      for (int w = 0; w < kRsWaves; ++w) {
        const int32_t c = cnt[w][t];
        cnt[w][t] = run;
        run += c;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRsItems; ++j)
      if (j * 64 + lane < count) {
        const int pos = cnt[wv][digit[j]] + rank[j];
        xk[pos] = key[j];
        xv[pos] = val[j];
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRsItems; ++j)
      if (j * 64 + lane < count) {
        key[j] = xk[w0 + j * 64 + lane];
        val[j] = xv[w0 + j * 64 + lane];
      }
  }
}

// Small arrays by one block (kout may be kin, vout vin).
template <class K>
__global__ __launch_bounds__(kRsThreads) void k_rs_block(const K* kin, const int32_t* vin,
                                                         int n, int bits, int mode, K* kout, int32_t* vout) {
  __shared__ int32_t cnt[kRsWaves][256];
  __shared__ int32_t lds4[4];
  __shared__ K xk[kSortTile];
  __shared__ int32_t xv[kSortTile];
  const int lane = threadIdx.x & 63, w0 = (threadIdx.x >> 6) * (64 * kRsItems);
  K key[kRsItems];
  int32_t val[kRsItems];
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = w0 + j * 64 + lane;
    key[j] = i < n ? kin[i] : K(0);
    val[j] = mode == kValArray && i < n ? vin[i] : i;
  }
  block_sort(key, val, n, bits, cnt, lds4, xk, xv);
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = w0 + j * 64 + lane;
    if (i >= n) continue;
    kout[i] = key[j];
    if (mode != kValNone) vout[i] = val[j];
  }
}

template <class K>
dwg_status radix_sort(K* const key[2], int32_t* const val[2], int mode, int64_t n, int bits, int32_t* work,
                      int* result, hipStream_t st) {
  const int passes = (bits + 7) / 8;
  if (passes > kRsMaxPasses || passes < 1) {
    set_error("internal: radix sort of %d bits", bits);
    return DWG_E_INVALID;
  }
  *result = passes & 1;
  if (n <= kSortTile) {
    hipLaunchKernelGGL((k_rs_block<K>), dim3(1), dim3(kRsThreads), 0, st, key[0], mode == kValArray ? val[0] : nullptr,
                       (int)n, bits, mode, key[*result], mode == kValNone ? nullptr : val[*result]);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  const int64_t tiles = cdiv(n, kRsTile);
  int32_t* const ticket = work + kRsMaxPasses * 256;
  unsigned long long* const state[2] = {reinterpret_cast<unsigned long long*>(work + kRsHead),
                                        reinterpret_cast<unsigned long long*>(work + kRsHead) + tiles * 256};
  const int64_t words = kRsHead + 2 * tiles * 256;  // totals, tickets and the first pass' states
  hipLaunchKernelGGL(k_rs_clear, dim3((unsigned)std::min<int64_t>(cdiv(words, 256), 1024)), dim3(256), 0, st, work, words);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL((k_rs_totals<K>), dim3((unsigned)std::min<int64_t>(cdiv(n, kRsThreads), kRsHistBlocks)),
                     dim3(kRsThreads), 0, st, key[0], n, passes, work);
  DWG_TRY_LAUNCH();
  for (int p = 0; p < passes; ++p) {
    const int a = p & 1, b = a ^ 1;
    const int m = mode == kValIota && p > 0 ? kValArray : mode;
    hipLaunchKernelGGL((k_rs_pass<K>), dim3((unsigned)tiles), dim3(kRsThreads), 0, st, key[a],
                       mode == kValNone ? nullptr : val[a], n, 8 * p, m, work + 256 * p, ticket + p, state[a], state[b],
                       key[b], mode == kValNone ? nullptr : val[b]);
    DWG_TRY_LAUNCH();
  }
  return DWG_OK;
}

// ---- Spatial order ----
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
  v &= 0x7fu;
  v = (v | (v << 8)) & 0x0000f00fu;
  v = (v | (v << 4)) & 0x000c30c3u;
  v = (v | (v << 2)) & 0x00249249u;
  return v;
}

__device__ __forceinline__ float radius_of(const float* D, int64_t j, float eps) {
  const float d = D ? D[j] : 0.0f;
  return d > eps ? d : eps;
}

// The frame of the sort keys: bounding box minimum, cells per unit, radius class threshold.
struct OrderFrame {
  float ox, oy, oz, sc, thr;
};

__device__ __forceinline__ OrderFrame order_frame(const float* box, float mean_radius) {
  const float ext = fmaxf(fmaxf(box[3] - box[0], box[4] - box[1]), fmaxf(box[5] - box[2], 1e-30f));
  return OrderFrame{box[0], box[1], box[2], 128.0f / ext, 4.0f * mean_radius};
}

__device__ __forceinline__ uint32_t order_key(const OrderFrame& f, float x, float y, float z, float radius) {
  const uint32_t cx = (uint32_t)min(max((int)((x - f.ox) * f.sc), 0), 127);
  const uint32_t cy = (uint32_t)min(max((int)((y - f.oy) * f.sc), 0), 127);
  const uint32_t cz = (uint32_t)min(max((int)((z - f.oz) * f.sc), 0), 127);
  const uint32_t cls = radius > f.thr ? 1u : 0u;
  return (cls << 21) | (spread3(cx) << 2) | (spread3(cy) << 1) | spread3(cz);
}

// Block-wide minimum of mn, maximum of mx (per axis) and sum of s: over the wavefronts by
// shuffles, then over LDS in order; valid in every thread.
constexpr int kOrderWaves = 16;
struct OrderLds {
  float red[6][kOrderWaves];
  double sum[kOrderWaves];
};
__device__ void block_extent(const float* mn, const float* mx, double s, OrderLds& lds, float* box, double* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  float lo[3] = {mn[0], mn[1], mn[2]}, hi[3] = {mx[0], mx[1], mx[2]};
  for (int o = 32; o > 0; o >>= 1) {
    for (int d = 0; d < 3; ++d) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, 64));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, 64));
    }
    s += __shfl_xor(s, o, 64);
  }
  __syncthreads();
  if (lane == 0) {
    for (int d = 0; d < 3; ++d) {
      lds.red[d][wv] = lo[d];
      lds.red[3 + d][wv] = hi[d];
    }
    lds.sum[wv] = s;
  }
  __syncthreads();
  double t = 0.0;
  for (int d = 0; d < 3; ++d) {
    lo[d] = lds.red[d][0];
    hi[d] = lds.red[3 + d][0];
  }
  for (int w = 0; w < nw; ++w) {
    for (int d = 0; d < 3; ++d) {
      lo[d] = fminf(lo[d], lds.red[d][w]);
      hi[d] = fmaxf(hi[d], lds.red[3 + d][w]);
    }
    t += lds.sum[w];
  }
  for (int d = 0; d < 3; ++d) {
    box[d] = lo[d];
    box[3 + d] = hi[d];
  }
  *total = t;
}

constexpr int kExtentBlocks = 256;

// Bounding box and sum of the radii, per block.
__global__ __launch_bounds__(256) void k_extent_partial(const float* __restrict__ P, int64_t n,
                                                        const float* __restrict__ D, float eps,
                                                        float* __restrict__ part, double* __restrict__ rpart) {
  __shared__ OrderLds lds;
  float mn[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, mx[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    for (int d = 0; d < 3; ++d) {
      const float v = P[d * n + i];
      mn[d] = fminf(mn[d], v);
      mx[d] = fmaxf(mx[d], v);
    }
    s += (double)radius_of(D, i, eps);
  }
  float box[6];
  double total;
  block_extent(mn, mx, s, lds, box, &total);
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = box[threadIdx.x];
  if (threadIdx.x == 0) rpart[blockIdx.x] = total;
}

// Keys of all points; every block first reduces the per-block extents (in the same order).
__global__ __launch_bounds__(256) void k_order_keys(const float* __restrict__ P, int64_t n, const float* __restrict__ D,
                                                    float eps, const float* __restrict__ part,
                                                    const double* __restrict__ rpart, int nparts,
                                                    uint32_t* __restrict__ key) {
  __shared__ OrderLds lds;
  float mn[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, mx[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
  double s = 0.0;
  for (int b = threadIdx.x; b < nparts; b += blockDim.x) {
    for (int d = 0; d < 3; ++d) {
      mn[d] = fminf(mn[d], part[b * 6 + d]);
      mx[d] = fmaxf(mx[d], part[b * 6 + 3 + d]);
    }
    s += rpart[b];
  }
  float box[6];
  double total;
  block_extent(mn, mx, s, lds, box, &total);
  const OrderFrame f = order_frame(box, (float)(total / (double)n));
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    key[i] = order_key(f, P[i], P[n + i], P[2 * n + i], radius_of(D, i, eps));
}

// The whole order of at most kSortTile points by one block.
__global__ __launch_bounds__(kRsThreads) void k_order_small(const float* __restrict__ P, int n,
                                                            const float* __restrict__ D, float eps,
                                                            int32_t* __restrict__ perm) {
  __shared__ OrderLds lds;
  __shared__ int32_t cnt[kRsWaves][256];
  __shared__ int32_t lds4[4];
  __shared__ uint32_t xk[kSortTile];
  __shared__ int32_t xv[kSortTile];
  const int lane = threadIdx.x & 63, w0 = (threadIdx.x >> 6) * (64 * kRsItems);
  float mn[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, mx[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
  float x[kRsItems][3], r[kRsItems];
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = w0 + j * 64 + lane;
    r[j] = x[j][0] = x[j][1] = x[j][2] = 0.0f;
    if (i >= n) continue;
    for (int d = 0; d < 3; ++d) {
      x[j][d] = P[d * n + i];
      mn[d] = fminf(mn[d], x[j][d]);
      mx[d] = fmaxf(mx[d], x[j][d]);
    }
    r[j] = radius_of(D, i, eps);
    s += (double)r[j];
  }
  float box[6];
  double total;
  block_extent(mn, mx, s, lds, box, &total);
  const OrderFrame f = order_frame(box, (float)(total / (double)n));
  uint32_t key[kRsItems];
  int32_t val[kRsItems];
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    key[j] = order_key(f, x[j][0], x[j][1], x[j][2], r[j]);
    val[j] = w0 + j * 64 + lane;
  }
  block_sort(key, val, n, kSortKeyBits, cnt, lds4, xk, xv);
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = w0 + j * 64 + lane;
    if (i < n) perm[i] = val[j];
  }
}

unsigned grid_n(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, 256), 2048)); }

}  // namespace

size_t radix_work_len(int64_t n) { return (size_t)(kRsHead + 4 * 256 * cdiv(n, kRsTile)); }

dwg_status radix_sort_pairs(uint64_t* const key[2], int32_t* const val[2], bool iota, int64_t n, int bits,
                            int32_t* work, int* result, hipStream_t st) {
  return radix_sort<uint64_t>(key, val, iota ? kValIota : kValArray, n, bits, work, result, st);
}

dwg_status radix_sort_keys(uint64_t* const key[2], int64_t n, int bits, int32_t* work, int* result, hipStream_t st) {
  return radix_sort<uint64_t>(key, nullptr, kValNone, n, bits, work, result, st);
}

size_t carve_sort(Carver& c, int64_t n, SortWork* out) {
  const size_t s0 = c.used;
  SortWork w;
  w.part = c.take<float>(kBboxParts);
  w.rpart = c.take<double>(kExtentBlocks);
  w.key[0] = c.take<uint32_t>((size_t)n);
  w.key[1] = c.take<uint32_t>((size_t)n);
  w.val = c.take<int32_t>((size_t)n);
  w.work = c.take<int32_t>(radix_work_len(n));
  if (out) *out = w;
  return c.used - s0;
}

dwg_status spatial_sort(const float* P, int64_t n, const float* delta, float eps, const SortWork& w,
                        int32_t* perm, hipStream_t st) {
  if (n <= kSortTile) {
    hipLaunchKernelGGL(k_order_small, dim3(1), dim3(kRsThreads), 0, st, P, (int)n, delta, eps, perm);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  const int nb = (int)std::min<int64_t>(cdiv(n, 256), kExtentBlocks);
  hipLaunchKernelGGL(k_extent_partial, dim3(nb), dim3(256), 0, st, P, n, delta, eps, w.part, w.rpart);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_order_keys, dim3(grid_n(n)), dim3(256), 0, st, P, n, delta, eps, w.part, w.rpart, nb, w.key[0]);
  DWG_TRY_LAUNCH();
  // three passes (a 22-bit key) leave the sorted pairs in the second buffers: perm
  static_assert((kSortKeyBits + 7) / 8 == 3, "an odd number of passes ends in the second buffers");
  int32_t* const vals[2] = {w.val, perm};
  int res = 0;
  return radix_sort<uint32_t>(w.key, vals, kValIota, n, kSortKeyBits, w.work, &res, st);
}

}  // namespace dwg
