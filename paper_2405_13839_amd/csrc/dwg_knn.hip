// Exact k-nearest-neighbour search on a uniform grid, the kernel radius delta (Sec. 5.2
// "Poisson Kernels": mean distance to the k nearest neighbours) and the k = 16 anchor
// features of the learned initial normals.
//
// Grid build: the box is the range of a stratified sample of at most kSample points (all of them
// below that), trimmed per axis to the sample's quantiles 1/1024 and 1 - 1/1024; the cell size
// is the one at which a point is expected to share its cell with kCellShare * k others, from
// the sample's pair counts on two coarse grids (k_grid_setup); counting sort of the reference
// points by cell (atomic ranks; the order inside a cell is arbitrary, which is harmless because
// candidates are ranked by the pair (squared distance, index)). Points outside the trimmed
// box sit in its border cells: a few points far from the rest then do not stretch the
// cells until the whole cloud shares one, and the search stays exact because projecting
// onto a box shortens no distance (see k_knn). Query: the 27 cells around the query's own, then
// Chebyshev rings of cells, a row of cells (one contiguous range of the sorted
// points) at a time, keeping the k best candidates in registers, until the k-th best
// distance is below the distance to the faces of the searched cube. One thread per query takes
// rings up to kFirstPassRings; the few queries still unfinished (isolated points) are then
// searched by a wavefront each (k_knn, k_knn_wave).
#include <cfloat>
#include <climits>
#include <cmath>

#include "dwg_internal.h"

namespace dwg {
namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;  // elements per thread of the tiled scan
constexpr int kScanTile = kScanBlock * kScanItems;
constexpr int kScanOneBlock = 1024;   // threads of the one-block scan
constexpr int64_t kScanOneMax = 8192; // longest array of the one-block scan (two of its rounds)

__global__ __launch_bounds__(256) void k_bbox_partial(const float* __restrict__ R, int64_t n,
                                                      float* __restrict__ part) {
  __shared__ float lds[6][256];
  float mn[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, mx[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    for (int d = 0; d < 3; ++d) {
      const float v = R[d * n + i];
      mn[d] = fminf(mn[d], v);
      mx[d] = fmaxf(mx[d], v);
    }
  }
  for (int d = 0; d < 3; ++d) {
    lds[d][threadIdx.x] = mn[d];
    lds[3 + d][threadIdx.x] = mx[d];
  }
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int d = 0; d < 3; ++d) {
        lds[d][threadIdx.x] = fminf(lds[d][threadIdx.x], lds[d][threadIdx.x + s]);
        lds[3 + d][threadIdx.x] = fmaxf(lds[3 + d][threadIdx.x], lds[3 + d][threadIdx.x + s]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = lds[threadIdx.x][0];
}

// Minimum and maximum per axis of the nblocks per-block partials, by one block of 256
// threads (min and max are exact in any order): v6 = (min x, min y, min z, max x, ...).
__device__ void reduce_bbox_parts(const float* __restrict__ part, int nblocks, float (*lds)[256], float* v6) {
  float v[6] = {FLT_MAX, FLT_MAX, FLT_MAX, -FLT_MAX, -FLT_MAX, -FLT_MAX};
  for (int b = threadIdx.x; b < nblocks; b += blockDim.x)
    for (int d = 0; d < 3; ++d) {
      v[d] = fminf(v[d], part[b * 6 + d]);
      v[3 + d] = fmaxf(v[3 + d], part[b * 6 + 3 + d]);
    }
  for (int d = 0; d < 6; ++d) lds[d][threadIdx.x] = v[d];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int d = 0; d < 3; ++d) {
        lds[d][threadIdx.x] = fminf(lds[d][threadIdx.x], lds[d][threadIdx.x + st]);
        lds[3 + d][threadIdx.x] = fmaxf(lds[3 + d][threadIdx.x], lds[3 + d][threadIdx.x + st]);
      }
    __syncthreads();
  }
  for (int d = 0; d < 6; ++d) v6[d] = lds[d][0];
}

// Final bounding box: out6 = (min x, min y, min z, max x, max y, max z). One block of 256.
__global__ __launch_bounds__(256) void k_bbox_final(const float* __restrict__ part, int nblocks,
                                                    float* __restrict__ out6) {
  __shared__ float lds[6][256];
  float v6[6];
  reduce_bbox_parts(part, nblocks, lds, v6);
  if (threadIdx.x < 6) out6[threadIdx.x] = v6[threadIdx.x];
}

// ---- Grid setup ----
constexpr int kSetupBlock = 1024;
// Points the grid is laid out from (4,096: areas of 131,072 points 369 us, 354 with 2,048; 10 nearest of
// 50,001 points 106, 101).
constexpr int kSample = 2048;
constexpr int kSamplePer = kSample / kSetupBlock;   // of them per thread
constexpr int kTrimBins = 1024;
constexpr int kTrimLevels = 3;
constexpr int kTrimEnough = 128;                    // bins: at least that many left end the trimming
constexpr int kCoarse = 32;                         // cells per axis of the finer counting grid
constexpr int kSetupTable = kCoarse * kCoarse * kCoarse;
// Other reference points that a reference point is expected to share its cell with, per
// neighbour searched for. The thread-per-query pass takes the 27 cells around the query, which
// reach 1 to 1.5 cells from it: on a surface 0.6 k points per cell put about 3 k of them there, and
// it finishes nearly every query that is not isolated. Whole calls for 0.45 / 0.5 / 0.6 / 0.7, us:
// radius of 1M points by 10 of 4,096 anchors (lists of pairs) 340 / 301 / 287 / 290, their learned normals (16 anchors)
// 462 / 427 / 400 / 424, 10 and 15 nearest of 131,071 points with their areas 418 / 405 / 398 / 409,
// 10 nearest of 50,001 points 114 / 110 / 120 / 128. (8 cells per reference point, whatever the cloud, give 0.1 k on a
// sampled surface of 4,096 points: rings 2 and 3, 84 rows of cells instead of 9.)
constexpr float kCellShare = 0.6f;

struct SetupLds {
  int hist[3 * kTrimBins];
  int wtot[kSetupBlock / 64];
  int found[3][2], shrunk[kTrimLevels];  // a flag per level: none is written again while others read it
  int64_t below_lo[3], below[3];
  double range[6];
  float red[6][kSetupBlock / 64];
  unsigned pairs[2];
  GridParams gp;
};

__device__ __forceinline__ uint32_t hash32(uint32_t x) {  // the integer mixer lowbias32 (C. Wellons, hash-prospector, 2018)
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  return x ^ (x >> 16);
}

// Index of sample s of S out of n points: all of them when n == S, else a pseudo-random point of
// the s-th of S equal strata (a fixed step would sample a raster of points in columns).
__device__ __forceinline__ int64_t sample_index(int s, int S, int64_t n) {
  if (n == S) return s;
  const double u = (double)hash32((uint32_t)s) * 0x1p-32;
  const int64_t i = (int64_t)(((double)s + u) * ((double)n / (double)S));
  return i < n ? i : n - 1;
}

// Cube root of a volume, to single precision.
__device__ __forceinline__ double cells_edge(double v) {
  const int e = ilogb(v) / 3;  // v = (m 2^(3e)), m a float's range whatever v
  return ldexp((double)cbrtf((float)ldexp(v, -3 * e)), e);
}

// Grid parameters for the cell edge h (grown until the grid has at most max_cells cells).
__device__ void grid_dims(const double* range, double h, int64_t max_cells, GridParams* gp) {
  float mn[3], mx[3];
  for (int d = 0; d < 3; ++d) {  // the FP64 range rounded outwards to FP32
    mn[d] = (float)range[2 * d];
    if ((double)mn[d] > range[2 * d]) mn[d] = nextafterf(mn[d], -INFINITY);
    mx[d] = (float)range[2 * d + 1];
    if ((double)mx[d] < range[2 * d + 1]) mx[d] = nextafterf(mx[d], INFINITY);
  }
  double ext[3];
  double emax = 0.0;
  for (int d = 0; d < 3; ++d) {
    ext[d] = (double)mx[d] - (double)mn[d];
    if (!(ext[d] >= 0.0 && ext[d] <= 1e30)) ext[d] = 1e30;  // infinite or NaN coordinates
    emax = fmax(emax, ext[d]);
  }
  if (!(emax > 0.0)) emax = 1.0;
  // slabs thinner than 1e-3 of the largest extent count as that thickness for the volume
  double vol = 1.0;
  for (int d = 0; d < 3; ++d) vol *= fmax(ext[d], 1e-3 * emax);
  const double hmin = cells_edge(vol / (double)max_cells);
  if (!(h >= hmin)) h = hmin;
  if (!(h <= emax)) h = emax;
  // every point of the box must fall inside the grid: grow h until the uncapped cell counts
  // multiply to at most max_cells (at most a few steps; the cap only bounds the loop)
  double dd[3] = {1.0, 1.0, 1.0};
  for (int it = 0; it < 4096; ++it) {
    double cells = 1.0;
    for (int d = 0; d < 3; ++d) {
      dd[d] = floor(ext[d] / h) + 1.0;
      cells *= dd[d];
    }
    if (cells <= (double)max_cells) break;
    h *= 1.05;
  }
  if (dd[0] * dd[1] * dd[2] > (double)max_cells) {  // not reached for finite extents; one cell
    dd[0] = dd[1] = dd[2] = 1.0;
    h = emax;
  }
  GridParams g;
  g.ox = mn[0];
  g.oy = mn[1];
  g.oz = mn[2];
  g.h = (float)h;
  g.ih = (float)(1.0 / h);
  g.nx = (int)dd[0];
  g.ny = (int)dd[1];
  g.nz = (int)dd[2];
  g.ncells = (int64_t)g.nx * g.ny * g.nz;
  *gp = g;
}

// Sum of v over the block into *out (LDS, zero before; integer atomics).
__device__ __forceinline__ void block_add(unsigned v, unsigned* out) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(out, v);
}

// Lays out the grid of the references R for searches of k neighbours, by one block of
// kSetupBlock threads; s.gp holds it when this returns (after a barrier). tab: kSetupTable LDS
// counters. What the sample says sets the cost of the search only, never its result.
__device__ void grid_setup(const float* __restrict__ R, int64_t n, int64_t max_cells, int k, SetupLds& s, int* tab) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int S = (int)(n < kSample ? n : kSample);
  float x[kSamplePer][3];
  float mn[3] = {FLT_MAX, FLT_MAX, FLT_MAX}, mx[3] = {-FLT_MAX, -FLT_MAX, -FLT_MAX};
#pragma unroll
  for (int j = 0; j < kSamplePer; ++j) {
    const int i = t + j * kSetupBlock;
    const int64_t o = sample_index(i < S ? i : 0, S, n);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      x[j][d] = R[d * n + o];
      mn[d] = fminf(mn[d], x[j][d]);
      mx[d] = fmaxf(mx[d], x[j][d]);
    }
  }
#pragma unroll
  for (int d = 0; d < 3; ++d)
    for (int o = 32; o > 0; o >>= 1) {
      mn[d] = fminf(mn[d], __shfl_xor(mn[d], o, 64));
      mx[d] = fmaxf(mx[d], __shfl_xor(mx[d], o, 64));
    }
  if (lane == 0)
    for (int d = 0; d < 3; ++d) {
      s.red[d][wv] = mn[d];
      s.red[3 + d][wv] = mx[d];
    }
  for (int i = t; i < 3 * kTrimBins; i += kSetupBlock) s.hist[i] = 0;
  for (int i = t; i < kSetupTable; i += kSetupBlock) tab[i] = 0;
  if (t < 2) s.pairs[t] = 0;
  if (t < kTrimLevels) s.shrunk[t] = 0;
  __syncthreads();
  if (t < 3) {
    float lo = s.red[t][0], hi = s.red[3 + t][0];
    for (int w = 1; w < kSetupBlock / 64; ++w) {
      lo = fminf(lo, s.red[t][w]);
      hi = fmaxf(hi, s.red[3 + t][w]);
    }
    s.range[2 * t] = lo;
    s.range[2 * t + 1] = hi;
    s.below[t] = 0;
  }
  __syncthreads();
  // Trimming: each level narrows an axis to the bins that hold the ranks floor(S / 1024) and
  // S - 1 - floor(S / 1024) of the sample's coordinates. A range whose ranks are not found
  // (NaN coordinates) is kept. Once no axis shrinks below kTrimEnough of its bins, its ends are
  // known to 1% of it and the rest is left (outliers far away take the further levels). 25 -> 20 us.
  const int64_t rlo = S / kTrimBins, rhi = S - 1 - S / kTrimBins;
  bool again = rlo > 0;
  for (int level = 0; level < kTrimLevels && again; ++level) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double lo = s.range[2 * d], hi = s.range[2 * d + 1];
      const double sc = hi > lo ? kTrimBins / (hi - lo) : 0.0;
#pragma unroll
      for (int j = 0; j < kSamplePer; ++j) {
        const double v = x[j][d];
        if (t + j * kSetupBlock < S && v >= lo && v <= hi) {
          const double f = (v - lo) * sc;
          const int b = f > 0.0 ? (f < kTrimBins - 1 ? (int)f : kTrimBins - 1) : 0;
          atomicAdd(&s.hist[d * kTrimBins + b], 1);
        }
      }
    }
    if (t < 6) s.found[t >> 1][t & 1] = -1;
    __syncthreads();
    // threads 256 d .. 256 d + 255 scan the bins of axis d, four each
    const int d = t >> 8, b0 = (t & 255) * 4;
    int c[4] = {0, 0, 0, 0}, sum = 0, inc = 0;
    if (d < 3) {
      for (int q = 0; q < 4; ++q) {
        c[q] = s.hist[d * kTrimBins + b0 + q];
        s.hist[d * kTrimBins + b0 + q] = 0;
        sum += c[q];
      }
      inc = sum;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
      }
      if (lane == 63) s.wtot[wv] = inc;
    }
    __syncthreads();
    if (d < 3) {
      int64_t cum = s.below[d] + inc - sum;
      for (int w = 4 * d; w < wv; ++w) cum += s.wtot[w];
      for (int q = 0; q < 4; ++q) {
        if (cum <= rlo && cum + c[q] > rlo) {
          s.found[d][0] = b0 + q;
          s.below_lo[d] = cum;
        }
        if (cum <= rhi && cum + c[q] > rhi) s.found[d][1] = b0 + q;
        cum += c[q];
      }
    }
    __syncthreads();
    if (t < 3) {
      const double lo = s.range[2 * t], hi = s.range[2 * t + 1];
      const int blo = s.found[t][0], bhi = s.found[t][1];
      if (blo >= 0 && bhi >= 0 && hi > lo) {
        const double w = (hi - lo) / kTrimBins;
        s.range[2 * t] = lo + blo * w;
        s.range[2 * t + 1] = bhi == kTrimBins - 1 ? hi : lo + (bhi + 1) * w;
        s.below[t] = s.below_lo[t];
        if (bhi - blo + 1 < kTrimEnough) s.shrunk[level] = 1;
      }
    }
    __syncthreads();
    again = s.shrunk[level] != 0;
  }
  // Pair counts of the sample on the trimmed box cut into 32 and 16 cells along its longest
  // axis: sum over the points of the other points in their cell.
  double emax = 0.0;
  for (int d = 0; d < 3; ++d) {
    const double e = s.range[2 * d + 1] - s.range[2 * d];
    if (e > emax) emax = e;
  }
  const bool flat = !(emax > 0.0 && emax <= 1e30);
  const float ie = flat ? 0.0f : (float)(kCoarse / emax);
  for (int g = 0; g < 2; ++g) {
    int cell[kSamplePer];
#pragma unroll
    for (int j = 0; j < kSamplePer; ++j) {
      int c3[3];
#pragma unroll
      for (int d = 0; d < 3; ++d)
        c3[d] = (int)fminf(fmaxf(floorf((x[j][d] - (float)s.range[2 * d]) * ie), 0.0f), (float)(kCoarse - 1)) >> g;
      cell[j] = (c3[2] * kCoarse + c3[1]) * kCoarse + c3[0];
      if (t + j * kSetupBlock < S) atomicAdd(&tab[cell[j]], 1);
    }
    __syncthreads();
    unsigned others = 0;
#pragma unroll
    for (int j = 0; j < kSamplePer; ++j)
      if (t + j * kSetupBlock < S) others += (unsigned)tab[cell[j]] - 1u;
    block_add(others, &s.pairs[g]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSamplePer; ++j) tab[cell[j]] = 0;
    __syncthreads();
  }
  if (t == 0) {
    // the points sharing a cell of edge e grow like e^D (D = 2 on a surface)
    const double scale = S > 1 ? (double)(n - 1) / ((double)S * (double)(S - 1)) : 1.0;
    const double fine = fmax((double)s.pairs[0], 0.5) * scale, coarse = fmax((double)s.pairs[1], 1.0) * scale;
    // (single precision: one thread's FP64 log, power and cube root took a third of the kernel, and
    // h sets the search's cost only)
    const float dim = fminf(3.0f, fmaxf(1.0f, log2f((float)(coarse / fine))));
    const double h = flat ? 1.0 : (emax / kCoarse) * exp2f(log2f((float)((double)kCellShare * k / fine)) / dim);
    grid_dims(s.range, h, max_cells, &s.gp);
  }
  __syncthreads();
}

__device__ __forceinline__ void cell_of(const GridParams& g, float x, float y, float z, int& cx,
                                        int& cy, int& cz) {
  // clamped as floats before the conversion, so that points far outside the box (and NaN,
  // which fmaxf maps to 0) land in its border cells
  cx = (int)fminf(fmaxf(floorf((x - g.ox) * g.ih), 0.0f), (float)(g.nx - 1));
  cy = (int)fminf(fmaxf(floorf((y - g.oy) * g.ih), 0.0f), (float)(g.ny - 1));
  cz = (int)fminf(fmaxf(floorf((z - g.oz) * g.ih), 0.0f), (float)(g.nz - 1));
}

__global__ void k_zero_i32(int32_t* __restrict__ a, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    a[i] = 0;
}

// Exclusive scan of a block's per-thread values in thread order (up to 1024 threads); the
// block's total in *total. lds: blockDim.x / 64 ints.
__device__ __forceinline__ int32_t block_exclusive(int32_t v, int32_t* lds, int32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int32_t inc = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  __syncthreads();
  if (lane == 63) lds[wv] = inc;
  __syncthreads();
  int32_t before = 0, all = 0;
  for (int w = 0; w < nw; ++w) {
    const int32_t x = lds[w];
    before += w < wv ? x : 0;
    all += x;
  }
  *total = all;
  return before + inc - v;
}

// In-place exclusive scan of a[0..n) by one block, total to a[n].
__global__ __launch_bounds__(kScanOneBlock) void k_scan_one(int32_t* __restrict__ a, int64_t n) {
  __shared__ int32_t lds[kScanOneBlock / 64];
  int32_t carry = 0;
  for (int64_t b0 = 0; b0 < n; b0 += 4 * kScanOneBlock) {
    const int64_t i = b0 + 4 * (int64_t)threadIdx.x;
    int32_t v[4], tot = 0, all;
    for (int k = 0; k < 4; ++k) {
      v[k] = i + k < n ? a[i + k] : 0;
      tot += v[k];
    }
    int32_t run = carry + block_exclusive(tot, lds, &all);
    for (int k = 0; k < 4; ++k) {
      if (i + k < n) a[i + k] = run;
      run += v[k];
    }
    carry += all;
  }
  if (threadIdx.x == 0) a[n] = carry;
}

// In-place exclusive scan in one pass over the array (chained scan with look-back, after Merrill and Garland,
// "Single-pass Parallel Prefix Scan with Decoupled Look-back", 2016): a block
// takes the next tile from a ticket counter, publishes the tile's sum, and adds up the sums of
// the tiles before it, a wavefront's 64 at a time, back to the nearest one whose full prefix is
// known. A tile's state is one 64-bit word (flag << 32 | value), written and read by device
// atomics, so the value needs no fence of its own. Every wait ends: a block waits only for
// tiles with smaller tickets, whose blocks are running and publish their sum before they wait
// themselves. The length is n_dev->ncells where n_dev is given (the launch then covers the
// largest possible length), else n. state[0] is the ticket, state[1 + tile] the tiles; all zero
// before the launch.
constexpr unsigned long long kTileSum = 1ull << 32, kTilePrefix = 2ull << 32;

__device__ __forceinline__ unsigned long long load_state(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_state(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the tiles before `tile` (by one wavefront; every lane gets it).
__device__ __forceinline__ int32_t look_back(const unsigned long long* __restrict__ tiles, int64_t tile) {
  const int lane = threadIdx.x & 63;
  int32_t sum = 0;
  for (int64_t top = tile - 1; top >= 0;) {
    const int64_t at = top - lane;
    const unsigned long long v = at >= 0 ? load_state(&tiles[at]) : kTilePrefix;
    const unsigned long long known = __ballot((v >> 32) != 0ull), full = __ballot((v >> 32) == 2ull);
    const int stop = full ? __ffsll((long long)full) - 1 : 63;  // lanes 0..stop are needed
    const unsigned long long need = stop == 63 ? ~0ull : ((2ull << stop) - 1ull);
    if ((known & need) != need) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    int32_t x = lane <= stop ? (int32_t)(uint32_t)v : 0;
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    sum += x;
    if (full) break;
    top -= 64;
  }
  return sum;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_chain(int32_t* __restrict__ a, int64_t n,
                                                           const GridParams* __restrict__ n_dev,
                                                           unsigned long long* __restrict__ state) {
  __shared__ int32_t lds[kScanBlock / 64];
  __shared__ int64_t s_tile;
  __shared__ int32_t s_before;
  if (n_dev) n = n_dev->ncells;
  if (threadIdx.x == 0) s_tile = (int64_t)atomicAdd(&state[0], 1ull);
  __syncthreads();
  const int64_t tile = s_tile;
  if (tile * kScanTile >= n) return;
  const int64_t i = tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int32_t v[kScanItems], tot = 0, all;
  if (i + kScanItems <= n) {
    const int4 lo = *reinterpret_cast<const int4*>(a + i), hi = *reinterpret_cast<const int4*>(a + i + 4);
    v[0] = lo.x, v[1] = lo.y, v[2] = lo.z, v[3] = lo.w, v[4] = hi.x, v[5] = hi.y, v[6] = hi.z, v[7] = hi.w;
  } else {
    for (int k = 0; k < kScanItems; ++k) v[k] = i + k < n ? a[i + k] : 0;
  }
  for (int k = 0; k < kScanItems; ++k) tot += v[k];
  int32_t run = block_exclusive(tot, lds, &all);
  if (threadIdx.x < 64) {
    unsigned long long* const tiles = state + 1;
    if (tile > 0 && threadIdx.x == 0) store_state(&tiles[tile], kTileSum | (uint32_t)all);
    const int32_t before = look_back(tiles, tile);
    if (threadIdx.x == 0) {
      store_state(&tiles[tile], kTilePrefix | (uint32_t)(before + all));
      s_before = before;
      if ((tile + 1) * kScanTile >= n) a[n] = before + all;
    }
  }
  __syncthreads();
  run += s_before;
  for (int k = 0; k < kScanItems; ++k) {
    const int32_t x = v[k];
    v[k] = run;
    run += x;
  }
  if (i + kScanItems <= n) {
    *reinterpret_cast<int4*>(a + i) = make_int4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<int4*>(a + i + 4) = make_int4(v[4], v[5], v[6], v[7]);
  } else {
    for (int k = 0; k < kScanItems; ++k)
      if (i + k < n) a[i + k] = v[k];
  }
}

// Grid layout of a reference set too large for k_grid_small (one block).
__global__ __launch_bounds__(kSetupBlock) void k_grid_setup(const float* __restrict__ R, int64_t n,
                                                            int64_t max_cells, int k,
                                                            GridParams* __restrict__ gp) {
  __shared__ SetupLds s;
  __shared__ int tab[kSetupTable];
  grid_setup(R, n, max_cells, k, s, tab);
  if (threadIdx.x == 0) *gp = s.gp;
}

// The whole grid of at most kSmallRefs references by one block: layout, counts and their scan in
// LDS, counting sort. One launch (about 20 us) for the five of the larger sets: the anchor grids
// (4,096 to 8,191 points) are built anew by every radius and feature call.
constexpr int kSmallRefs = 8192;
constexpr int kSmallPer = kSmallRefs / kSetupBlock;

constexpr int kBuckets = 4096;  // of the cell order of queries (k_order)

// Clears what a search of the grid counts in: the bucket totals and the number of deferred items.
// The grid's own kernels do it for a search that follows at once (lists and radii of a cloud's own grid);
// k_order_clear does it before each search of an anchor grid.
__device__ __forceinline__ void clear_queries(int64_t first, int64_t step, int32_t* __restrict__ total,
                                              int32_t* __restrict__ defer) {
  for (int64_t i = first; i < kBuckets; i += step) total[i] = 0;
  if (first == 0) defer[0] = 0;
}

__global__ void k_order_clear(int32_t* __restrict__ total, int32_t* __restrict__ defer) {
  clear_queries(blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x, total, defer);
}

__global__ __launch_bounds__(kSetupBlock) void k_grid_small(const float* __restrict__ R, int64_t n,
                                                            int64_t max_cells, int k,
                                                            GridParams* __restrict__ gp,
                                                            int32_t* __restrict__ start,
                                                            float4* __restrict__ sorted, int32_t* __restrict__ total,
                                                            int32_t* __restrict__ defer) {
  clear_queries(threadIdx.x, kSetupBlock, total, defer);
  __shared__ SetupLds s;
  __shared__ int tab[kSetupTable];
  __shared__ int32_t lds[kSetupBlock / 64];
  grid_setup(R, n, max_cells < kSetupTable ? max_cells : kSetupTable, k, s, tab);  // tab is zero again
  const GridParams g = s.gp;
  const int t = threadIdx.x;
  if (t == 0) *gp = g;
  float4 p[kSmallPer];
  int cell[kSmallPer], rank[kSmallPer];
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j) {
    const int64_t i = t + j * kSetupBlock;
    cell[j] = -1;
    if (i < n) {
      p[j] = make_float4(R[i], R[n + i], R[2 * n + i], __int_as_float((int)i));
      int cx, cy, cz;
      cell_of(g, p[j].x, p[j].y, p[j].z, cx, cy, cz);
      cell[j] = (cz * g.ny + cy) * g.nx + cx;
      rank[j] = atomicAdd(&tab[cell[j]], 1);
    }
  }
  __syncthreads();
  const int nc = (int)g.ncells;
  int32_t carry = 0;
  for (int b0 = 0; b0 < nc; b0 += kSetupBlock) {
    const int i = b0 + t;
    int32_t all;
    const int32_t before = carry + block_exclusive(i < nc ? tab[i] : 0, lds, &all);
    if (i < nc) {
      tab[i] = before;
      start[i] = before;
    }
    carry += all;
  }
  if (t == 0) start[nc] = carry;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSmallPer; ++j)
    if (cell[j] >= 0) sorted[tab[cell[j]] + rank[j]] = p[j];
}

// Clears the cell counts (ncells + 1 of them) and the scan state (as many words as tiles of the
// actual grid need).
__global__ void k_grid_zero(const GridParams* __restrict__ gp, int32_t* __restrict__ count,
                            unsigned long long* __restrict__ state, int32_t* __restrict__ total,
                            int32_t* __restrict__ defer) {
  const int64_t nc = gp->ncells, words = 1 + (nc + kScanTile - 1) / kScanTile;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = t0; i <= nc; i += step) count[i] = 0;
  for (int64_t i = t0; i < words; i += step) state[i] = 0ull;
  clear_queries(t0, step, total, defer);
}

// Cell of each reference point and its rank among the cell's points (arbitrary order).
__global__ void k_cell_count(const float* __restrict__ R, int64_t n, const GridParams* __restrict__ gp,
                             int32_t* __restrict__ key, int32_t* __restrict__ rank, int32_t* __restrict__ count) {
  const GridParams g = *gp;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    int cx, cy, cz;
    cell_of(g, R[i], R[n + i], R[2 * n + i], cx, cy, cz);
    const int32_t c = (int32_t)(((int64_t)cz * g.ny + cy) * g.nx + cx);
    key[i] = c;
    rank[i] = atomicAdd(&count[c], 1);
  }
}

// Scatter reference points into cell order: sorted[pos] = (x, y, z, index bits).
__global__ void k_scatter(const float* __restrict__ R, int64_t n, const int32_t* __restrict__ key,
                          const int32_t* __restrict__ rank, const int32_t* __restrict__ start,
                          float4* __restrict__ sorted) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    sorted[start[key[i]] + rank[i]] = make_float4(R[i], R[n + i], R[2 * n + i], __int_as_float((int)i));
}

// A candidate (d2, j) as one FP64 number: the bits of d2 (>= 0) plus 2^20 in the high word, j (>= 0)
// in the low word. Positive FP64 numbers order like their bits, so keys order like the pairs
// (d2, j); 2^20 keeps every key a normal number and d2 = +inf a finite one. A NaN d2 makes no key (its
// bits can wrap around to a small high word): it is turned away by a comparison of the distances.
constexpr uint32_t kKeyBias = 0x00100000u;
constexpr uint32_t kKeyInf = 0x7f800000u + kKeyBias;

__device__ __forceinline__ uint32_t key_high(double k) { return (uint32_t)__double2hiint(k); }
__device__ __forceinline__ float key_d2(double k) { return __uint_as_float(key_high(k) - kKeyBias); }

// min and max of two keys. Keys are never NaN; written as instructions because fmin and fmax
// first quiet a possible signalling NaN, which is one more FP64 instruction per slot.
__device__ __forceinline__ double key_min(double a, double b) {
  double r;
  __asm__("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double key_max(double a, double b) {
  double r;
  __asm__("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The index of an entry that no reference has filled: a NaN query's, or one of a set with too few
// references that are not NaN. dwg_knn hands it out; the other users of a list never read by it.
constexpr int32_t kNoRef = 0x7fffffff;
__device__ __forceinline__ int32_t filled(int32_t j, int32_t other) { return j == kNoRef ? other : j; }

// The K best candidates of a query, ascending. As pairs: an inserted key x makes b[u]
// max(b[u - 1], min(b[u], x)), two FP64 instructions per slot (ranking the pairs by compares and
// selects took eight).
template <int K>
struct PairList {
  static constexpr bool kIndexed = true;
  double b[K];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int u = 0; u < K; ++u) b[u] = __hiloint2double((int)kKeyInf, kNoRef);
  }
  __device__ __forceinline__ void offer(float d2, int j) {
    if (!(d2 <= key_d2(b[K - 1]))) return;
    const double x = __hiloint2double((int)(__float_as_uint(d2) + kKeyBias), j);
#pragma unroll
    for (int u = K - 1; u >= 1; --u) b[u] = key_max(b[u - 1], key_min(b[u], x));
    b[0] = key_min(b[0], x);
  }
  __device__ __forceinline__ float d2(int u) const { return key_d2(b[u]); }
  __device__ __forceinline__ int index(int u) const { return __double2loint(b[u]); }
};

// As squared distances alone, where only the radius they give is asked for: the median of
// (b[u - 1], b[u], x), one FP32 instruction per slot (which of equally distant references is taken
// does not matter then). 1M queries of 4,096 anchors, k = 10: 116 us, with pairs 166.
template <int K>
struct DistList {
  static constexpr bool kIndexed = false;
  float b[K];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int u = 0; u < K; ++u) b[u] = INFINITY;
  }
  __device__ __forceinline__ void offer(float d2, int) {
    if (!(d2 < b[K - 1])) return;
#pragma unroll
    for (int u = K - 1; u >= 1; --u) b[u] = __builtin_amdgcn_fmed3f(b[u - 1], b[u], d2);
    b[0] = fminf(b[0], d2);
  }
  __device__ __forceinline__ float d2(int u) const { return b[u]; }
  __device__ __forceinline__ int index(int) const { return 0; }
};

// What a finished query writes: its neighbour list, or the kernel radius that the list gives.
enum EmitMode { kEmitList = 0, kEmitMean = 1, kEmitWindow = 2, kEmitScaled = 3 };
struct KnnEmit {
  int mode;
  int32_t* idx;   // [m][k]
  float* dist;    // [m][k] or NULL
  float* delta;   // [m]; kEmitScaled (the indices too, 0 for those not filled, whose mean distance is
                  // infinite): the inverse of the mean distance
  float scale;    // kEmitMean
  float vmin, vmax;  // kEmitWindow
};

// 1 / (s / k), 0 when s is 0: the scale of the anchor features.
__device__ __forceinline__ float inverse_mean(float s, int k) {
  s *= 1.0f / (float)k;
  return s > 0.0f ? 1.0f / s : 0.0f;
}

template <int K, class List>
__device__ __forceinline__ void emit_query(const KnnEmit& e, int64_t q, const List& b) {
  float d[K];
#pragma unroll
  for (int u = 0; u < K; ++u) d[u] = sqrtf(b.d2(u));
  if (List::kIndexed && e.mode == kEmitList) {
#pragma unroll
    for (int u = 0; u < K; ++u) {
      e.idx[q * K + u] = b.index(u);
      if (e.dist) e.dist[q * K + u] = d[u];
    }
  } else if (e.mode == kEmitMean || (List::kIndexed && e.mode == kEmitScaled)) {
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < K; ++u) s += d[u];
    if (!List::kIndexed || e.mode == kEmitMean) {
      e.delta[q] = e.scale * (s / (float)K);
      return;
    }
    e.delta[q] = inverse_mean(s, K);
#pragma unroll
    for (int u = 0; u < K; ++u) e.idx[q * K + u] = filled(b.index(u), 0);
  } else {
    // the mean of the distances that lie in [vmin, vmax]; when none does, the mean of all k
    // clamped to [vmin, vmax] (Sec. 5.2 "Poisson Kernels")
    double s = 0.0, all = 0.0;
    int c = 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const double x = d[u];
      all += x;
      if (x >= e.vmin && x <= e.vmax) {
        s += x;
        ++c;
      }
    }
    double r = c > 0 ? s / c : all / K;
    if (c == 0) r = r < e.vmin ? e.vmin : (r > e.vmax ? e.vmax : r);
    e.delta[q] = (float)r;
  }
}

// The same by a wavefront whose lane u holds key u (u < k).
__device__ __forceinline__ void emit_wave(const KnnEmit& e, int64_t q, int k, double key) {
  const int lane = threadIdx.x & 63;
  const float d = sqrtf(key_d2(key));
  if (e.mode == kEmitList) {
    if (lane < k) {
      e.idx[q * k + lane] = __double2loint(key);
      if (e.dist) e.dist[q * k + lane] = d;
    }
    return;
  }
  float s = 0.0f;
  double sd = 0.0, all = 0.0;
  int c = 0;
  for (int u = 0; u < k; ++u) {
    const float du = __shfl(d, u, 64);
    s += du;
    all += (double)du;
    if ((double)du >= e.vmin && (double)du <= e.vmax) {
      sd += (double)du;
      ++c;
    }
  }
  if (e.mode == kEmitMean) {
    if (lane == 0) e.delta[q] = e.scale * (s / (float)k);
  } else if (e.mode == kEmitScaled) {
    if (lane == 0) e.delta[q] = inverse_mean(s, k);
    if (lane < k) e.idx[q * k + lane] = filled(__double2loint(key), 0);
  } else {
    double r = c > 0 ? sd / c : all / k;
    if (c == 0) r = r < e.vmin ? e.vmin : (r > e.vmax ? e.vmax : r);
    if (lane == 0) e.delta[q] = (float)r;
  }
}

// Lower bound of the distance from a query to every reference outside the cube of cells
// [c - r, c + r]: the smallest distance of its projection onto the grid's box to a face of the
// cube that has cells beyond it (+inf when none has). f: the projection's cell coordinates.
// The margin covers the rounding of the cell coordinates (both points', relative to the
// number of cells) and of the squared distance it is compared with.
__device__ __forceinline__ float outside_bound(const GridParams& g, const float* f, int cx, int cy, int cz, int r) {
  float lb = INFINITY;
  const int c[3] = {cx, cy, cz}, nn[3] = {g.nx, g.ny, g.nz};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float in = f[d] - (float)c[d];  // in [0, 1]
    if (c[d] - r > 0) lb = fminf(lb, (float)r + in);
    if (c[d] + r < nn[d] - 1) lb = fminf(lb, (float)r + 1.0f - in);
  }
  const float margin = 1e-6f + 5e-7f * (float)max(g.nx, max(g.ny, g.nz));
  return fmaxf(lb - margin, 0.0f) * (g.h * 0.999999f);
}

// Cell coordinates of the query's projection onto the grid's box, each in [0, cells].
__device__ __forceinline__ void cell_coords(const GridParams& g, float x, float y, float z, int cx, int cy, int cz,
                                            float* f) {
  f[0] = fminf(fmaxf((x - g.ox) * g.ih, (float)cx), (float)(cx + 1));
  f[1] = fminf(fmaxf((y - g.oy) * g.ih, (float)cy), (float)(cy + 1));
  f[2] = fminf(fmaxf((z - g.oz) * g.ih, (float)cz), (float)(cz + 1));
}

// A query of the search: output row q, position, and the reference index it skips (-1: none).
struct KnnQuery {
  int64_t q;
  float x, y, z;
  int skip;
};

// Where the queries of a search are read: work item p is the p-th entry (x, y, z, query number) of
// `items`, or, without items, query q0 + p of the planar array Q with leading dimension ld. Skip
// mode: 0 none; 1 reference i for query i; 2 reference i / stride for query i when i % stride == 0
// (i counted from the start of Q).
struct QuerySet {
  const float* Q;
  int64_t ld, q0, m;
  const float4* items;
  int skip_mode;
  int64_t stride;
};

__device__ __forceinline__ KnnQuery knn_query_of(const QuerySet& s, int64_t p) {
  KnnQuery k;
  if (s.items) {
    const float4 it = s.items[p];
    k.q = __float_as_int(it.w);
    k.x = it.x;
    k.y = it.y;
    k.z = it.z;
  } else {
    k.q = p;
    k.x = s.Q[s.q0 + p];
    k.y = s.Q[s.ld + s.q0 + p];
    k.z = s.Q[2 * s.ld + s.q0 + p];
  }
  const int64_t gq = s.q0 + k.q;
  k.skip = -1;
  if (s.skip_mode == 1) k.skip = (int)gq;
  if (s.skip_mode == 2 && ((uint32_t)gq % (uint32_t)s.stride) == 0) k.skip = (int)((uint32_t)gq / (uint32_t)s.stride);
  return k;
}

// The cells of the cube of half-width r around cell (cx, cy, cz) outside that of half-width rp
// (rp < r; -1: the whole cube) in the grid row (z, y), as at most two ranges [b0, e0), [b1, e1)
// of `sorted`: the whole row [xl, xh] (clipped to the grid) when |z - cz| or |y - cy| exceeds rp,
// else its two ends. The cells of a row are consecutive, so a range costs two loads of `start`
// however many cells it spans.
__device__ __forceinline__ void shell_row(const GridParams& g, const int32_t* __restrict__ start, int cx, int cy,
                                          int cz, int rp, int z, int y, int xl, int xh, int32_t& b0, int32_t& e0,
                                          int32_t& b1, int32_t& e1) {
  const int64_t row = ((int64_t)z * g.ny + y) * g.nx;
  b0 = e0 = b1 = e1 = 0;
  if (max(abs(z - cz), abs(y - cy)) > rp) {
    b0 = start[row + xl];
    e0 = start[row + xh + 1];
    return;
  }
  if (cx - rp - 1 >= xl) {
    b0 = start[row + xl];
    e0 = start[row + cx - rp];
  }
  if (cx + rp + 1 <= xh) {
    b1 = start[row + cx + rp + 1];
    e1 = start[row + xh + 1];
  }
}

// Search of one query by one thread over the cubes of half-width 1, 2, .. rcap: true when it is
// finished (b holds its list), false when it needs more rings.
template <int K, class List>
__device__ __forceinline__ bool knn_thread(const GridParams& g, const int32_t* __restrict__ start,
                                           const float4* __restrict__ sorted, const KnnQuery& kq, int rcap, List& b) {
  const float qx = kq.x, qy = kq.y, qz = kq.z;
  const int skip = kq.skip;
  b.clear();
  int cx, cy, cz;
  cell_of(g, qx, qy, qz, cx, cy, cz);
  float f[3];
  cell_coords(g, qx, qy, qz, cx, cy, cz, f);
  const int rmax = max(g.nx, max(g.ny, g.nz));
  // Points are taken four at a time, with no branch but the insertion's, the row's last one standing in
  // for those past its end: one wait per four loads (one at a time with the next one in flight: 10
  // nearest of 50,001 points 117 us, 113 / 108 / 106 for batches of 2 / 3 / 4). A NaN is never
  // taken.
  auto scan = [&](int32_t pp, int32_t e) {
    constexpr int kBatch = 4;
    for (; pp < e; pp += kBatch) {
      float4 sp[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) sp[u] = sorted[min(pp + u, e - 1)];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = __float_as_int(sp[u].w);
        const float ex = sp[u].x - qx, ey = sp[u].y - qy, ez = sp[u].z - qz;
        const bool takes = j != skip && (u == 0 || pp + u < e);
        b.offer(takes ? fmaf(ez, ez, fmaf(ey, ey, ex * ex)) : NAN, j);
      }
    }
  };
  // The cube of half-width 1: nine rows of up to three cells, the query's own row first, their
  // eighteen ends loaded together.
  {
    const int xl = max(cx - 1, 0), xh = min(cx + 1, g.nx - 1);
    constexpr int kOrder[9][2] = {{0, 0}, {0, -1}, {0, 1}, {-1, 0}, {1, 0}, {-1, -1}, {-1, 1}, {1, -1}, {1, 1}};
    int32_t b0[9], e0[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const int z = cz + kOrder[i][0], y = cy + kOrder[i][1];
      const bool in = z >= 0 && z < g.nz && y >= 0 && y < g.ny;
      const int64_t row = in ? ((int64_t)z * g.ny + y) * g.nx : 0;
      b0[i] = start[row + xl];
      e0[i] = in ? start[row + xh + 1] : b0[i];
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) scan(b0[i], e0[i]);
  }
  // Then a ring at a time. The search ends once the k-th best distance is within outside_bound.
  // (A point, or the query, outside the grid's box sits in the border cell that holds its
  // projection onto the box; projecting both onto the box shortens no distance, so the bound
  // still holds.)
  for (int r = 1;; ++r) {
    const float lb = outside_bound(g, f, cx, cy, cz, r);
    const float kth = b.d2(K - 1);  // +inf while the list is not full
    if (lb == INFINITY || (kth < INFINITY && kth <= lb * lb) || r >= rmax) return true;
    if (r >= rcap) return false;
    const int rr = r + 1;
    const int zl = max(cz - rr, 0), zh = min(cz + rr, g.nz - 1);
    const int yl = max(cy - rr, 0), yh = min(cy + rr, g.ny - 1);
    const int xl = max(cx - rr, 0), xh = min(cx + rr, g.nx - 1);
    for (int z = zl; z <= zh; ++z) {
      for (int y = yl; y <= yh; ++y) {
        int32_t b0, e0, b1, e1;
        shell_row(g, start, cx, cy, cz, r, z, y, xl, xh, b0, e0, b1, e1);
        scan(b0, e0);
        scan(b1, e1);
      }
    }
  }
}

// The k nearest references of every query of the set; results go to the rows q of `em`.
// Two passes, so that a few isolated queries (outliers, whose search spans thousands of
// cells) do not hold up the wavefronts of everyone else: k_knn (one thread per work item p)
// searches the cubes up to half-width rcap and appends the items it has not finished to
// defer[1..] (defer[0] counts them); k_knn_wave then searches each deferred item with a whole
// wavefront. A query's result, the k smallest (distance^2, index) pairs, does not depend on the
// order in which candidates are met, so it is the same whichever pass finishes it. Work items in
// cell order let the lanes of a wavefront walk the same rows of cells: the same loads, loops of
// nearly the same length.
template <int K, class List>
__global__ __launch_bounds__(256) void k_knn(QuerySet qs, const GridParams* __restrict__ gp,
                                             const int32_t* __restrict__ start,
                                             const float4* __restrict__ sorted, int rcap,
                                             int32_t* __restrict__ defer, KnnEmit em) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= qs.m) return;
  const GridParams g = *gp;
  const KnnQuery kq = knn_query_of(qs, p);
  List b;
  if (knn_thread<K>(g, start, sorted, kq, rcap, b))
    emit_query<K>(em, kq.q, b);
  else
    defer[1 + atomicAdd(&defer[0], 1)] = (int32_t)p;
}

// ---- Cell order for queries in no particular order (the points of a cloud against its anchors).
// A counting sort by a Morton code of the query's cell, coarsened to 4 bits per axis: block counts
// in LDS added to the totals, a scan, and a second pass in which every block reserves its range
// of each bucket (the order inside a bucket is arbitrary, which changes no result). 1M queries of
// 4,096 anchors, k = 10: the search takes 457 us in the given order (a wavefront's lanes then load
// 64 different lines at a time) and less than half of it in this one; sorting inside blocks
// of 2,048 queries gained nothing, since a wavefront's queries then still lie in some 40 cells.
constexpr int kOrderBlock = 1024;
constexpr int kOrderPer = 8;
constexpr int kOrderTile = kOrderBlock * kOrderPer;

__device__ __forceinline__ uint32_t spread4(uint32_t v) {
  return (v & 1u) | (v & 2u) << 2 | (v & 4u) << 4 | (v & 8u) << 6;
}

__device__ __forceinline__ int bucket_of(const GridParams& g, int sh, float x, float y, float z) {
  int cx, cy, cz;
  cell_of(g, x, y, z, cx, cy, cz);
  return (int)(spread4((uint32_t)cx >> sh) | spread4((uint32_t)cy >> sh) << 1 | spread4((uint32_t)cz >> sh) << 2);
}

// The shift that leaves 4 bits of every cell coordinate.
__device__ __forceinline__ int bucket_shift(const GridParams& g) {
  const int top = max(g.nx, max(g.ny, g.nz)) - 1;
  return top > 15 ? 28 - __clz(top) : 0;
}

// FILL = false: adds the block's bucket counts to total. FILL = true: total holds the buckets'
// first slots and serves as their cursor; writes the items.
template <bool FILL>
__global__ __launch_bounds__(kOrderBlock) void k_order(QuerySet qs, const GridParams* __restrict__ gp,
                                                       int32_t* __restrict__ total, float4* __restrict__ items) {
  __shared__ int32_t cnt[kBuckets];
  const int t = threadIdx.x;
  const GridParams g = *gp;
  const int sh = bucket_shift(g);
  const int64_t base = (int64_t)blockIdx.x * kOrderTile;
  for (int i = t; i < kBuckets; i += kOrderBlock) cnt[i] = 0;
  __syncthreads();
  float x[kOrderPer][3];
  int bucket[kOrderPer], rank[kOrderPer];
#pragma unroll
  for (int u = 0; u < kOrderPer; ++u) {
    const int64_t p = base + t + u * kOrderBlock;
    bucket[u] = -1;
    if (p < qs.m) {
      for (int d = 0; d < 3; ++d) x[u][d] = qs.Q[d * qs.ld + qs.q0 + p];
      bucket[u] = bucket_of(g, sh, x[u][0], x[u][1], x[u][2]);
      rank[u] = atomicAdd(&cnt[bucket[u]], 1);
    }
  }
  __syncthreads();
  for (int i = t; i < kBuckets; i += kOrderBlock)
    if (const int32_t c = cnt[i]) {
      const int32_t first = atomicAdd(&total[i], c);
      if (FILL) cnt[i] = first;
    }
  if (!FILL) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kOrderPer; ++u)
    if (bucket[u] >= 0)
      items[cnt[bucket[u]] + rank[u]] =
          make_float4(x[u][0], x[u][1], x[u][2], __int_as_float((int)(base + t + u * kOrderBlock)));
}

// Orders the LDS accesses of a wavefront that shares data between its own lanes only.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The value of lane l - 1 of the row of 16 lanes (0 in its first lane).
__device__ __forceinline__ double lane_below(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x111, 0xf, 0xf, true);  // row_shr:1
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x111, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// The key of the lane whose number differs in the given bits, within a row of 16 lanes.
constexpr int kXor1 = 0xb1, kXor2 = 0x4e, kXor3 = 0x1b, kXor7 = 0x141, kXor8 = 0x128, kXor15 = 0x140;
__device__ __forceinline__ double lane_xor4(double v) { return dpp_double<kXor3>(dpp_double<kXor7>(v)); }

// Of this lane's key and its partner's, the smaller where the lane is the lower of the two.
__device__ __forceinline__ double exchange(double v, double other, bool lower) {
  return (v < other) == lower ? v : other;
}

// Sorts the keys of a row (ascending) that first falls and then rises or the reverse.
__device__ __forceinline__ double merge_row(double v, int lane) {
  v = exchange(v, dpp_double<kXor8>(v), !(lane & 8));
  v = exchange(v, lane_xor4(v), !(lane & 4));
  v = exchange(v, dpp_double<kXor2>(v), !(lane & 2));
  return exchange(v, dpp_double<kXor1>(v), !(lane & 1));
}

// The 16 smallest of the list `key` (ascending in each row, the same in every row) and the 64 lanes'
// x, as such a list: the rows are sorted (a bitonic network), and two sorted rows a, b hold their 16
// smallest in min(a_i, b_15-i). 135 instructions, as many as a dozen insertions.
__device__ __forceinline__ double merge_keys(double key, double x) {
  const int lane = threadIdx.x & 63;
  x = exchange(x, dpp_double<kXor1>(x), !(lane & 1));
  x = exchange(x, dpp_double<kXor3>(x), !(lane & 2));
  x = exchange(x, dpp_double<kXor1>(x), !(lane & 1));
  x = exchange(x, dpp_double<kXor7>(x), !(lane & 4));
  x = exchange(x, dpp_double<kXor2>(x), !(lane & 2));
  x = exchange(x, dpp_double<kXor1>(x), !(lane & 1));
  x = exchange(x, dpp_double<kXor15>(x), !(lane & 8));
  x = exchange(x, lane_xor4(x), !(lane & 4));
  x = exchange(x, dpp_double<kXor2>(x), !(lane & 2));
  x = exchange(x, dpp_double<kXor1>(x), !(lane & 1));
  {
    const unsigned lo = (unsigned)__double2loint(x), hi = (unsigned)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    x = key_min(__hiloint2double((int)b[0], (int)a[0]), dpp_double<kXor15>(__hiloint2double((int)b[1], (int)a[1])));
    x = merge_row(x, lane);
  }
  {
    const unsigned lo = (unsigned)__double2loint(x), hi = (unsigned)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    x = key_min(__hiloint2double((int)b[0], (int)a[0]), dpp_double<kXor15>(__hiloint2double((int)b[1], (int)a[1])));
    x = merge_row(x, lane);
  }
  return merge_row(key_min(key, dpp_double<kXor15>(x)), lane);
}

// Inclusive sum over the lanes.
__device__ __forceinline__ int32_t wave_scan(int32_t v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
  return v;
}

// The items k_knn left unfinished, one wavefront per item (a grid-stride loop over the
// wavefronts of the launch). The cube around the query grows by half (half-width 2, 3, 4, 6, 9,
// ...), or to the half-width that the k-th best distance needs where that is less; the lanes share out
// the rows of cells that each step adds, and take the rows' points 64 at a time whatever row they
// lie in: a lane's row is the last one that starts at or before its place in the sequence. (Four rows
// per lane and step, or growing straight to the k-th best distance, took 1.5 times as long.) The
// list of the k best is spread over the lanes of a row of 16, one key per lane (the same in every row):
// a candidate that beats the last key is broadcast and inserted with one minimum and one
// maximum, whatever k; more than kMergeFrom candidates are sorted and merged at once. Instruction
// issue bounds it: 800 per item, most of them insertions of the first 64 candidates one by one
// and a list of positions written row by row, when 1M queries of 4,096 anchors took 112 us;
// 66 now. The work per step is bounded by the grid's rows.
constexpr int kMergeFrom = 12;

__global__ __launch_bounds__(256) void k_knn_wave(QuerySet qs, const GridParams* __restrict__ gp,
                                                  const int32_t* __restrict__ start,
                                                  const float4* __restrict__ sorted,
                                                  const int32_t* __restrict__ defer, int k, KnnEmit em) {
  __shared__ int32_t mark_all[4][64];
  const int lane = threadIdx.x & 63;
  int32_t* const mark = mark_all[threadIdx.x >> 6];
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t nd = defer[0];
  const GridParams g = *gp;
  const int rmax = max(g.nx, max(g.ny, g.nz));
  for (int64_t item = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; item < nd; item += nwaves) {
    const KnnQuery kq = knn_query_of(qs, defer[1 + item]);
    const float qx = kq.x, qy = kq.y, qz = kq.z;
    const int skip = kq.skip;
    double key = __hiloint2double((int)kKeyInf, kNoRef);      // list entry lane % 16
    uint32_t worst = kKeyInf;                                 // high word of entry k - 1
    int cx, cy, cz;
    cell_of(g, qx, qy, qz, cx, cy, cz);
    float f[3];
    cell_coords(g, qx, qy, qz, cx, cy, cz, f);
    for (int rp = -1, r = 2;;) {
      const int zl = max(cz - r, 0), zh = min(cz + r, g.nz - 1);
      const int yl = max(cy - r, 0), yh = min(cy + r, g.ny - 1);
      const int xl = max(cx - r, 0), xh = min(cx + r, g.nx - 1);
      const int nyr = yh - yl + 1;
      const int64_t rows = (int64_t)(zh - zl + 1) * nyr;
      for (int64_t l0 = 0; l0 < rows; l0 += 64) {
        const int64_t l = l0 + lane;
        int32_t b0 = 0, e0 = 0, b1 = 0, e1 = 0;  // this lane's row: up to two ranges of sorted
        if (l < rows)
          shell_row(g, start, cx, cy, cz, rp, zl + (int)(l / nyr), yl + (int)(l % nyr), xl, xh, b0, e0, b1, e1);
        const int32_t len0 = e0 - b0, len = len0 + (e1 - b1);
        const int32_t upto = wave_scan(len), from = upto - len, all = __builtin_amdgcn_readlane(upto, 63);
        int carry = 0;  // the row of the place before the next 64
        for (int32_t base = 0; base < all; base += 64) {
          mark[lane] = 0;
          wave_lds_fence();
          if (len > 0 && from >= base && from < base + 64) mark[from - base] = lane + 1;
          wave_lds_fence();
          const int32_t m = mark[lane];
          const unsigned long long first = __ballot(m != 0) & (~0ull >> (63 - lane));
          const int started = __shfl(m, first ? 63 - __clzll((long long)first) : lane, 64);
          const int row = first ? started - 1 : carry;
          carry = __builtin_amdgcn_readlane(row, 63);
          const int32_t at = base + lane - __shfl(from, row, 64), l0r = __shfl(len0, row, 64);
          const int32_t lo = __shfl(b0, row, 64), hi1 = __shfl(b1, row, 64);
          uint32_t hi = 0xffffffffu;
          int j = kNoRef;
          if (base + lane < all) {
            const float4 sp = sorted[at < l0r ? lo + at : hi1 + (at - l0r)];
            j = __float_as_int(sp.w);
            const float ex = sp.x - qx, ey = sp.y - qy, ez = sp.z - qz;
            const float d2 = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
            if (j != skip && d2 <= INFINITY) hi = __float_as_uint(d2) + kKeyBias;  // not a NaN
          }
          unsigned long long mask = __ballot(hi <= worst);
          if (__popcll(mask) > kMergeFrom) {
            const bool in = hi <= worst;
            key = merge_keys(key, __hiloint2double(in ? (int)hi : (int)kKeyInf, in ? j : kNoRef));
            worst = (uint32_t)__builtin_amdgcn_readlane(__double2hiint(key), k - 1);
            continue;
          }
          while (mask) {
            const int src = __ffsll((long long)mask) - 1;
            mask &= mask - 1ull;
            const uint32_t ch = (uint32_t)__builtin_amdgcn_readlane((int)hi, src);
            if (ch > worst) continue;
            const double x = __hiloint2double((int)ch, __builtin_amdgcn_readlane(j, src));
            key = key_max(lane_below(key), key_min(key, x));
            worst = (uint32_t)__builtin_amdgcn_readlane(__double2hiint(key), k - 1);
          }
        }
      }
      const float lb = outside_bound(g, f, cx, cy, cz, r);
      const bool full = worst < kKeyInf;
      const float reach = __uint_as_float(worst - kKeyBias);  // squared
      if (lb == INFINITY || (full && reach <= lb * lb) || r >= rmax) break;
      rp = r;
      const int grown = min(r + (r >> 1), rmax);
      r = full ? max(r + 1, min(grown, (int)fminf(sqrtf(reach) * g.ih + 1.0f, (float)rmax))) : grown;
    }
    emit_wave(em, kq.q, k, key);
  }
}

__global__ void k_gather_anchors(const float* __restrict__ P, int64_t n, int64_t stride, int64_t na,
                                 float* __restrict__ A, float4* __restrict__ A4) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= na) return;
  const int64_t i = a * stride;
  const float4 v = make_float4(P[i], P[n + i], P[2 * n + i], 0.0f);
  A[a] = v.x;
  A[na + a] = v.y;
  A[2 * na + a] = v.z;
  A4[a] = v;
}

// feat[i][3t + d] = (anchor_t - p_i)_d / s_i, s_i = mean of the 16 anchor distances, for
// the points q0 + i, i = 0..m-1 (idx, inv, feat are chunk-local): a thread per (point, anchor), so
// that a wavefront reads and writes consecutive memory.
__global__ void k_features(const float* __restrict__ P, int64_t n, int64_t q0, int64_t m,
                           const float4* __restrict__ A4, const int32_t* __restrict__ idx,
                           const float* __restrict__ inv, float* __restrict__ feat) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m * DWG_FEAT_K;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = t / DWG_FEAT_K, gi = q0 + i;
    const float4 a = A4[idx[t]];
    const float is = inv[i];
    feat[3 * t + 0] = (a.x - P[gi]) * is;
    feat[3 * t + 1] = (a.y - P[n + gi]) * is;
    feat[3 * t + 2] = (a.z - P[2 * n + gi]) * is;
  }
}

constexpr int kBboxBlocks = 256;

int64_t max_cells_for(int64_t nr) { return std::max<int64_t>(8 * nr, 64); }

// Unit eigenvector of the smallest eigenvalue of a symmetric 3x3 matrix (FP64): eigenvalues
// by the trigonometric solution of the characteristic cubic (Smith, CACM 1961), the vector
// as the largest cross product of two rows of (A - lambda I), sign left as it falls. An
// isotropic matrix gives (0, 0, 1).
__device__ void smallest_eigvec(const double a[6], double v[3]) {
  const double a00 = a[0], a01 = a[1], a02 = a[2], a11 = a[3], a12 = a[4], a22 = a[5];
  const double p1 = a01 * a01 + a02 * a02 + a12 * a12;
  const double q = (a00 + a11 + a22) / 3.0;
  const double p2 = (a00 - q) * (a00 - q) + (a11 - q) * (a11 - q) + (a22 - q) * (a22 - q) + 2.0 * p1;
  const double p = sqrt(p2 / 6.0);
  v[0] = 0.0;
  v[1] = 0.0;
  v[2] = 1.0;
  if (!(p > 0.0)) return;
  const double b00 = (a00 - q) / p, b11 = (a11 - q) / p, b22 = (a22 - q) / p;
  const double b01 = a01 / p, b02 = a02 / p, b12 = a12 / p;
  double r = 0.5 * (b00 * (b11 * b22 - b12 * b12) - b01 * (b01 * b22 - b12 * b02) + b02 * (b01 * b12 - b11 * b02));
  r = fmin(1.0, fmax(-1.0, r));
  const double phi = acos(r) / 3.0;
  const double lam = q + 2.0 * p * cos(phi + 2.0943951023931954923);  // smallest
  const double r0[3] = {a00 - lam, a01, a02}, r1[3] = {a01, a11 - lam, a12}, r2[3] = {a02, a12, a22 - lam};
  double c[3][3];
  const double* rows[3][2] = {{r0, r1}, {r0, r2}, {r1, r2}};
  int best = 0;
  double bn = -1.0;
  for (int t = 0; t < 3; ++t) {
    const double* x = rows[t][0];
    const double* y = rows[t][1];
    c[t][0] = x[1] * y[2] - x[2] * y[1];
    c[t][1] = x[2] * y[0] - x[0] * y[2];
    c[t][2] = x[0] * y[1] - x[1] * y[0];
    const double nn = c[t][0] * c[t][0] + c[t][1] * c[t][1] + c[t][2] * c[t][2];
    if (nn > bn) {
      bn = nn;
      best = t;
    }
  }
  if (!(bn > 0.0)) return;
  const double inv = 1.0 / sqrt(bn);
  v[0] = c[best][0] * inv;
  v[1] = c[best][1] * inv;
  v[2] = c[best][2] * inv;
}

// PCA normals (Sec. 5.1 "Normal Initialization"): covariance of p_i and its k nearest other
// points about their mean (FP64), eigenvector of the smallest eigenvalue, turned to point away
// from the origin (n . p_i > 0; at n . p_i == 0 the largest-magnitude component positive).
__global__ void k_pca_normals(const float* __restrict__ P, int64_t n, const int32_t* __restrict__ idx, int k,
                              float* __restrict__ N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double mx = P[i], my = P[n + i], mz = P[2 * n + i];
  for (int t = 0; t < k; ++t) {
    const int64_t j = filled(idx[i * k + t], (int32_t)i);
    mx += P[j];
    my += P[n + j];
    mz += P[2 * n + j];
  }
  const double inv = 1.0 / (double)(k + 1);
  mx *= inv;
  my *= inv;
  mz *= inv;
  double a[6] = {0, 0, 0, 0, 0, 0};
  for (int t = -1; t < k; ++t) {
    const int64_t j = t < 0 ? i : (int64_t)filled(idx[i * k + t], (int32_t)i);
    const double x = P[j] - mx, y = P[n + j] - my, z = P[2 * n + j] - mz;
    a[0] += x * x;
    a[1] += x * y;
    a[2] += x * z;
    a[3] += y * y;
    a[4] += y * z;
    a[5] += z * z;
  }
  double v[3];
  smallest_eigvec(a, v);
  double s = v[0] * P[i] + v[1] * P[n + i] + v[2] * P[2 * n + i];
  if (s == 0.0) {
    const double m0 = fabs(v[0]), m1 = fabs(v[1]), m2 = fabs(v[2]);
    s = (m0 >= m1 && m0 >= m2) ? v[0] : (m1 >= m2 ? v[1] : v[2]);
  }
  if (s < 0.0) {
    v[0] = -v[0];
    v[1] = -v[1];
    v[2] = -v[2];
  }
  N[i] = (float)v[0];
  N[n + i] = (float)v[1];
  N[2 * n + i] = (float)v[2];
}

// Area weight of p_i (Sec. 5.1 "Computing Area Weights"): the plane through p_i normal to the
// smallest-eigenvalue eigenvector of the covariance of p_i and its m nearest other points
// (FP64), those points projected onto it, and the area of p_i's cell in the 2D Voronoi
// diagram of the projections: the square [-R, R]^2 (R = the largest projected distance, which
// bounds the cell of a point whose neighbours lie on one side) cut by the half-planes
// x . q_j <= |q_j|^2 / 2; the square's axes are u = n x e_k / |n x e_k| (e_k the axis with the
// smallest |n_k|, the first on ties) and n x u. Coincident neighbours (q_j = 0) bound nothing
// and are skipped; all-coincident neighbourhoods give 0.
//
// A block takes kCellPoints points. All its threads fetch the neighbours (one word of idx after
// another, the points scattered), one thread per point fits the plane, four threads per point
// project and then take every fourth line each. FP64 arithmetic and its latency bound it: with one
// thread per point throughout and a division per pair of lines, 131,072 points (two wavefronts
// per SIMD) took 202 us; four threads 129, the projections in the neighbours' place in LDS (eight
// blocks per CU instead of five) 111, and the loop over the lines without branches 87.
constexpr int kCellPoints = 64;

__global__ __launch_bounds__(4 * kCellPoints) void k_voronoi_area(const float* __restrict__ P, int64_t n,
                                                                  const int32_t* __restrict__ idx, int m,
                                                                  float* __restrict__ area) {
  // the neighbours, then in their place their projections
  __shared__ double2 qs[kMaxK][kCellPoints];
  __shared__ double axes[6][kCellPoints];  // u, w of the plane
  float(*nb)[kMaxK][kCellPoints] = reinterpret_cast<float(*)[kMaxK][kCellPoints]>(qs);
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * kCellPoints;
  const int np = (int)(n - base < kCellPoints ? n - base : kCellPoints);
  for (int e = tid; e < np * m; e += 4 * kCellPoints) {
    const int pt = e / m, t = e - pt * m;
    const int64_t j = filled(idx[base * m + e], (int32_t)(base + pt));
    nb[0][t][pt] = P[j];
    nb[1][t][pt] = P[n + j];
    nb[2][t][pt] = P[2 * n + j];
  }
  __syncthreads();
  if (tid < np) {
    const int64_t i = base + tid;
    const double px = P[i], py = P[n + i], pz = P[2 * n + i];
    double mx = px, my = py, mz = pz;
    for (int t = 0; t < m; ++t) {
      mx += nb[0][t][tid];
      my += nb[1][t][tid];
      mz += nb[2][t][tid];
    }
    const double inv = 1.0 / (double)(m + 1);
    mx *= inv;
    my *= inv;
    mz *= inv;
    double a[6] = {0, 0, 0, 0, 0, 0};
    for (int t = -1; t < m; ++t) {
      const double x = (t < 0 ? px : (double)nb[0][t][tid]) - mx;
      const double y = (t < 0 ? py : (double)nb[1][t][tid]) - my;
      const double z = (t < 0 ? pz : (double)nb[2][t][tid]) - mz;
      a[0] += x * x;
      a[1] += x * y;
      a[2] += x * z;
      a[3] += y * y;
      a[4] += y * z;
      a[5] += z * z;
    }
    double nv[3];
    smallest_eigvec(a, nv);
    // orthonormal basis (u, w) of the plane: u = nv x (the axis least aligned with nv)
    const double ax = fabs(nv[0]), ay = fabs(nv[1]), az = fabs(nv[2]);
    const double e0 = (ax <= ay && ax <= az) ? 1.0 : 0.0;
    const double e1 = (e0 == 0.0 && ay <= az) ? 1.0 : 0.0;
    const double e2 = (e0 == 0.0 && e1 == 0.0) ? 1.0 : 0.0;
    double u0 = nv[1] * e2 - nv[2] * e1, u1 = nv[2] * e0 - nv[0] * e2, u2 = nv[0] * e1 - nv[1] * e0;
    const double ul = sqrt(u0 * u0 + u1 * u1 + u2 * u2);
    u0 /= ul;
    u1 /= ul;
    u2 /= ul;
    axes[0][tid] = u0;
    axes[1][tid] = u1;
    axes[2][tid] = u2;
    axes[3][tid] = nv[1] * u2 - nv[2] * u1;
    axes[4][tid] = nv[2] * u0 - nv[0] * u2;
    axes[5][tid] = nv[0] * u1 - nv[1] * u0;
  }
  __syncthreads();
  // From here the four threads of a point are neighbouring lanes of one wavefront.
  const int pt = tid >> 2, l = tid & 3;
  float nx4[kMaxK / 4], ny4[kMaxK / 4], nz4[kMaxK / 4];
#pragma unroll
  for (int k = 0; k < kMaxK / 4; ++k) {
    nx4[k] = nb[0][l + 4 * k][pt];
    ny4[k] = nb[1][l + 4 * k][pt];
    nz4[k] = nb[2][l + 4 * k][pt];
  }
  __syncthreads();
  if (pt >= np) return;
  const int64_t i = base + pt;
  double R = 0.0;
  {
    const double px = P[i], py = P[n + i], pz = P[2 * n + i];
    const double u0 = axes[0][pt], u1 = axes[1][pt], u2 = axes[2][pt];
    const double w0 = axes[3][pt], w1 = axes[4][pt], w2 = axes[5][pt];
#pragma unroll
    for (int k = 0; k < kMaxK / 4; ++k) {
      const int t = l + 4 * k;
      if (t >= m) continue;
      const double dx = nx4[k] - px, dy = ny4[k] - py, dz = nz4[k] - pz;
      const double x = dx * u0 + dy * u1 + dz * u2, y = dx * w0 + dy * w1 + dz * w2;
      qs[t][pt] = make_double2(x, y);
      const double r = sqrt(x * x + y * y);
      R = r > R ? r : R;
    }
  }
  for (int o = 1; o < 4; o <<= 1) {
    const double r = __shfl_xor(R, o, 64);
    R = r > R ? r : R;
  }
  wave_lds_fence();
  if (!(R > 0.0)) {
    if (l == 0) area[i] = 0.0f;
    return;
  }
  // Cell = the square [-R, R]^2 cut by the half-planes x . q_t <= |q_t|^2 / 2 (the bisectors
  // with the projected neighbours). The origin lies strictly inside every constraint, so the
  // cell is star-shaped about it and its area is the sum over its edges of
  // (1/2) x (distance of the edge's line from the origin) x (edge length). Each line's edge is
  // the interval of the line that the other constraints leave: with x = f + s tau (f the foot
  // of the perpendicular from the origin, tau = (-n_y, n_x)), a constraint n_u . x <= b_u bounds
  // s by num / den from one side, and the edge contributes b_t (s_max - s_min) / 2. The bounds
  // are compared as fractions of positive denominators and divided once per line. A line repeated
  // exactly (a repeated neighbour) counts once; a coincident neighbour (q = 0) bounds nothing.
  const int lines = m + 4;  // neighbour bisectors, then the square's 4 edges
  double s2 = 0.0;  // twice the area
  for (int t = l; t < lines; t += 4) {
    const int e = t - m;
    double ax = e == 0 ? 1.0 : (e == 1 ? -1.0 : 0.0), ay = e == 2 ? 1.0 : (e == 3 ? -1.0 : 0.0), bt = R;
    if (e < 0) {
      ax = qs[t][pt].x;
      ay = qs[t][pt].y;
      bt = 0.5 * (ax * ax + ay * ay);  // 0: no constraint
    }
    if (bt == 0.0) continue;
    const double l2 = ax * ax + ay * ay;
    const double fx = ax * bt / l2, fy = ay * bt / l2;
    const double tx = -ay, ty = ax;
    // s_max = hn / hd, s_min = -ln / ld; no bound yet: +- 1 / 0
    double hn = 1.0, hd = 0.0, ln = 1.0, ld = 0.0;
    bool empty = false;
    auto bound = [&](bool high, bool low, double num, double pd) {
      const bool less = num * (high ? hd : ld) < (high ? hn : ln) * pd;
      hn = high && less ? num : hn;
      hd = high && less ? pd : hd;
      ln = low && less ? num : ln;
      ld = low && less ? pd : ld;
    };
    for (int u = 0; u < m; ++u) {
      const double2 q = qs[u][pt];
      const double bu = 0.5 * (q.x * q.x + q.y * q.y);
      const bool same = q.x == ax && q.y == ay && bu == bt;
      empty = empty || (same && u < t);  // only its first copy has an edge
      const bool cuts = !same && bu != 0.0;
      const double den = tx * q.x + ty * q.y;
      const double num = bu - (fx * q.x + fy * q.y);
      bound(cuts && den > 0.0, cuts && den < 0.0, num, fabs(den));
      empty = empty || (cuts && den == 0.0 && num < 0.0);  // parallel and outside
    }
    // the square: x <= R and x >= -R, y likewise (num = 0 for an edge of its own line)
    bound(tx > 0.0, tx < 0.0, R - fx, fabs(tx));
    bound(tx < 0.0, tx > 0.0, R + fx, fabs(tx));
    bound(ty > 0.0, ty < 0.0, R - fy, fabs(ty));
    bound(ty < 0.0, ty > 0.0, R + fy, fabs(ty));
    empty = empty || (tx == 0.0 && (fx > R || fx < -R)) || (ty == 0.0 && (fy > R || fy < -R));
    const double smax = hn / hd, smin = -(ln / ld);
    if (!empty && smax > smin) s2 += bt * (smax - smin);
  }
  for (int o = 1; o < 4; o <<= 1) s2 += __shfl_xor(s2, o, 64);
  if (l == 0) area[i] = (float)(0.5 * s2);
}

// Gauss map (Sec. 5.1 "Normal Initialization"): n_i = p_i / |p_i| (about the origin);
// a point at the origin gets (0, 0, 1).
__global__ void k_gauss_normals(const float* __restrict__ P, int64_t n, float* __restrict__ N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double x = P[i], y = P[n + i], z = P[2 * n + i];
  const double r = sqrt(x * x + y * y + z * z);
  if (r > 0.0) {
    N[i] = (float)(x / r);
    N[n + i] = (float)(y / r);
    N[2 * n + i] = (float)(z / r);
  } else {
    N[i] = 0.0f;
    N[n + i] = 0.0f;
    N[2 * n + i] = 1.0f;
  }
}

unsigned grid_for(int64_t n, int block = 256, int64_t cap = 65535) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, block), cap));
}

// Half-width of the cube searched by the thread-per-query pass: its 27 cells hold the answer of
// nearly every query that is not isolated, and one more ring costs every wavefront with one
// unfinished query 16 more rows (2 against 1, at 0.5 k points per cell, us: the 10 nearest of 50,001
// points 213 against 141, the radius of 1M points 402 against 384).
constexpr int kFirstPassRings = 1;

// Blocks of the wavefront-per-item pass (4 wavefronts each): 8 wavefronts per SIMD, so that
// the dependent loads of one item's ring walk overlap with those of others.
constexpr int kWaveBlocks = 2048;

// Queries from which putting them in cell order pays: the four launches of the sort take about
// 20 us and as much again per 1M queries.
constexpr int64_t kOrderMin = 16384;

// How the queries of a search are ordered: kOwnOrder = they are the references (work in cell
// order), kAnyOrder = no order (sorted first when there are enough), kGivenOrder = already in a
// spatial order that also groups the isolated queries (the level-set faces, emitted cell by cell in
// Morton order): the thread-per-query kernel then searches every query to the end (no limit,
// nothing deferred), since a wavefront per deferred query would only spread those out.
enum QueryOrder { kOwnOrder, kAnyOrder, kGivenOrder };

template <int K>
void launch_knn_k(hipStream_t st, const QuerySet& qs, const KnnWork& w, int rcap, const KnnEmit& em) {
  const dim3 grid((unsigned)cdiv(qs.m, 256));
  if (em.mode == kEmitMean || em.mode == kEmitWindow)
    hipLaunchKernelGGL((k_knn<K, DistList<K>>), grid, dim3(256), 0, st, qs, w.gp, w.start, w.sorted, rcap, w.defer, em);
  else
    hipLaunchKernelGGL((k_knn<K, PairList<K>>), grid, dim3(256), 0, st, qs, w.gp, w.start, w.sorted, rcap, w.defer, em);
}

// Grid of the nr references R for searches of k neighbours.
dwg_status build_grid(const float* R, int64_t nr, int k, const KnnWork& w, hipStream_t st) {
  const int64_t mc = max_cells_for(nr);
  if (nr <= kSmallRefs) {
    hipLaunchKernelGGL(k_grid_small, dim3(1), dim3(kSetupBlock), 0, st, R, nr, mc, k, w.gp, w.start, w.sorted,
                       w.total, w.defer);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  hipLaunchKernelGGL(k_grid_setup, dim3(1), dim3(kSetupBlock), 0, st, R, nr, mc, k, w.gp);
  DWG_TRY_LAUNCH();
  // the launches cover the largest possible grid (the actual one has <= mc cells)
  hipLaunchKernelGGL(k_grid_zero, dim3(grid_for(mc + 1, 256, 1024)), dim3(256), 0, st, w.gp, w.start, w.state,
                     w.total, w.defer);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_cell_count, dim3(grid_for(nr)), dim3(256), 0, st, R, nr, w.gp, w.key, w.rank, w.start);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_scan_chain, dim3((unsigned)cdiv(mc, kScanTile)), dim3(kScanBlock), 0, st, w.start, mc, w.gp,
                     w.state);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_scatter, dim3(grid_for(nr)), dim3(256), 0, st, R, nr, w.key, w.rank, w.start, w.sorted);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

// kOwnOrder: the queries are exactly the m references of the grid, q0 = 0, skip_mode 1. first: no search
// has used the grid since it was built.
dwg_status knn_query(const float* Q, int64_t qld, int64_t q0, int64_t m, const KnnWork& w, int skip_mode,
                     int64_t stride, int k, const KnnEmit& em, hipStream_t st, QueryOrder order, bool first = false) {
  if (m > w.mq) {  // the deferred list holds at most w.mq items
    set_error("internal: %lld kNN queries exceed the carved capacity %lld", (long long)m, (long long)w.mq);
    return DWG_E_INVALID;
  }
  if (m <= 0) return DWG_OK;
  QuerySet qs{Q, qld, q0, m, order == kOwnOrder ? w.sorted : nullptr, skip_mode, stride};
  if (order != kGivenOrder && !first) {
    hipLaunchKernelGGL(k_order_clear, dim3(kBuckets / 256), dim3(256), 0, st, w.total, w.defer);
    DWG_TRY_LAUNCH();
  }
  if (order == kAnyOrder && m >= kOrderMin) {
    const dim3 grid((unsigned)cdiv(m, kOrderTile)), block(kOrderBlock);
    hipLaunchKernelGGL((k_order<false>), grid, block, 0, st, qs, w.gp, w.total, w.items);
    DWG_TRY_LAUNCH();
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneBlock), 0, st, w.total, (int64_t)kBuckets);
    DWG_TRY_LAUNCH();
    hipLaunchKernelGGL((k_order<true>), grid, block, 0, st, qs, w.gp, w.total, w.items);
    DWG_TRY_LAUNCH();
    qs.items = w.items;
  }
  const int rcap = order == kGivenOrder ? INT_MAX : kFirstPassRings;
  switch (k) {
#define DWG_K(KK) \
  case KK: launch_knn_k<KK>(st, qs, w, rcap, em); break;
    DWG_K(1) DWG_K(2) DWG_K(3) DWG_K(4) DWG_K(5) DWG_K(6) DWG_K(7) DWG_K(8)
    DWG_K(9) DWG_K(10) DWG_K(11) DWG_K(12) DWG_K(13) DWG_K(14) DWG_K(15) DWG_K(16)
#undef DWG_K
    default: set_error("k out of range"); return DWG_E_INVALID;
  }
  DWG_TRY_LAUNCH();
  if (order != kGivenOrder) {
    hipLaunchKernelGGL(k_knn_wave, dim3(kWaveBlocks), dim3(256), 0, st, qs, w.gp, w.start, w.sorted, w.defer, k, em);
    DWG_TRY_LAUNCH();
  }
  return DWG_OK;
}

KnnEmit emit_list(int32_t* idx, float* dist) { return KnnEmit{kEmitList, idx, dist, nullptr, 0.0f, 0.0f, 0.0f}; }
KnnEmit emit_mean(float* delta, float scale) { return KnnEmit{kEmitMean, nullptr, nullptr, delta, scale, 0.0f, 0.0f}; }

// Grid over R, then the k nearest references of each of the m queries (self_skip: R itself).
dwg_status knn_emit(const float* R, int64_t nr, const float* Q, int64_t m, int self_skip, int k, const KnnEmit& em,
                    void* ws, hipStream_t stream) {
  Carver c(ws);
  KnnWork w;
  carve_knn(c, nr, m, &w);
  dwg_status s = build_grid(R, nr, k, w, stream);
  if (s != DWG_OK) return s;
  // queries that are the references themselves (same array, same count) run in cell order
  const QueryOrder order = self_skip && Q == R && m == nr ? kOwnOrder : kAnyOrder;
  return knn_query(Q, m, 0, m, w, self_skip ? 1 : 0, 1, k, em, stream, order, true);
}

}  // namespace

dwg_status knn_grid(const float* R, int64_t nr, int k, const KnnWork& w, hipStream_t st) {
  return build_grid(R, nr, k, w, st);
}

dwg_status knn_search(const float* Q, int64_t qld, int64_t q0, int64_t m, const KnnWork& w, int k, int32_t* idx,
                      float* dist, hipStream_t st) {
  return knn_query(Q, qld, q0, m, w, 0, 1, k, emit_list(idx, dist), st, kGivenOrder);
}

size_t carve_knn(Carver& c, int64_t nr, int64_t mq, KnnWork* out) {
  const int64_t mc = max_cells_for(nr);
  const size_t s0 = c.used;
  KnnWork w;
  w.mq = mq;
  w.defer = c.take<int32_t>((size_t)mq + 1);
  w.gp = c.take<GridParams>(1);
  w.key = c.take<int32_t>((size_t)nr);
  w.rank = c.take<int32_t>((size_t)nr);
  w.start = c.take<int32_t>((size_t)mc + 1);
  w.state = c.take<unsigned long long>((size_t)cdiv(mc, kScanTile) + 1);
  w.sorted = c.take<float4>((size_t)nr);
  w.total = c.take<int32_t>((size_t)kBuckets + 1);
  w.items = c.take<float4>((size_t)mq);
  if (out) *out = w;
  return c.used - s0;
}

dwg_status launch_bbox(const float* R, int64_t n, float* part, float* out6, hipStream_t st) {
  hipLaunchKernelGGL(k_bbox_partial, dim3(kBboxBlocks), dim3(256), 0, st, R, n, part);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(256), 0, st, part, kBboxBlocks, out6);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

size_t scan_sums_len(int64_t n) { return 2 * ((size_t)cdiv(n, kScanTile) + 1); }

dwg_status exclusive_scan(int32_t* a, int64_t n, int32_t* sums, hipStream_t st) {
  if (n <= kScanOneMax) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kScanOneBlock), 0, st, a, n);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  const int64_t words = (int64_t)scan_sums_len(n);
  hipLaunchKernelGGL(k_zero_i32, dim3(grid_for(words)), dim3(256), 0, st, sums, words);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_scan_chain, dim3((unsigned)cdiv(n, kScanTile)), dim3(kScanBlock), 0, st, a, n,
                     static_cast<const GridParams*>(nullptr), reinterpret_cast<unsigned long long*>(sums));
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

size_t knn_ws_bytes(int64_t n_ref, int64_t n_qry) {
  (void)n_qry;
  Carver c(nullptr);
  carve_knn(c, n_ref, n_qry, nullptr);
  return c.used;
}

dwg_status knn_run(const float* R, int64_t nr, const float* Q, int64_t m, int self_skip, int k, int32_t* idx,
                   float* dist, void* ws, hipStream_t stream) {
  return knn_emit(R, nr, Q, m, self_skip, k, emit_list(idx, dist), ws, stream);
}

dwg_status delta_mean(const float* P, int64_t n, int k, float scale, float* delta, void* ws, hipStream_t stream) {
  return knn_emit(P, n, P, n, 1, k, emit_mean(delta, scale), ws, stream);
}

size_t anchor_ws_bytes(int64_t n, int64_t chunk, int64_t n_anchor) {
  Carver c(nullptr);
  AnchorCtx x;
  carve_anchor(c, n, chunk, n_anchor, &x);
  return c.used;
}

size_t carve_anchor(Carver& c, int64_t n, int64_t chunk, int64_t n_anchor, AnchorCtx* out) {
  const size_t s0 = c.used;
  AnchorCtx x;
  x.stride = std::max<int64_t>(1, n / std::max<int64_t>(n_anchor, 1));
  x.na = cdiv(n, x.stride);
  x.chunk = chunk;
  x.A = c.take<float>(3 * (size_t)x.na);
  x.A4 = c.take<float4>((size_t)x.na);
  x.idx = c.take<int32_t>((size_t)chunk * DWG_FEAT_K);
  x.inv = c.take<float>((size_t)chunk);
  carve_knn(c, x.na, chunk, &x.w);
  if (out) *out = x;
  return c.used - s0;
}

dwg_status pca_normals(const float* P, int64_t n, int k, float* N, void* ws, hipStream_t stream) {
  Carver c(ws);
  int32_t* idx = c.take<int32_t>((size_t)n * k);
  dwg_status s = knn_run(P, n, P, n, 1, k, idx, nullptr, static_cast<char*>(ws) + c.used, stream);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_pca_normals, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, stream, P, n, idx, k, N);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status voronoi_area(const float* P, int64_t n, int m, float* area, void* ws, hipStream_t stream) {
  Carver c(ws);
  int32_t* idx = c.take<int32_t>((size_t)n * m);
  dwg_status s = knn_run(P, n, P, n, 1, m, idx, nullptr, static_cast<char*>(ws) + c.used, stream);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_voronoi_area, dim3((unsigned)cdiv(n, kCellPoints)), dim3(4 * kCellPoints), 0, stream, P, n,
                     idx, m, area);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status delta_window(const float* P, int64_t n, int k, float vmin, float vmax, float* delta, void* ws,
                        hipStream_t stream) {
  return knn_emit(P, n, P, n, 1, k, KnnEmit{kEmitWindow, nullptr, nullptr, delta, 0.0f, vmin, vmax}, ws, stream);
}

dwg_status gauss_normals(const float* P, int64_t n, float* N, hipStream_t stream) {
  hipLaunchKernelGGL(k_gauss_normals, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, stream, P, n, N);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

// Anchors: every stride-th point, stride = max(1, n / n_anchor); their grid, for searches of k.
dwg_status anchor_build(const float* P, int64_t n, int k, const AnchorCtx& x, hipStream_t stream) {
  hipLaunchKernelGGL(k_gather_anchors, dim3((unsigned)cdiv(x.na, 256)), dim3(256), 0, stream, P, n, x.stride,
                     x.na, x.A, x.A4);
  DWG_TRY_LAUNCH();
  return build_grid(x.A, x.na, k, x.w, stream);
}

// The 16 nearest anchors of the points q0 .. q0 + m - 1 (m <= chunk) into x.idx, and the inverse of
// their mean distance into x.inv.
dwg_status anchor_lists(const float* P, int64_t n, int64_t q0, int64_t m, const AnchorCtx& x, hipStream_t stream) {
  return knn_query(P, n, q0, m, x.w, 2, x.stride, DWG_FEAT_K, KnnEmit{kEmitScaled, x.idx, nullptr, x.inv, 0.0f, 0.0f, 0.0f},
                   stream, kAnyOrder);
}

// Features of the points q0 .. q0 + m - 1 (m <= chunk) into feat [m][48].
dwg_status anchor_features(const float* P, int64_t n, int64_t q0, int64_t m, const AnchorCtx& x, float* feat,
                           hipStream_t stream) {
  dwg_status s = anchor_lists(P, n, q0, m, x, stream);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_features, dim3((unsigned)std::min<int64_t>(cdiv(m * DWG_FEAT_K, 256), 65535)), dim3(256), 0,
                     stream, P, n, q0, m, x.A4, x.idx, x.inv, feat);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

// delta_i = scale x mean distance from p_i to its k nearest anchors (the anchor i itself
// excluded), for all points in chunks of x.chunk.
dwg_status anchor_delta(const float* P, int64_t n, const AnchorCtx& x, int k, float scale, float* delta,
                        hipStream_t stream) {
  for (int64_t q0 = 0; q0 < n; q0 += x.chunk) {
    const int64_t cnt = std::min<int64_t>(x.chunk, n - q0);
    dwg_status s = knn_query(P, n, q0, cnt, x.w, 2, x.stride, k, emit_mean(delta + q0, scale), stream, kAnyOrder);
    if (s != DWG_OK) return s;
  }
  return DWG_OK;
}

dwg_status features_run(const float* P, int64_t n, int64_t n_anchor, float* feat, void* ws, hipStream_t stream) {
  Carver c(ws);
  AnchorCtx x;
  carve_anchor(c, n, n, n_anchor, &x);
  dwg_status s = anchor_build(P, n, DWG_FEAT_K, x, stream);
  if (s != DWG_OK) return s;
  return anchor_features(P, n, 0, n, x, feat, stream);
}

}  // namespace dwg
