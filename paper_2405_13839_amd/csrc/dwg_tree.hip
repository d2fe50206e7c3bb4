// Octree evaluation of the (screened) GWN and its gradient (Sec. 5.2 "Octree Traversal",
// after the fast winding numbers of Barill et al. 2018).
//
// Octree. The root cell is the cube [lo, lo + ext]^3 (lo = per-axis minimum of the sources,
// ext = largest per-axis extent). A source's cell at the deepest level D = 21 has integer
// coordinates floor((x - lo) * 2^21 / ext) clamped to [0, 2^21 - 1], computed in FP64; its
// 63-bit Morton code interleaves them with x the most significant bit of each triple.
// Sources are sorted by (code, index). A node is a non-empty cell, a leaf when it holds at
// most `leaf` sources or sits at level D; a cell whose sources all lie in one child cell is
// represented by the deepest cell of that chain (same sources, so the same summaries and
// decisions), which bounds the node count by 2n - 1. Nodes are numbered in depth-first
// pre-order; a node's first child is the next node and `skip` is the first node after its
// subtree.
//
// Build (once per source set), all flat and deterministic:
//   codes -> stable LSD radix sort (8 passes of 8 bits; ranks inside a block from wave
//   ballots) -> per sorted source, the range of levels of the nodes that start there ->
//   exclusive scan -> nodes in pre-order. A node at level L starting at sorted position i
//   exists iff i starts its level-L cell and the parent cell holds more than `leaf`
//   sources; the deepest level at which the cell of i holds more than `leaf` sources is the
//   largest shared prefix of the codes at positions (j, j + leaf) over windows containing i.
// Node summaries (Sec. 5.2): area A and area-weighted centre c.m, FP64 sums in a fixed order;
// r = largest |p_j - c.m| (FP64);
// dmax = largest kernel radius max(delta_j, eps); opening radius crit = max(beta r, r + dmax)
// (the second term keeps every source of a far node outside its clamp radius). Per
// iteration, the moment M = sum m_j (m_j = a_j n_j / 4 pi, FP64 sums of the staged FP32
// moments).
//
// Traversal. One wavefront walks the pre-order node list with one node index for all 64 of
// its queries (sorted, so they are neighbours) and per-lane "skip until" indices: a lane
// for which node i is far adds the node's dipole and ignores the rest of its subtree; the
// wave descends (i + 1) when any active lane must open node i, sums a leaf's sources for the
// lanes that opened it, and otherwise jumps to skip. Every query thus sees exactly the
// per-query decisions of the paper's depth-first traversal; node loads are wave-uniform.
// A leaf opened by at most half of the lanes is spread over the idle ones (groups of lanes
// each take every k-th source for one query; partial sums return through LDS).
// The FP64 criterion |q - c.m|^2 > crit^2 decides (unscaled); the far dipole and the leaf
// pairs use the FP32 pair arithmetic of the all-pairs kernel in its scaled coordinates (leaf
// pairs from positions staged relative to the leaf's centre).
#include <cmath>

#include "dwg_internal.h"
#include "dwg_morton.h"
#include "dwg_pair.h"

namespace dwg {
namespace {

using namespace pairk;
using morton::kDepth;

// Node count written by the build, never above the carved capacity.
__device__ __forceinline__ int64_t node_count(const int32_t* total_p, int64_t cap) {
  const int64_t t = *total_p;
  return t < cap ? t : cap;
}

unsigned grid_cap(int64_t n, int64_t cap = 16384) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, 256), cap));
}

// Blocks of the kernels that take a node per 16 lanes. How many nodes there are is known on the
// device only: about n / 4 at 16 sources a leaf on a surface, 2 n at most.
unsigned node_grid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, 32), 16384)); }

// Number of levels 1..D at which codes a and b share their cell (D when equal).
__device__ __forceinline__ int shared_levels(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  if (x == 0) return kDepth;
  const int h = 63 - __clzll((long long)x);
  return kDepth - h / 3 - 1;
}

// End (exclusive) of the level-L cell that contains sorted position i.
__device__ int64_t cell_end(const uint64_t* __restrict__ code, int64_t n, int64_t i, int L) {
  if (L == 0) return n;
  const int sh = 3 * (kDepth - L);
  const uint64_t pre = code[i] >> sh;
  int64_t lo = i + 1, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((code[mid] >> sh) == pre)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// frame = (lo x, lo y, lo z, 2^21 / ext), ext = the largest extent (scale 0 when ext == 0).
__global__ void k_tree_frame(const float* __restrict__ box, double* __restrict__ frame) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double ex = (double)box[3] - (double)box[0];
  const double ey = (double)box[4] - (double)box[1];
  const double ez = (double)box[5] - (double)box[2];
  double ext = ex;
  if (ey > ext) ext = ey;
  if (ez > ext) ext = ez;
  frame[0] = box[0];
  frame[1] = box[1];
  frame[2] = box[2];
  frame[3] = ext > 0.0 ? 2097152.0 / ext : 0.0;
}

__global__ void k_tree_keys(const float* __restrict__ P, int64_t n, const double* __restrict__ frame,
                            uint64_t* __restrict__ key) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c[3];
    morton::cell21(P, n, i, frame, c);
    key[i] = morton::code3(c[0], c[1], c[2]);
  }
}

// Per sorted source i: the levels [ldiff, lend] of the uncompressed nodes starting at i and
// the number of kept (deepest-of-chain) nodes among them.
__global__ void k_tree_mark(const uint64_t* __restrict__ code, int64_t n, int leaf, int32_t* __restrict__ lev,
                            int32_t* __restrict__ cnt) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int ldiff = i == 0 ? 0 : shared_levels(code[i - 1], code[i]) + 1;
    int deep = -1;
    const int64_t j0 = i - leaf > 0 ? i - leaf : 0;
    const int64_t j1 = i < n - 1 - leaf ? i : n - 1 - leaf;
    for (int64_t j = j0; j <= j1; ++j) {
      const int s = shared_levels(code[j], code[j + leaf]);
      deep = s > deep ? s : deep;
    }
    const int lend = deep + 1 < kDepth ? deep + 1 : kDepth;
    int c = 0;
    if (ldiff <= lend) {
      int64_t e = cell_end(code, n, i, ldiff);
      for (int L = ldiff; L < lend; ++L) {
        const int64_t e2 = cell_end(code, n, i, L + 1);
        if (e2 != e) ++c;
        e = e2;
      }
      ++c;
    }
    lev[i] = ldiff | (lend << 8);
    cnt[i] = c;
  }
}

// Writes the kept nodes: (start, end, skip, level | leaf << 8).
__global__ void k_tree_emit(const uint64_t* __restrict__ code, int64_t n, int leaf, const int32_t* __restrict__ lev,
                            const int32_t* __restrict__ off, int64_t cap, int4* __restrict__ node) {
  const int32_t total = off[n];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int ldiff = lev[i] & 255, lend = lev[i] >> 8;
    if (ldiff > lend) continue;
    int64_t k = off[i];
    int64_t e = cell_end(code, n, i, ldiff);
    for (int L = ldiff; L <= lend; ++L) {
      const int64_t e2 = L < lend ? cell_end(code, n, i, L + 1) : -1;
      if (L == lend || e2 != e) {
        if (k < cap) {
          const int skip = e == n ? total : off[e];
          const int lf = (e - i <= leaf || L == kDepth) ? 1 : 0;
          node[k] = make_int4((int)i, (int)e, skip, L | (lf << 8));
        }
        ++k;
      }
      e = e2;
    }
  }
}

// FP64 sums over nodes. A node of at most kGroupSources sources is summed by the 16 lanes of a
// DPP row, four nodes to a wavefront; a larger one by its whole wavefront, whole tiles of
// kSumTile sorted sources from their sums, which a launch before has formed. (A thread per chunk
// of 256 sources, adding them one after another through the permutation, bounded the build:
// 1.88 ms for the summaries of 1M sources, 225 us of 20,011, however few the chunks were; 167 and
// 40 us now. Per iteration the moments took 45 and 18 us as differences of FP64 prefix sums, 37
// and 10 now.) The sums' order is fixed by the node's position alone.
constexpr int kSumTile = 256;
constexpr int kGroupSources = 64;

template <int N>
__device__ __forceinline__ double row_ror(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over the row's 16 lanes, the same bits in each.
__device__ __forceinline__ double row_sum(double v) {
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) {
    const double x = __shfl_xor(v, o, 64);
    v = x > v ? x : v;
  }
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// What is summed: add(j, x) adds the K values of sorted source j.
struct MomentSum {  // the staged moments
  static constexpr int K = 3;
  const float4* __restrict__ src;
  __device__ __forceinline__ void add(int64_t j, double* x) const {
    const float4 b = src[2 * j + 1];
    x[0] += b.x;
    x[1] += b.y;
    x[2] += b.z;
  }
};
struct AreaSum {  // a, a px, a py, a pz
  static constexpr int K = 4;
  const float4* __restrict__ pos;
  __device__ __forceinline__ void add(int64_t j, double* x) const {
    const float4 p = pos[j];
    const double a = p.w;
    x[0] += a;
    x[1] += a * (double)p.x;
    x[2] += a * (double)p.y;
    x[3] += a * (double)p.z;
  }
};

// Sums v of the node [s, e) of this lane's row (e = s: no node), in every lane of the row.
template <class F>
__device__ __forceinline__ void node_sum(const F& f, const double* __restrict__ tile, int s, int e, double* v) {
  const int lane = threadIdx.x & 63, l = lane & 15;
  const bool big = e - s > kGroupSources;
#pragma unroll
  for (int c = 0; c < F::K; ++c) v[c] = 0.0;
  if (!big)
    for (int j = s + l; j < e; j += 16) f.add(j, v);
#pragma unroll
  for (int c = 0; c < F::K; ++c) v[c] = row_sum(v[c]);
  for (uint64_t todo = __ballot(big && l == 0); todo; todo &= todo - 1) {
    const int who = __ffsll((unsigned long long)todo) - 1;
    const int bs = __builtin_amdgcn_readlane(s, who), be = __builtin_amdgcn_readlane(e, who);
    int t0 = (bs + kSumTile - 1) / kSumTile, t1 = be / kSumTile;  // whole tiles of the node
    const int head = t0 < t1 ? t0 * kSumTile : be, tail = t0 < t1 ? t1 * kSumTile : be;
    double x[F::K];
#pragma unroll
    for (int c = 0; c < F::K; ++c) x[c] = 0.0;
    for (int j = bs + lane; j < head; j += 64) f.add(j, x);
    for (int t = t0 + lane; t < t1; t += 64)
#pragma unroll
      for (int c = 0; c < F::K; ++c) x[c] += tile[(int64_t)t * 4 + c];
    for (int j = tail + lane; j < be; j += 64) f.add(j, x);
#pragma unroll
    for (int c = 0; c < F::K; ++c) {
      const double total = wave_sum(x[c]);
      if ((lane >> 4) == (who >> 4)) v[c] = total;
    }
  }
}

// Tile sums, a wavefront per tile; the first launch of an evaluation, so it notes the clock.
template <class F>
__global__ __launch_bounds__(256) void k_tile_sums(F f, int64_t n, int64_t tiles, double* __restrict__ tile,
                                                   const int32_t* __restrict__ stop, uint64_t* __restrict__ begin) {
  if (*stop) return;
  if ((blockIdx.x | threadIdx.x) == 0) *begin = wall_clock64();
  const int lane = threadIdx.x & 63;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < tiles; t += (int64_t)gridDim.x * 4) {
    double x[F::K];
#pragma unroll
    for (int c = 0; c < F::K; ++c) x[c] = 0.0;
#pragma unroll
    for (int u = 0; u < kSumTile / 64; ++u) {
      const int64_t j = t * kSumTile + u * 64 + lane;
      if (j < n) f.add(j, x);
    }
#pragma unroll
    for (int c = 0; c < F::K; ++c) {
      x[c] = wave_sum(x[c]);
      if (lane == 0) tile[4 * t + c] = x[c];
    }
  }
}

// Sorted copies of the sources (position and area; radius max(delta, eps)) and their tile sums.
// The gathers bound it (five scattered words a source, four sources in flight a lane): 73 us for
// 1M sources.
__global__ __launch_bounds__(256) void k_tree_sorted(const float* __restrict__ P, const float* __restrict__ area,
                                                     const float* __restrict__ D, float eps,
                                                     const int32_t* __restrict__ val, int64_t n, int64_t tiles,
                                                     int32_t* __restrict__ perm, float4* __restrict__ pos,
                                                     float* __restrict__ rad, double* __restrict__ tile) {
  const int lane = threadIdx.x & 63;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < tiles; t += (int64_t)gridDim.x * 4) {
    double x[4] = {0.0, 0.0, 0.0, 0.0};
    float4 p[kSumTile / 64];
    float d[kSumTile / 64];
#pragma unroll
    for (int u = 0; u < kSumTile / 64; ++u) {
      const int64_t j = t * kSumTile + u * 64 + lane;
      const int64_t o = val[j < n ? j : n - 1];
      p[u] = make_float4(P[o], P[n + o], P[2 * n + o], area[o]);
      d[u] = D ? D[o] : 0.0f;
      if (j < n) perm[j] = (int32_t)o;
    }
#pragma unroll
    for (int u = 0; u < kSumTile / 64; ++u) {
      const int64_t j = t * kSumTile + u * 64 + lane;
      if (j >= n) continue;
      pos[j] = p[u];
      rad[j] = d[u] > eps ? d[u] : eps;
      const double a = p[u].w;
      x[0] += a;
      x[1] += a * (double)p[u].x;
      x[2] += a * (double)p[u].y;
      x[3] += a * (double)p[u].z;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[c] = wave_sum(x[c]);
      if (lane == 0) tile[4 * t + c] = x[c];
    }
  }
}

__device__ __forceinline__ double distance(const float4& p, double gx, double gy, double gz) {
  const double ex = (double)p.x - gx, ey = (double)p.y - gy, ez = (double)p.z - gz;
  return sqrt(ex * ex + ey * ey + ez * ez);
}

// Squared opening radius max(beta r, r + dmax)^2.
__device__ __forceinline__ double opening2(double r, double dm, double beta) {
  double crit = beta * r;
  if (r + dm > crit) crit = r + dm;
  return crit * crit;
}

// Node centres, and the opening radii of nodes up to kSumTile sources; larger nodes' maxima are
// cleared for k_tree_far. 32 us for the nodes of 1M sources.
__global__ __launch_bounds__(256) void k_tree_geo(const int4* __restrict__ node, const int32_t* __restrict__ total_p,
                                                  int64_t cap, AreaSum f, const float* __restrict__ rad,
                                                  const double* __restrict__ tile, double beta,
                                                  double4* __restrict__ geo, unsigned long long* __restrict__ rbits,
                                                  uint32_t* __restrict__ dbits) {
  const int64_t total = node_count(total_p, cap);
  const int lane = threadIdx.x & 63, l = lane & 15;
  const int64_t step = (int64_t)gridDim.x * 16;
  for (int64_t k0 = ((int64_t)blockIdx.x * 256 + (threadIdx.x & ~63)) >> 4; k0 < total; k0 += step) {
    const int64_t k = k0 + (lane >> 4);
    int s = 0, e = 0;
    if (k < total) {
      const int4 nd = node[k];
      s = nd.x;
      e = nd.y;
    }
    double v[4];
    node_sum(f, tile, s, e, v);
    double gx = 0.0, gy = 0.0, gz = 0.0;
    if (v[0] != 0.0) {
      gx = v[1] / v[0];
      gy = v[2] / v[0];
      gz = v[3] / v[0];
    } else if (s < e) {  // no area: the first source
      const float4 p = f.pos[s];
      gx = p.x;
      gy = p.y;
      gz = p.z;
    }
    double r = 0.0;
    float dm = 0.0f;
    if (e - s <= kGroupSources)
      for (int j = s + l; j < e; j += 16) {
        const double d = distance(f.pos[j], gx, gy, gz);
        r = d > r ? d : r;
        dm = fmaxf(dm, rad[j]);
      }
    for (int o = 8; o > 0; o >>= 1) {
      const double x = __shfl_xor(r, o, 64);
      r = x > r ? x : r;
      dm = fmaxf(dm, __shfl_xor(dm, o, 64));
    }
    const bool mid = e - s > kGroupSources && e - s <= kSumTile;
    for (uint64_t todo = __ballot(mid && l == 0); todo; todo &= todo - 1) {
      const int who = __ffsll((unsigned long long)todo) - 1;
      const int bs = __builtin_amdgcn_readlane(s, who), be = __builtin_amdgcn_readlane(e, who);
      const double cx = __shfl(gx, who, 64), cy = __shfl(gy, who, 64), cz = __shfl(gz, who, 64);
      double x = 0.0;
      float y = 0.0f;
      for (int j = bs + lane; j < be; j += 64) {
        const double d = distance(f.pos[j], cx, cy, cz);
        x = d > x ? d : x;
        y = fmaxf(y, rad[j]);
      }
      x = wave_max(x);
      y = wave_max(y);
      if ((lane >> 4) == (who >> 4)) {
        r = x;
        dm = y;
      }
    }
    if (l == 0 && k < total) {
      geo[k] = make_double4(gx, gy, gz, opening2(r, (double)dm, beta));
      if (e - s > kSumTile) {
        rbits[k] = 0ull;
        dbits[k] = 0u;
      }
    }
  }
}

// r and dmax of the nodes above kSumTile sources: a wavefront holds kFarTile sorted sources, walks
// the pre-order list down to the nodes that hold some of them, and adds its maxima (atomic max of
// the bit patterns, which order like unsigned integers for non-negative values; one that the node
// already has is not sent, since every wavefront of the root's reaches the same address). The
// walk's dependent loads bound it: 56 us for 1M sources, 18 for 20,011.
constexpr int kFarTile = 512;
__global__ __launch_bounds__(64) void k_tree_far(const int4* __restrict__ node, const int32_t* __restrict__ total_p,
                                                 int64_t cap, const float4* __restrict__ pos,
                                                 const float* __restrict__ rad, int64_t n,
                                                 const double4* __restrict__ geo,
                                                 unsigned long long* __restrict__ rbits,
                                                 uint32_t* __restrict__ dbits) {
  const int total = (int)node_count(total_p, cap);
  const int lane = threadIdx.x;
  const int64_t lo = (int64_t)blockIdx.x * kFarTile, hi = lo + kFarTile < n ? lo + kFarTile : n;
  float4 p[kFarTile / 64];
  float d[kFarTile / 64];
#pragma unroll
  for (int u = 0; u < kFarTile / 64; ++u) {
    const int64_t j = lo + u * 64 + lane < n ? lo + u * 64 + lane : n - 1;
    p[u] = pos[j];
    d[u] = rad[j];
  }
  for (int i = 0; i < total;) {
    const int4 nd = node[i];
    const int s = __builtin_amdgcn_readfirstlane(nd.x), e = __builtin_amdgcn_readfirstlane(nd.y);
    const int skip = __builtin_amdgcn_readfirstlane(nd.z);
    if (s >= hi) break;
    if (e <= lo || e - s <= kSumTile) {
      i = skip > i ? skip : i + 1;
      continue;
    }
    const double4 g = geo[i];
    double r = 0.0;
    float dm = 0.0f;
#pragma unroll
    for (int u = 0; u < kFarTile / 64; ++u) {
      const int64_t j = lo + u * 64 + lane;
      const double x = distance(p[u], g.x, g.y, g.z);
      const bool in = j >= s && j < e;
      r = in && x > r ? x : r;
      dm = in ? fmaxf(dm, d[u]) : dm;
    }
    r = wave_max(r);
    dm = wave_max(dm);
    if (lane == 0) {
      const unsigned long long rb = (unsigned long long)__double_as_longlong(r);
      const uint32_t db = __float_as_uint(dm);
      if (rb > __hip_atomic_load(&rbits[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&rbits[i], rb);
      if (db > __hip_atomic_load(&dbits[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&dbits[i], db);
    }
    ++i;
  }
}

__global__ void k_tree_crit(const int4* __restrict__ node, const int32_t* __restrict__ total_p, int64_t cap,
                            double beta, const unsigned long long* __restrict__ rbits,
                            const uint32_t* __restrict__ dbits, double4* __restrict__ geo) {
  const int64_t total = node_count(total_p, cap);
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int4 nd = node[k];
    if (nd.y - nd.x > kSumTile)
      geo[k].w = opening2(__longlong_as_double((long long)rbits[k]), (double)__uint_as_float(dbits[k]), beta);
  }
}

// Node moments for the current normals: M = sum of the staged m_j over the node (FP64).
__global__ __launch_bounds__(256) void k_tree_mom(const int4* __restrict__ node, const int32_t* __restrict__ total_p,
                                                  int64_t cap, MomentSum f, const double* __restrict__ tile,
                                                  const int32_t* __restrict__ stop, float4* __restrict__ mom) {
  if (*stop) return;
  const int64_t total = node_count(total_p, cap);
  const int lane = threadIdx.x & 63;
  const int64_t step = (int64_t)gridDim.x * 16;
  for (int64_t k0 = ((int64_t)blockIdx.x * 256 + (threadIdx.x & ~63)) >> 4; k0 < total; k0 += step) {
    const int64_t k = k0 + (lane >> 4);
    int s = 0, e = 0;
    if (k < total) {
      const int4 nd = node[k];
      s = nd.x;
      e = nd.y;
    }
    double v[3];
    node_sum(f, tile, s, e, v);
    if ((lane & 15) == 0 && k < total) mom[k] = make_float4((float)v[0], (float)v[1], (float)v[2], 0.0f);
  }
}

template <int NA, bool KAHAN>
__device__ __forceinline__ void fold(float* sum, float* cmp, const float* acc) {
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    if (KAHAN) {
      const float y = acc[a] - cmp[a];
      const float t = sum[a] + y;
      cmp[a] = (t - sum[a]) - y;
      sum[a] = t;
    } else {
      sum[a] += acc[a];
    }
  }
}

// Leaf-relative staging of the source positions for the leaf pairs, in place: kappa (p_j - c)
// with c the leaf's centre rounded to FP32, which the traversal also subtracts from the
// query, so a near pair's difference is rounded relative to the leaf's neighbourhood, not to
// |p|. Every sorted source lies in exactly one leaf (one writer per source); .w keeps the
// staged 1/(kappa max(delta, eps)), and the moments beside it are untouched.
__global__ void k_tree_leafpos(const int4* __restrict__ node, const int32_t* __restrict__ total_p, int64_t cap,
                               const double4* __restrict__ geo, float4* __restrict__ src, int64_t n, float kappa) {
  const int64_t total = node_count(total_p, cap);
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int4 nd = node[k];
    if (!(nd.w >> 8)) continue;
    const double4 g = geo[k];
    const float cx = (float)g.x, cy = (float)g.y, cz = (float)g.z;
    const int64_t e = nd.y < n ? nd.y : n;
    for (int64_t j = nd.x; j < e; ++j) {
      const float4 a = src[2 * j];
      src[2 * j] = make_float4(kappa * (a.x - cx), kappa * (a.y - cy), kappa * (a.z - cz), a.w);
    }
  }
}

// Traversal: one thread per sorted query, one node index per wavefront (see the file head).
// Contributions are summed in FP32 into `acc` and folded into the (Kahan-compensated when
// KAHAN) running sums after every kFoldLeaves leaf visits of the wavefront and at the end
// (a fold is 4 VALU per accumulator; folding after every visit was ~2% slower at 1M). The
// next node is usually i + 1 (a node opened, or a leaf, whose skip is i + 1), so its data is
// loaded one step ahead.
//
// The pre-order node list is cut into equal segments, each walked on its own for every
// wavefront of queries, with partial sums per segment that the epilogue adds in order. A segment
// starts inside a subtree: it first goes down from the root to its first node, testing only that
// node's ancestors, to learn which lanes have one of them as a far dipole (that dipole belongs to
// the segment that holds the ancestor). Every node is then taken by the same queries as in one
// walk. What bounds it is the length of one walk where the queries are few (a wavefront of
// 20,011 points walks for 260 us alone, and their 313 wavefronts leave two SIMDs in three
// empty: 265 us a launch as one segment) and the last walks to end where they are many (1M points,
// 15,626 wavefronts: 4.95 ms a launch as one, 4.4 as 9 segments). The rule aims at 131,072
// wavefronts (16,384: 24.8 ms for four launches and the rest of a pass at 1M, 65,536: 24.2, 131,072:
// 23.7, 262,144: 23.9), so the partial sums stay below 28 bytes for each of 2^23 + m queries; of at
// least 64 sources' nodes each, and at most 64 segments, whose partial sums then cost more to add
// than they save. Evaluation / whole iteration, us:
//   points             1,000   2,500   5,000   10,000    20,000    40,000    80,000
//   512 sources, 32   65 / 95 72 / 103 67 / 104 72 / 112 96 / 145 149 / 210 289 / 354
//   128 sources, 64   35 / 65 37 / 70  36 / 76  47 / 92  80 / 134 127 / 200 268 / 348
//   128 sources, 128  35 / 65 37 / 70  36 / 76  46 / 93  81 / 141 135 / 233 271 / 369
//   64 sources, 64    26 / 55 31 / 65  32 / 74  47 / 92  82 / 134 127 / 199 267 / 348
constexpr int kFoldLeaves = 4;
// Threads per block of the traversal: its wavefronts share no data and never wait for each
// other (each has its own LDS area and no barrier), but a block's place on a CU is free only when
// its last wavefront has ended. From kLoneQueries queries on a block is one wavefront (1M points:
// 20.0 against 20.9 ms for four launches and the rest of a pass, a level-set update of 100K points,
// 250K queries, 2.49 against 2.53); below, four (20,011 points: 0.77 against 0.79 ms a pass).
constexpr int kTreeBlock = 256;
constexpr int64_t kLoneQueries = 131072;
constexpr int64_t kSegmentWaves = 131072, kSegmentSources = 64, kMaxSegments = 64;
// A leaf visit is spread over the idle lanes when that saves at least this many iterations.
constexpr int kSplitMinSaved = 2;

// A leaf of ns sources opened by na lanes of a wavefront: the log2 of the number k of lane
// groups its loop is spread over (0 = not spread), the largest power of two with k na <= 64
// and k <= ns, kept only when ceil(ns / k) saves at least kSplitMinSaved iterations.
__device__ __forceinline__ int leaf_split_log2(int na, int ns) {
  if (na < 1 || ns < 2) return 0;
  const int by_lanes = __clz((unsigned)(na - 1)) - 26;  // 6 - ceil(log2 na): 2^j na <= 64
  const int by_sources = 31 - __clz((unsigned)ns);      // floor(log2 ns): 2^j <= ns
  int lk = by_lanes < by_sources ? by_lanes : by_sources;
  if (lk > 0 && ns - ((ns + (1 << lk) - 1) >> lk) < kSplitMinSaved) lk = 0;
  return lk > 0 ? lk : 0;
}

// Workgroups are dealt to the 8 XCDs in turn (block b to XCD b mod 8), and each XCD has an L2
// of its own. XCD x evaluates the x-th contiguous run of the nb query blocks, every segment of
// the node list for its run, so the blocks resident on one XCD hold neighbouring queries, which visit
// nearly the same nodes and leaf sources, and that XCD's L2 holds one region of the tree
// rather than every eighth block's share of all of it. (Dealing the segments to the XCDs as
// well gave some of them the near field of their queries and others only far nodes: twice the
// time at 2 segments.) The launch has tree_grid(nb, segments) blocks; false: this one has nothing to do.
__device__ __forceinline__ bool xcd_block(unsigned b, unsigned nb, unsigned segments, unsigned* block,
                                          unsigned* segment) {
  const unsigned longest = (nb + 7) / 8, q = nb / 8, r = nb % 8, x = b % 8, k = b / 8;
  const unsigned at = k % longest;
  *segment = k / longest;
  *block = x * q + (x < r ? x : r) + at;
  return at < q + (x < r ? 1u : 0u) && *segment < segments;
}
unsigned tree_grid(int64_t nb, int segments) { return (unsigned)(8 * cdiv(nb, 8) * segments); }

// Seven wavefronts per SIMD: left to itself the compiler takes 73 VGPRs (six; 25.5 ms a pass at
// 1M against 23.1), and at eight it spills (25.9).
template <int BLOCK, bool GRAD, bool SCREENED, bool KAHAN>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(7))) void k_tree_eval(
    const float* __restrict__ Q, int64_t m, const int32_t* __restrict__ qperm, const int4* __restrict__ node,
    const double4* __restrict__ geo, const float4* __restrict__ mom, const int32_t* __restrict__ total_p, int64_t cap,
    const float4* __restrict__ src, int64_t n_src, Scr sk, float kappa, float* __restrict__ part, int64_t mpad,
    unsigned segments, const int32_t* __restrict__ stop) {
  if (*stop) return;
  constexpr int NA = GRAD ? kNAcc : 1;
  // per wavefront: the queries of a split leaf visit by rank, and the lanes' partial sums
  __shared__ float4 lds_q[BLOCK / 64][64];
  __shared__ float lds_p[BLOCK / 64][64][NA == 1 ? 1 : 8];
  const int wv = (int)(threadIdx.x >> 6);
  unsigned qblock, segment;
  if (!xcd_block(blockIdx.x, (unsigned)(mpad / BLOCK), segments, &qblock, &segment)) return;
  const int64_t qi = (int64_t)qblock * BLOCK + threadIdx.x;
  const int64_t o = qperm[qi < m ? qi : m - 1];
  const float ux = Q[o], uy = Q[m + o], uz = Q[2 * m + o];
  const double dqx = ux, dqy = uy, dqz = uz;  // the opening test runs in unscaled FP64
  const double dk = kappa;
  float sum[NA], cmp[NA], acc[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) sum[a] = cmp[a] = acc[a] = 0.0f;
  int nn = __builtin_amdgcn_readfirstlane(*total_p);
  if (nn > cap) nn = (int)cap;
  const int first = (int)((int64_t)nn * segment / segments), end = (int)((int64_t)nn * (segment + 1) / segments);
  int skip_to = 0;
  int i = 0;
  while (i < first) {  // down to the segment's first node
    const int nskip = __builtin_amdgcn_readfirstlane(node[i].z);
    if (nskip <= first) {  // a subtree before it
      i = nskip > i ? nskip : i + 1;
      continue;
    }
    if (i >= skip_to) {
      const double4 g = geo[i];
      const double dx = g.x - dqx, dy = g.y - dqy, dz = g.z - dqz;
      if (dx * dx + dy * dy + dz * dz > g.w) skip_to = nskip;
    }
    ++i;
  }
  if (segment > 0) {  // the first node that any lane has left
    int least = skip_to;
    for (int o = 32; o > 0; o >>= 1) least = min(least, __shfl_xor(least, o, 64));
    i = max(i, __builtin_amdgcn_readfirstlane(least));
  }
  nn = end;
  int visits = 0;  // leaf visits of the wavefront since the last fold
  const int i0 = i < nn ? i : 0;
  int4 nd = node[i0];
  double4 g = geo[i0];
  float4 mm = mom[i0];
  while (i < nn) {
    const int nskip = __builtin_amdgcn_readfirstlane(nd.z);
    bool open = false, direct = false;
    if (i >= skip_to) {
      const double dx = g.x - dqx, dy = g.y - dqy, dz = g.z - dqz;
      const double d2 = dx * dx + dy * dy + dz * dz;
      if (d2 > g.w) {
        const float fx = (float)(dk * dx), fy = (float)(dk * dy), fz = (float)(dk * dz);
        if (SCREENED)
          pair_screened_d<GRAD, true>(fx, fy, fz, 0.0f, mm, sk, acc);
        else
          pair_plain_d<GRAD, true>(fx, fy, fz, 0.0f, mm, acc);
        skip_to = nskip;
      } else if (nd.w >> 8) {
        direct = true;
      } else {
        open = true;
      }
    }
    // The next node is loaded only now: scalar loads return out of order, so the wait in
    // front of this step's test covered every scalar load in flight; issued after the test,
    // the next node's loads have the rest of this step to arrive. (Loading the node after
    // this one's subtree too, the other possible successor, cost more registers than it
    // saved.)
    __asm__ __volatile__("" ::: "memory");
    const int nxt = i + 1 < nn ? i + 1 : i;
    const int4 nd1 = node[nxt];
    const double4 g1 = geo[nxt];
    const float4 mm1 = mom[nxt];
    int next;
    if (__any(open)) {
      next = i + 1;
    } else {
      if (__any(direct)) {
        const int s0 = __builtin_amdgcn_readfirstlane(nd.x);
        int s1 = __builtin_amdgcn_readfirstlane(nd.y);
        if (s1 > n_src) s1 = (int)n_src;
        // the query relative to the leaf's centre, as its sources are staged (k_tree_leafpos)
        const float lx = kappa * (ux - (float)g.x), ly = kappa * (uy - (float)g.y), lz = kappa * (uz - (float)g.z);
        // With a lanes opening the leaf, k = 2^lk groups of a lanes (k a <= 64) can take an
        // interleaved k-th of its sources each for one query, in ceil(s / k) iterations
        // instead of s; the groups' partial sums then go back to the querying lanes.
        const uint64_t dmask = __ballot(direct);
        const int lk = __builtin_amdgcn_readfirstlane(leaf_split_log2(__popcll(dmask), s1 - s0));
        if (lk == 0) {
          if (direct) {
            // the lanes that did not open the leaf sit the whole loop out (one exec mask for
            // the loop, not one per source). Two sources per iteration: their scalar loads
            // are waited for once and their rsq and exp issue in pairs (1-3.5% faster than one
            // per iteration at beta 2.3-32); the spread loop below keeps one, as two there
            // take the kernel to 78 VGPRs and 6 wavefronts per SIMD, which ran slower.
            int j = s0;
#pragma unroll 1
            for (; j + 1 < s1; j += 2) {  // two independent sources per iteration
              const float4 a0 = src[2 * (int64_t)j], b0 = src[2 * (int64_t)j + 1];
              const float4 a1 = src[2 * (int64_t)j + 2], b1 = src[2 * (int64_t)j + 3];
              if (SCREENED) {
                pair_screened<GRAD, false>(a0, b0, lx, ly, lz, sk, acc);
                pair_screened<GRAD, false>(a1, b1, lx, ly, lz, sk, acc);
              } else {
                pair_plain<GRAD, false>(a0, b0, lx, ly, lz, acc);
                pair_plain<GRAD, false>(a1, b1, lx, ly, lz, acc);
              }
            }
            if (j < s1) {
              const float4 a = src[2 * (int64_t)j], b = src[2 * (int64_t)j + 1];
              if (SCREENED)
                pair_screened<GRAD, false>(a, b, lx, ly, lz, sk, acc);
              else
                pair_plain<GRAD, false>(a, b, lx, ly, lz, acc);
            }
          }
        } else {
          const int lane = (int)(threadIdx.x & 63);
          const int rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(dmask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned)dmask, 0u));
          float4* qs = lds_q[wv];
          if (direct) qs[rank] = make_float4(lx, ly, lz, 0.0f);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          const int grp = lane & ((1 << lk) - 1), who = lane >> lk;
          float pac[NA];
#pragma unroll
          for (int a = 0; a < NA; ++a) pac[a] = 0.0f;
          if (who < __popcll(dmask)) {
            const float4 qq = qs[who];
#pragma unroll 1
            for (int j = s0 + grp; j < s1; j += 1 << lk) {
              const float4 a = src[2 * (int64_t)j], b = src[2 * (int64_t)j + 1];
              if (SCREENED)
                pair_screened<GRAD, false>(a, b, qq.x, qq.y, qq.z, sk, pac);
              else
                pair_plain<GRAD, false>(a, b, qq.x, qq.y, qq.z, pac);
            }
          }
          float* ps = lds_p[wv][lane];
#pragma unroll
          for (int a = 0; a < NA; ++a) ps[a] = pac[a];
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          if (direct) {
#pragma unroll 1
            for (int gi = 0; gi < (1 << lk); ++gi) {
              const float* pg = lds_p[wv][(rank << lk) + gi];
#pragma unroll
              for (int a = 0; a < NA; ++a) acc[a] += pg[a];
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        if (++visits == kFoldLeaves) {
          visits = 0;
          fold<NA, KAHAN>(sum, cmp, acc);
#pragma unroll
          for (int a = 0; a < NA; ++a) acc[a] = 0.0f;
        }
      }
      next = nskip > i ? nskip : i + 1;  // pre-order: skip > i always; guards the loop regardless
    }
    if (next == i + 1) {
      nd = nd1;
      g = g1;
      mm = mm1;
    } else if (next < nn) {
      nd = node[next];
      g = geo[next];
      mm = mom[next];
    }
    i = __builtin_amdgcn_readfirstlane(next);
  }
  fold<NA, KAHAN>(sum, cmp, acc);
#pragma unroll
  for (int a = 0; a < NA; ++a)
    part[((int64_t)segment * NA + a) * mpad + qi] = KAHAN ? sum[a] - cmp[a] : sum[a];
}

// Work of the traversal (the counts of dwg_octree_work). The decisions are those of
// k_tree_eval (the same FP64 opening test, the same wave-wide walk over the same wavefronts of
// 64 sorted queries), without its arithmetic. Per-query counts leave out lanes past m (they
// repeat query m - 1, which sits in the same wavefront, so they change no wave-wide step);
// wavefront counts come from lane 0 of each wavefront with a query below m. Integer atomics
// make the totals independent of the order of the blocks.
__global__ __launch_bounds__(256) void k_tree_work(const float* __restrict__ Q, int64_t m,
                                                   const int32_t* __restrict__ qperm, const int4* __restrict__ node,
                                                   const double4* __restrict__ geo,
                                                   const int32_t* __restrict__ total_p, int64_t cap, int64_t n_src,
                                                   unsigned long long* __restrict__ out) {
  __shared__ unsigned long long red[kTreeWorkCounts][4];
  const int64_t qi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = qi < m;
  const int64_t o = qperm[live ? qi : m - 1];
  const double dqx = Q[o], dqy = Q[m + o], dqz = Q[2 * m + o];
  int nn = __builtin_amdgcn_readfirstlane(*total_p);
  if (nn > cap) nn = (int)cap;
  unsigned long long nfar = 0, npair = 0, wfar = 0, wleaf = 0;
  int skip_to = 0;
  int i = 0;
  while (i < nn) {
    const int4 nd = node[i];
    const double4 g = geo[i];
    const int nskip = __builtin_amdgcn_readfirstlane(nd.z);
    bool far = false, open = false, direct = false;
    if (i >= skip_to) {
      const double dx = g.x - dqx, dy = g.y - dqy, dz = g.z - dqz;
      const double d2 = dx * dx + dy * dy + dz * dz;
      if (d2 > g.w) {
        far = true;
        ++nfar;
        skip_to = nskip;
      } else if (nd.w >> 8) {
        direct = true;
      } else {
        open = true;
      }
    }
    if (__any(far)) ++wfar;
    int next;
    if (__any(open)) {
      next = i + 1;
    } else {
      const int s1 = nd.y < n_src ? nd.y : (int)n_src;
      if (direct) npair += (unsigned long long)(s1 - nd.x);
      const uint64_t dmask = __ballot(direct);
      if (dmask) {
        const int ns = s1 - __builtin_amdgcn_readfirstlane(nd.x);
        const int lk = leaf_split_log2(__popcll(dmask), ns);
        wleaf += (unsigned long long)((ns + (1 << lk) - 1) >> lk);
      }
      next = nskip > i ? nskip : i + 1;
    }
    i = __builtin_amdgcn_readfirstlane(next);
  }
  if (!live) nfar = npair = 0;
  for (int off = 32; off > 0; off >>= 1) {
    nfar += __shfl_xor(nfar, off, 64);
    npair += __shfl_xor(npair, off, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) {
    // lane 0 is live whenever any lane of its wavefront is
    red[0][wv] = nfar;
    red[1][wv] = npair;
    red[2][wv] = live ? wfar : 0;
    red[3][wv] = live ? wleaf : 0;
  }
  __syncthreads();
  if (threadIdx.x < kTreeWorkCounts)
    atomicAdd(&out[threadIdx.x], red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3]);
}

__global__ void k_zero_u64(unsigned long long* __restrict__ a, int k) {
  if ((int)threadIdx.x < k) a[threadIdx.x] = 0ull;
}

__global__ void k_copy_i32(const int32_t* __restrict__ a, int64_t n, int32_t* __restrict__ b) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

// (start, end, level, skip) per node for dwg_octree.
__global__ void k_tree_export(const int4* __restrict__ node, const int32_t* __restrict__ total_p, int64_t cap,
                              int32_t* __restrict__ out) {
  const int64_t total = node_count(total_p, cap);
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int4 nd = node[k];
    out[4 * k + 0] = nd.x;
    out[4 * k + 1] = nd.y;
    out[4 * k + 2] = nd.w & 255;
    out[4 * k + 3] = nd.z;
  }
}

template <int BLOCK, bool GRAD, bool SCREENED, bool KAHAN>
void launch_eval_b(const float* Q, int64_t m, const int32_t* qperm, const GwnWork& w, const TreeWork& t,
                   float kappa, hipStream_t st) {
  hipLaunchKernelGGL((k_tree_eval<BLOCK, GRAD, SCREENED, KAHAN>), dim3(tree_grid(w.mpad / BLOCK, w.split)), dim3(BLOCK),
                     0, st, Q, m, qperm, t.node, t.geo, t.mom, t.off + t.n, t.cap, w.src, t.n, kScaledScr, kappa,
                     w.part, w.mpad, (unsigned)w.split, w.stop);
}

template <bool GRAD, bool SCREENED, bool KAHAN>
void launch_eval_t(const float* Q, int64_t m, const int32_t* qperm, const GwnWork& w, const TreeWork& t,
                   float kappa, hipStream_t st) {
  if (m >= kLoneQueries)
    launch_eval_b<64, GRAD, SCREENED, KAHAN>(Q, m, qperm, w, t, kappa, st);
  else
    launch_eval_b<kTreeBlock, GRAD, SCREENED, KAHAN>(Q, m, qperm, w, t, kappa, st);
}

}  // namespace

int64_t tree_cap(int64_t n) { return 2 * n + 1; }

int tree_segments(int64_t n_src, int64_t n_qry) {
  const int64_t waves = cdiv(n_qry, 64);
  const int64_t s = std::min<int64_t>(cdiv(kSegmentWaves, waves), cdiv(n_src, kSegmentSources));
  return (int)std::max<int64_t>(1, std::min<int64_t>(s, kMaxSegments));
}

// cdiv(B, x) x <= B - 1 + x for the wavefronts; the columns are padded to eight of them.
int64_t segment_columns(int64_t n_src, int64_t n_qry) {
  const int64_t waves = padded_queries(n_qry) / 64, most = std::min<int64_t>(cdiv(n_src, kSegmentSources), kMaxSegments);
  return 64 * std::min<int64_t>(most * waves, kSegmentWaves + waves + (kQBlock / 64) * kMaxSegments);
}

dwg_status morton_frame(const float* P, int64_t n, float* bpart, float* box, double* frame, hipStream_t st) {
  dwg_status s = launch_bbox(P, n, bpart, box, st);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_tree_frame, dim3(1), dim3(64), 0, st, box, frame);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

size_t carve_tree(Carver& c, int64_t n, int leaf, double beta, TreeWork* out) {
  const size_t s0 = c.used;
  TreeWork t{};
  t.n = n;
  t.cap = tree_cap(n);
  t.leaf = leaf;
  t.beta = beta;
  t.bpart = c.take<float>(kBboxParts);
  t.box = c.take<float>(8);
  t.frame = c.take<double>(4);
  t.key[0] = c.take<uint64_t>((size_t)n);
  t.key[1] = c.take<uint64_t>((size_t)n);
  t.val[0] = c.take<int32_t>((size_t)n);
  t.val[1] = c.take<int32_t>((size_t)n);
  t.work = c.take<int32_t>(radix_work_len(n));
  t.lev = c.take<int32_t>((size_t)n);
  t.off = c.take<int32_t>((size_t)n + 1);
  t.osums = c.take<int32_t>(scan_sums_len(n));
  t.node = c.take<int4>((size_t)t.cap);
  t.geo = c.take<double4>((size_t)t.cap);
  t.mom = c.take<float4>((size_t)t.cap);
  t.rbits = c.take<unsigned long long>((size_t)t.cap);
  t.dbits = c.take<uint32_t>((size_t)t.cap);
  t.pos = c.take<float4>((size_t)n);
  t.rad = c.take<float>((size_t)n);
  t.tile = c.take<double>((size_t)(4 * cdiv(n, kSumTile)));
  if (out) *out = t;
  return c.used - s0;
}

dwg_status tree_build(const float* P, const float* area, const float* delta, int64_t n, float eps,
                      const TreeWork& t, int32_t* perm, hipStream_t st) {
  dwg_status s = morton_frame(P, n, t.bpart, t.box, t.frame, st);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_tree_keys, dim3(grid_cap(n)), dim3(256), 0, st, P, n, t.frame, t.key[0]);
  DWG_TRY_LAUNCH();
  int res = 0;
  s = radix_sort_pairs(t.key, t.val, true, n, 64, t.work, &res, st);
  if (s != DWG_OK) return s;
  // eight passes: the sorted codes and indices are back in buffer 0
  hipLaunchKernelGGL(k_tree_mark, dim3(grid_cap(n)), dim3(256), 0, st, t.key[0], n, t.leaf, t.lev, t.off);
  DWG_TRY_LAUNCH();
  s = exclusive_scan(t.off, n, t.osums, st);
  if (s != DWG_OK) return s;
  hipLaunchKernelGGL(k_tree_emit, dim3(grid_cap(n)), dim3(256), 0, st, t.key[0], n, t.leaf, t.lev, t.off, t.cap,
                     t.node);
  DWG_TRY_LAUNCH();
  if (!area) {  // topology only (dwg_octree)
    hipLaunchKernelGGL(k_copy_i32, dim3(grid_cap(n)), dim3(256), 0, st, t.val[0], n, perm);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  const int32_t* total = t.off + n;
  const int64_t tiles = cdiv(n, kSumTile);
  hipLaunchKernelGGL(k_tree_sorted, dim3((unsigned)cdiv(tiles, 4)), dim3(256), 0, st, P, area, delta, eps, t.val[0],
                     n, tiles, perm, t.pos, t.rad, t.tile);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_tree_geo, dim3(node_grid(n)), dim3(256), 0, st, t.node, total, t.cap, AreaSum{t.pos}, t.rad,
                     t.tile, t.beta, t.geo, t.rbits, t.dbits);
  DWG_TRY_LAUNCH();
  if (n <= kSumTile) return DWG_OK;
  hipLaunchKernelGGL(k_tree_far, dim3((unsigned)cdiv(n, kFarTile)), dim3(64), 0, st, t.node, total, t.cap, t.pos,
                     t.rad, n, t.geo, t.rbits, t.dbits);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_tree_crit, dim3(grid_cap(t.cap)), dim3(256), 0, st, t.node, total, t.cap, t.beta, t.rbits,
                     t.dbits, t.geo);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status tree_stage_leaves(const GwnWork& w, const TreeWork& t, float kappa, hipStream_t st) {
  hipLaunchKernelGGL(k_tree_leafpos, dim3(grid_cap(t.cap)), dim3(256), 0, st, t.node, t.off + t.n, t.cap, t.geo, w.src,
                     t.n, kappa);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status tree_moments(const GwnWork& w, const TreeWork& t, hipStream_t st) {
  const MomentSum f{w.src};
  const int64_t tiles = cdiv(t.n, kSumTile);
  hipLaunchKernelGGL(k_tile_sums<MomentSum>, dim3((unsigned)cdiv(tiles, 4)), dim3(256), 0, st, f, t.n, tiles, t.tile,
                     w.stop, w.clock());
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_tree_mom, dim3(node_grid(t.n)), dim3(256), 0, st, t.node, t.off + t.n, t.cap, f, t.tile,
                     w.stop, t.mom);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status tree_eval(const float* Q, int64_t m, const dwg_kernel_params& kp, bool grad, const GwnWork& w,
                     const TreeWork& t, hipStream_t st) {
  const bool scr = kp.lambda > 0.0f;
  const bool kah = kp.compensated != 0;
  const float kappa = position_scale(kp);
#define DWG_TREE_CASE(G, S, K) \
  if (grad == G && scr == S && kah == K) launch_eval_t<G, S, K>(Q, m, w.perm_q, w, t, kappa, st);
  DWG_TREE_CASE(true, false, true)
  DWG_TREE_CASE(true, false, false)
  DWG_TREE_CASE(true, true, true)
  DWG_TREE_CASE(true, true, false)
  DWG_TREE_CASE(false, false, true)
  DWG_TREE_CASE(false, false, false)
  DWG_TREE_CASE(false, true, true)
  DWG_TREE_CASE(false, true, false)
#undef DWG_TREE_CASE
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status tree_work(const float* Q, int64_t m, const int32_t* qperm, const TreeWork& t, unsigned long long* out,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, out, kTreeWorkCounts);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_tree_work, dim3((unsigned)cdiv(m, 256)), dim3(256), 0, st, Q, m, qperm, t.node, t.geo,
                     t.off + t.n, t.cap, t.n, out);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status tree_export(const TreeWork& t, int32_t* nodes_out, int64_t cap_out, int64_t* count_host,
                       hipStream_t st) {
  int32_t total = 0;
  DWG_TRY_HIP(hipMemcpyAsync(&total, t.off + t.n, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  DWG_TRY_HIP(hipStreamSynchronize(st));
  *count_host = total;
  if (total > cap_out) {
    set_error("octree has %d nodes, output holds %lld", total, (long long)cap_out);
    return DWG_E_INVALID;
  }
  hipLaunchKernelGGL(k_tree_export, dim3(grid_cap(total)), dim3(256), 0, st, t.node, t.off + t.n, cap_out, nodes_out);
  DWG_TRY_LAUNCH();
  DWG_TRY_HIP(hipStreamSynchronize(st));
  return DWG_OK;
}

}  // namespace dwg
