// All-pairs GWN / gradient kernels, the normal-update epilogue and the FP64 statistics of
// one DWG iteration (Sec. 3 Eq. 2-3, Sec. 4.2 Eq. 5, Sec. 4.3 Eq. 6-7, Sec. 5.1-5.2).
//
// Data layout in HBM (all carved from the caller's workspace; "sorted" = the spatial order
// of dwg_sort.hip, perm[i] = original index of sorted position i):
//   src   [2*npad] float4  sorted sources: (p_j, 1/(kappa max(delta_j, eps))), (m_j, 0) with
//                          m_j = a_j n_j / (4 pi); padding sources are all zero, which makes
//                          their contribution exactly zero in the general path.
//   kk    [npad]           a_j / (4 pi) per sorted source (restaging after the update)
//   tbox  [2*ntiles]       per source tile: (min xyz, max radius), (max xyz, 0)
//   part  [split][7][mpad] per-split partial sums of w, A, B per sorted query
//   theta [m] double       angle between consecutive normals (degrees), sorted order
// Positions and boxes are in the caller's units; kappa = s log2(e) for the screened kernel
// (1 for the plain one) is applied to pair differences inside the kernels.
// Queries are gathered from the caller's planar [3][m] array through the query permutation.
#include <cmath>

#include "dwg_internal.h"
#include "dwg_pair.h"

namespace dwg {
namespace {

using namespace pairk;

constexpr double kRadToDeg = 57.295779513082320876798;

// Tile classes of the all-pairs kernel: general (clamp and coincidence handled), far (no pair
// clamped or coincident) and separated (far, and every pair at least as long as the largest
// distance of a query from the block's centre), each with its own pair loop.
enum TileKind { kGeneral = 0, kFar = 1, kSeparated = 2 };

// One LDS tile of sources against the thread's QPT queries. The tile holds the separated
// form (a = (-2 p, |p|^2), b = (m, m . p), iw apart); the general and far loops recover the
// difference p - q exactly as fma(-2 p, -1/2, -q).
template <int QPT, int NS, int TS, bool GRAD, bool SCREENED, int KIND>
__device__ __forceinline__ void tile_loop(const float4* sa, const float4* sb, const float* sw, const float* qx,
                                          const float* qy, const float* qz, const float* qq, const Scr k,
                                          float (*acc)[NS]) {
#pragma unroll (GRAD ? 2 : 4)
  for (int j = 0; j < TS; ++j) {
    const float4 a = sa[j];
    const float4 b = sb[j];
    const float iw = KIND == kGeneral ? sw[j] : 0.0f;
    if (KIND == kSeparated) {
      // Every query's r^2 and rsq first, then the rest: the rsq latency is then covered by
      // the work that does not depend on it (m . q). Left to itself the compiler interleaves
      // the queries' chains and issues each rsq right before its first use (measured 568 ms
      // per 1M x 1M screened launch against 524 ms in this order).
      float r2[QPT], ir[QPT];
#pragma unroll
      for (int q = 0; q < QPT; ++q) r2[q] = sep_r2(a, qx[q], qy[q], qz[q], qq[q]);
#pragma unroll
      for (int q = 0; q < QPT; ++q) ir[q] = rsq(r2[q]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < QPT; ++q) {
        if (SCREENED)
          pair_screened_sep<GRAD>(a, b, qx[q], qy[q], qz[q], r2[q], ir[q], k, acc[q]);
        else
          pair_plain_sep<GRAD>(a, b, qx[q], qy[q], qz[q], ir[q], acc[q]);
      }
    } else {
#pragma unroll
      for (int q = 0; q < QPT; ++q) {
        const float dx = fmaf(a.x, -0.5f, -qx[q]), dy = fmaf(a.y, -0.5f, -qy[q]), dz = fmaf(a.z, -0.5f, -qz[q]);
        if (SCREENED)
          pair_screened_d<GRAD, KIND == kFar>(dx, dy, dz, iw, b, k, acc[q]);
        else
          pair_plain_d<GRAD, KIND == kFar>(dx, dy, dz, iw, b, acc[q]);
      }
      if (KIND == kFar && SCREENED && GRAD) {
        // Instruction order of one source against the QPT = 2 queries (scheduling only): the
        // two LDS reads, the 12 VALU of both differences and r^2, both rsq, 8 VALU, both exp,
        // then the rest. Left to itself the compiler issues the four rsq (and four exp) of the
        // unrolled pair of sources back to back; this order measured 528-531 ms against
        // 546-551 ms per 1M x 1M launch when every far tile took this loop.
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // DS read
        __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);  // VALU
        __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);   // transcendental
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 34, 0);
      }
    }
  }
}

// All-pairs kernel. Block = NT threads holding QPT queries each, NT x QPT = 512 (sorted query
// q0 + k*NT + tid); grid.y = source split. Sources are staged in LDS TS at a time and read
// back as broadcasts; TS divides the 256 sources of a tile. Per tile, each wavefront decides whether the tile is far
// from all of its queries -- box distance above the tile's largest radius, so no pair can be
// clamped, coincident or too short for 1/r^3 -- and then runs the shorter far-pair loop; a far tile whose box
// distance is also at least the largest distance of one of its queries from the block's centre
// takes the separated far loop (r^2 and m . (p - q) from per-source |p|^2 and m . p). (Deciding
// by the block's box puts fewer tiles in the short loops: values at 131K queries off the surface of 50K
// points 1.99 -> 1.85 ms; 1M x 1M equal.)
// Each tile's contributions go to FP32 partials, folded into running sums
// (Kahan-compensated when KAHAN). The compensation terms live in LDS, one column per
// thread: they are touched once per tile, and the 14 registers they would take hold the
// screened kernel at 4 waves per SIMD instead of 5 (the kernel asks for 5, which it fits
// without spills).
// Positions enter the pair arithmetic relative to a point c of the block and scaled by kappa:
// kappa (x - c), formed when the tile is filled (with |p|^2 and m . p in the fourth
// components). The rounding of a near pair's difference is then relative to the pair's
// distance from c, not to |x| (kappa x rounded in FP32 would move r by up to |x| 2^-24,
// enough to flip the clamp branch of pairs within ~1e-5 of r = delta in a scene of size 2).
// c is the block's middle query (sorted position q0 + 256), not the centre of its box:
// where the spatial order jumps inside a block (a lone point far from the rest of its
// block), the box centre lies far from every query and all of the block's near pairs lose
// precision; the middle query keeps the block's bulk exact relative to itself, and the far
// query's pairs are long.
__device__ __forceinline__ float first_lane(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

template <int NT, int QPT, int TS, bool GRAD, bool SCREENED, bool KAHAN>
__device__ __forceinline__ void gwn_block(const float* __restrict__ Q, int64_t m, const int32_t* __restrict__ qperm,
                                          const float4* __restrict__ src, int64_t nsteps, int64_t nfull,
                                          int64_t steps_per_split, const float4* __restrict__ tbox, Scr sk, float kappa,
                                          float* __restrict__ part, int64_t mpad) {
  static_assert(NT * QPT == kQBlock && kTile % TS == 0 && TS <= kTile, "block shape");
  constexpr int NA = GRAD ? kNAcc : 1;
  constexpr int NS = GRAD ? kNAcc + 1 : 1;  // + sum of t in the separated loop
  __shared__ float4 sa[TS];
  __shared__ float4 sb[TS];
  __shared__ float sw[TS];
  const int tid = threadIdx.x;
  const int64_t q0 = (int64_t)blockIdx.x * kQBlock;
  const int64_t oc = qperm[min(q0 + kQBlock / 2, m - 1)];
  const float cx = Q[oc], cy = Q[m + oc], cz = Q[2 * m + oc];
  float qx[QPT], qy[QPT], qz[QPT], qq[QPT];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    int64_t qi = q0 + k * NT + tid;
    if (qi >= m) qi = m - 1;
    const int64_t o = qperm[qi];
    const float x = Q[o], y = Q[m + o], z = Q[2 * m + o];
    lo[0] = fminf(lo[0], x), hi[0] = fmaxf(hi[0], x);
    lo[1] = fminf(lo[1], y), hi[1] = fmaxf(hi[1], y);
    lo[2] = fminf(lo[2], z), hi[2] = fmaxf(hi[2], z);
    qx[k] = kappa * (x - cx);
    qy[k] = kappa * (y - cy);
    qz[k] = kappa * (z - cz);
    qq[k] = fmaf(qz[k], qz[k], fmaf(qy[k], qy[k], qx[k] * qx[k]));
  }
  // box of the wavefront's queries, and the largest distance of one from c (its farthest corner)
  float rq2 = 0.0f;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    for (int o = 32; o > 0; o >>= 1) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o, 64));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o, 64));
    }
    lo[d] = first_lane(lo[d]);
    hi[d] = first_lane(hi[d]);
    const float c = d == 0 ? cx : (d == 1 ? cy : cz), r = fmaxf(hi[d] - c, c - lo[d]);
    rq2 += r * r;
  }
  __shared__ float cmp[KAHAN ? QPT * NA : 1][NT];  // thread-private columns
  float sum[QPT][NA];
#pragma unroll
  for (int k = 0; k < QPT; ++k)
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      sum[k][a] = 0.0f;
      if (KAHAN) cmp[k * NA + a][tid] = 0.0f;
    }

  const int64_t u0 = (int64_t)blockIdx.y * steps_per_split;
  const int64_t u1 = min(u0 + steps_per_split, nsteps);
  for (int64_t u = u0; u < u1; ++u) {
    const int64_t t = TS == kTile ? u : u / (kTile / TS);
    __syncthreads();
#pragma unroll
    for (int i = tid; i < TS; i += NT) {
      const float4 a = src[2 * (u * TS + i)];
      const float4 b = src[2 * (u * TS + i) + 1];
      const float px = kappa * (a.x - cx), py = kappa * (a.y - cy), pz = kappa * (a.z - cz);
      sa[i] = make_float4(-2.0f * px, -2.0f * py, -2.0f * pz, fmaf(pz, pz, fmaf(py, py, px * px)));
      sb[i] = make_float4(b.x, b.y, b.z, fmaf(b.z, pz, fmaf(b.y, py, b.x * px)));
      sw[i] = a.w;
    }
    const float4 tlo = tbox[2 * t], thi = tbox[2 * t + 1];
    const float gx = fmaxf(0.0f, fmaxf(lo[0] - thi.x, tlo.x - hi[0]));
    const float gy = fmaxf(0.0f, fmaxf(lo[1] - thi.y, tlo.y - hi[1]));
    const float gz = fmaxf(0.0f, fmaxf(lo[2] - thi.z, tlo.z - hi[2]));
    const float gap2 = gx * gx + gy * gy + gz * gz;
    // tiles with padding (t >= nfull) always take the general path
    const bool far = __builtin_amdgcn_readfirstlane(t < nfull && gap2 > 0.0f && gap2 > 1.0001f * tlo.w * tlo.w);
    const bool sep = __builtin_amdgcn_readfirstlane(far && gap2 >= rq2);
    __syncthreads();
    float acc[QPT][NS];
#pragma unroll
    for (int k = 0; k < QPT; ++k)
#pragma unroll
      for (int a = 0; a < NS; ++a) acc[k][a] = 0.0f;
    if (sep) {
      tile_loop<QPT, NS, TS, GRAD, SCREENED, kSeparated>(sa, sb, sw, qx, qy, qz, qq, sk, acc);
      if (GRAD) {
#pragma unroll
        for (int k = 0; k < QPT; ++k) {  // A = -sum(t P) / 2 - q sum(t)
          acc[k][1] = fmaf(-0.5f, acc[k][1], -qx[k] * acc[k][NS - 1]);
          acc[k][2] = fmaf(-0.5f, acc[k][2], -qy[k] * acc[k][NS - 1]);
          acc[k][3] = fmaf(-0.5f, acc[k][3], -qz[k] * acc[k][NS - 1]);
        }
      }
    } else if (far) {
      tile_loop<QPT, NS, TS, GRAD, SCREENED, kFar>(sa, sb, sw, qx, qy, qz, qq, sk, acc);
    } else {
      tile_loop<QPT, NS, TS, GRAD, SCREENED, kGeneral>(sa, sb, sw, qx, qy, qz, qq, sk, acc);
    }
#pragma unroll
    for (int k = 0; k < QPT; ++k)
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        if (KAHAN) {
          const float y = acc[k][a] - cmp[k * NA + a][tid];
          const float tt = sum[k][a] + y;
          cmp[k * NA + a][tid] = (tt - sum[k][a]) - y;
          sum[k][a] = tt;
        } else {
          sum[k][a] += acc[k][a];
        }
      }
  }
  float* out = part + (int64_t)blockIdx.y * NA * mpad;
#pragma unroll
  for (int k = 0; k < QPT; ++k) {
    const int64_t qi = q0 + k * NT + tid;  // < mpad by construction of mpad
#pragma unroll
    for (int a = 0; a < NA; ++a) out[a * mpad + qi] = KAHAN ? sum[k][a] - cmp[k * NA + a][tid] : sum[k][a];
  }
}

// With the gradient: two queries per thread. 105 VGPRs would fit 4 waves per SIMD; asked for 5, the
// kernel does without spills.
template <bool SCREENED, bool KAHAN>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_gwn(
    const float* __restrict__ Q, int64_t m, const int32_t* __restrict__ qperm, const float4* __restrict__ src,
    int64_t nsteps, int64_t nfull, int64_t steps_per_split, const float4* __restrict__ tbox, Scr sk, float kappa,
    float* __restrict__ part, int64_t mpad, const int32_t* __restrict__ stop, uint64_t* __restrict__ begin) {
  if (*stop) return;
  if ((blockIdx.x | blockIdx.y | threadIdx.x) == 0) *begin = wall_clock64();
  gwn_block<kBlock, kQpt, kTile, true, SCREENED, KAHAN>(Q, m, qperm, src, nsteps, nfull, steps_per_split, tbox, sk,
                                                        kappa, part, mpad);
}

// Values only.
template <bool SCREENED, bool KAHAN>
__global__ __launch_bounds__(kBlock) void k_gwn_w(
    const float* __restrict__ Q, int64_t m, const int32_t* __restrict__ qperm, const float4* __restrict__ src,
    int64_t nsteps, int64_t nfull, int64_t steps_per_split, const float4* __restrict__ tbox, Scr sk, float kappa,
    float* __restrict__ part, int64_t mpad, const int32_t* __restrict__ stop, uint64_t* __restrict__ begin) {
  if (*stop) return;
  if ((blockIdx.x | blockIdx.y | threadIdx.x) == 0) *begin = wall_clock64();
  gwn_block<kBlock, kQpt, kTile, false, SCREENED, KAHAN>(Q, m, qperm, src, nsteps, nfull, steps_per_split, tbox, sk,
                                                       kappa, part, mpad);
}

// Small launches: one query per thread and steps of kSmallStep sources, so that a few blocks of
// queries still fill the chip (see small_launch).
constexpr int kSmallStep = 32;
template <bool GRAD, bool SCREENED, bool KAHAN>
__global__ __launch_bounds__(kQBlock) void k_gwn_small(
    const float* __restrict__ Q, int64_t m, const int32_t* __restrict__ qperm, const float4* __restrict__ src,
    int64_t nsteps, int64_t nfull, int64_t steps_per_split, const float4* __restrict__ tbox, Scr sk, float kappa,
    float* __restrict__ part, int64_t mpad, const int32_t* __restrict__ stop, uint64_t* __restrict__ begin) {
  if (*stop) return;
  if ((blockIdx.x | blockIdx.y | threadIdx.x) == 0) *begin = wall_clock64();
  gwn_block<kQBlock, 1, kSmallStep, GRAD, SCREENED, KAHAN>(Q, m, qperm, src, nsteps, nfull, steps_per_split, tbox, sk, kappa,
                                                           part, mpad);
}

// Stage the sources in spatial order: (p, 1/(kappa max(delta,eps))) and m = a n / (4 pi)
// (kappa = the position scale of the kernel, 1 when plain; positions stay unscaled, the
// evaluation kernels scale differences).
// A NaN delta poisons the source's m so that the result is NaN as in the definition. Clears the
// stop flag of an iteration. With tbox (the all-pairs kernels'), a block is a source tile and writes its
// box (real sources only) and largest radius max(delta, eps), in the unscaled units of the
// positions (the staged 1/radius carries kappa), or kLeastFar where that is more: no tile is far from a query
// of which a pair is so short that 1/r^3 overflows. (As one more term of the test in the kernel: 1M x 1M 510 -> 529 ms.)
constexpr float kLeastFar = 0x1p-42f;  // scaled length below which the general loop's guard, r^2 2^126 for 1/r, is at work

__global__ __launch_bounds__(kTile) void k_stage(const float* __restrict__ P, const float* __restrict__ N,
                        const float* __restrict__ A, const float* __restrict__ D, int64_t n,
                        float eps, float kappa, const int32_t* __restrict__ perm,
                        float4* __restrict__ src, float* __restrict__ kk, int32_t* __restrict__ stop,
                        float4* __restrict__ tbox) {
  const int64_t j = (int64_t)blockIdx.x * kTile + threadIdx.x;  // < npad
  if (j == 0) *stop = 0;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = make_float4(0.f, 0.f, 0.f, 0.f);
  float k = 0.0f;
  if (j < n) {
    const int64_t o = perm[j];
    const float d = D ? D[o] : 0.0f;
    const float fl = kappa * (d > eps ? d : eps);
    const float id = fl > 0.0f ? 1.0f / fl : INFINITY;
    k = A[o] * kInv4Pi;
    if (d != d) k = NAN;
    a = make_float4(P[o], P[n + o], P[2 * n + o], id);
    b = make_float4(k * N[o], k * N[n + o], k * N[2 * n + o], 0.0f);
  }
  src[2 * j] = a;
  src[2 * j + 1] = b;
  kk[j] = k;
  if (!tbox) return;
  __shared__ float lds[7][kTile / 64];
  float v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0f};
  if (j < n) {
    v[0] = v[3] = a.x;
    v[1] = v[4] = a.y;
    v[2] = v[5] = a.z;
    v[6] = 1.0f / (kappa * a.w);  // radius (0 when 1/radius is +inf)
    if (!(v[6] == v[6])) v[6] = INFINITY;
  }
#pragma unroll
  for (int d = 0; d < 7; ++d) {
    for (int o = 32; o > 0; o >>= 1) {
      const float x = __shfl_xor(v[d], o, 64);
      v[d] = d < 3 ? fminf(v[d], x) : fmaxf(v[d], x);
    }
    if ((threadIdx.x & 63) == 0) lds[d][threadIdx.x >> 6] = v[d];
  }
  __syncthreads();
  if (threadIdx.x > 0) return;
#pragma unroll
  for (int d = 0; d < 7; ++d)
    for (int w = 0; w < kTile / 64; ++w) v[d] = d < 3 ? fminf(v[d], lds[d][w]) : fmaxf(v[d], lds[d][w]);
  tbox[2 * blockIdx.x] = make_float4(v[0], v[1], v[2], fmaxf(v[6], kLeastFar / kappa));
  tbox[2 * blockIdx.x + 1] = make_float4(v[3], v[4], v[5], 0.0f);
}


// Sum of `split` partials of accumulator `a` for sorted query i, in split order, eight loads in
// flight at a time; whole batches without a check of each (the update of 2,000 points 11.2 -> 9.3 us,
// of 20,011 13.1 -> 11.0, the epilogue of 100K queries 28.6 -> 24.8; batches of 16 no faster, at 1M
// points slower). The sum is compensated, also where the partials are not: finer splits and segments then
// cost no precision. A Kahan step (Kahan 1965) loses the low bits of the running sum where the partial is the larger of
// the two, which is the rule in an octree walk (one segment holds the near field): TWO takes the exact error
// of every addition instead (Knuth's two-sum), for two additions more. Error of octree gradients against 64 bits, over
// 1,500 to 100,000 points, in units of one walk without segments: 1.02 with Kahan steps from 20,000 points on, 1.00
// with exact ones (four iterations 0.77 to 0.93); without compensation 1.1 to 1.4, now 0.9 to 0.96. All-pairs,
// not compensated, 16,000 to 50,000 points, in units of the coarser splits: 1.06 to 1.11, now 0.89 to 0.96.
template <bool TWO>
__device__ __forceinline__ float combine(const float* part, int split, int64_t mpad, int na, int a, int64_t i) {
  const float* p = part + (int64_t)a * mpad + i;
  const int64_t step = (int64_t)na * mpad;
  float s = 0.0f, c = 0.0f;
  auto add = [&](float x) {
    if (TWO) {
      const float t = s + x, b = t - s;
      c -= (s - (t - b)) + (x - b);
      s = t;
    } else {
      const float y = x - c;
      const float t = s + y;
      c = (t - s) - y;
      s = t;
    }
  };
  constexpr int kBatch = 8;
  int p0 = 0;
  for (; p0 + kBatch <= split; p0 += kBatch) {
    float x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) x[u] = p[(p0 + u) * step];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) add(x[u]);
  }
  if (p0 < split) {
    float x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) x[u] = p[(p0 + u < split ? p0 + u : split - 1) * step];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (p0 + u >= split) break;
      add(x[u]);
    }
  }
  return TWO && !(c == c) ? s : s - c;  // an infinite partial has no error to take
}

// The epilogue kernels take QB queries per block: its kEpiBlock threads first sum the splits of
// every (accumulator, query) pair, a wavefront per accumulator, then QB of them finish a query
// each. One thread per query summing its 7 x split partials in turn took 97 us for 100K queries
// and 48 splits (1.4 TB/s).
constexpr int kEpiBlock = 64 * kNAcc;
constexpr int kEpiWaves = kNAcc;
constexpr int64_t kEpiSmall = 32768;  // queries up to which QB = 64: at 256 a few blocks would do it all

template <int QB, bool TWO>
__device__ __forceinline__ void combine_block(const float* part, int split, int64_t mpad, int na, int64_t q0,
                                              float (*acc)[QB]) {
  for (int i = threadIdx.x; i < na * QB; i += kEpiBlock)
    acc[i / QB][i % QB] = combine<TWO>(part, split, mpad, na, i / QB, q0 + i % QB);
  __syncthreads();
}

// Block-wide FP64 sum (deterministic: fixed shuffle tree, then fixed LDS order).
__device__ double block_sum(double v, double* lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += lds[k];
  return r;  // valid on thread 0
}

// Output scaling of the accumulators: w = ws w', grad = as A - bs B'.
struct Scale {
  float ws, as, bs;
};
Scale scale_of(const dwg_kernel_params& kp) {
  if (!(kp.lambda > 0.0f)) return Scale{1.0f, 3.0f, 1.0f};
  // screened sums in scaled coordinates: w' carries 1/kappa^2, A and B' carry 1/kappa^3
  const double k = position_scale(kp);
  return Scale{(float)(k * k / 3.0), (float)(k * k * k), (float)(k * k * k / 3.0)};
}

// Evaluation epilogue: combine splits; write w and grad at the query's original index;
// FP64 block partial of w.
template <int QB, bool TWO>
__global__ __launch_bounds__(kEpiBlock) void k_combine(const float* __restrict__ part, int split,
                                                       int64_t mpad, int64_t m, bool grad, Scale sc,
                                                       const int32_t* __restrict__ qperm,
                                                       float* __restrict__ wout,
                                                       float* __restrict__ gout,
                                                       double* __restrict__ blk) {
  __shared__ float acc[kNAcc][QB];
  __shared__ double lds[kEpiWaves];
  const int64_t q0 = (int64_t)blockIdx.x * QB;  // mpad is a multiple of QB
  combine_block<QB, TWO>(part, split, mpad, grad ? kNAcc : 1, q0, acc);
  const int t = threadIdx.x;
  const int64_t i = q0 + t;
  double wv = 0.0;
  if (t < QB && i < m) {
    const int64_t o = qperm[i];
    const float w = sc.ws * acc[0][t];
    if (grad)
      for (int d = 0; d < 3; ++d) gout[d * m + o] = fmaf(sc.as, acc[1 + d][t], -sc.bs * acc[4 + d][t]);
    if (wout) wout[o] = w;
    wv = (double)w;
  }
  const double bs = block_sum(wv, lds);
  if (threadIdx.x == 0) blk[blockIdx.x] = bs;
}

// Iteration epilogue (Eq. 7): n_new = -grad/|grad| (kept when |grad| is 0 or not finite),
// written in place at the point's original index; restage m for the next iteration;
// theta_i (degrees, FP64); FP64 block partials of w and of the chord |n_new - n_old|. Clears the
// histograms of the selection that follows. After the iteration has stopped, nothing changes.
template <int QB, bool TWO>
__global__ __launch_bounds__(kEpiBlock) void k_update(const float* __restrict__ part, int split,
                                                      int64_t mpad, int64_t n, Scale sc,
                                                      const int32_t* __restrict__ perm,
                                                      const float* __restrict__ kk,
                                                      float* __restrict__ N,
                                                      float4* __restrict__ src,
                                                      double* __restrict__ theta,
                                                      double* __restrict__ blk, int nblk,
                                                      uint32_t* __restrict__ hist,
                                                      const int32_t* __restrict__ stop, uint64_t* __restrict__ end) {
  __shared__ float acc[kNAcc][QB];
  __shared__ double lds[kEpiWaves];
  const int64_t q0 = (int64_t)blockIdx.x * QB;
  if (*stop) return;
  clear_hist(hist, n);
  if ((blockIdx.x | threadIdx.x) == 0) *end = wall_clock64();
  combine_block<QB, TWO>(part, split, mpad, kNAcc, q0, acc);
  const int t = threadIdx.x;
  const int64_t i = q0 + t;
  double wv = 0.0, cv = 0.0;
  if (t < QB && i < n) {
    const float w = sc.ws * acc[0][t];
    float g[3];
    for (int d = 0; d < 3; ++d) g[d] = fmaf(sc.as, acc[1 + d][t], -sc.bs * acc[4 + d][t]);
    const int64_t o = perm[i];
    const float o0 = N[o], o1 = N[n + o], o2 = N[2 * n + o];
    const double gl = sqrt((double)g[0] * g[0] + (double)g[1] * g[1] + (double)g[2] * g[2]);
    float n0 = o0, n1 = o1, n2 = o2;
    if (gl > 0.0 && gl <= 1.7976931348623157e308) {
      n0 = (float)(-(double)g[0] / gl);
      n1 = (float)(-(double)g[1] / gl);
      n2 = (float)(-(double)g[2] / gl);
    }
    const double e0 = (double)n0 - o0, e1 = (double)n1 - o1, e2 = (double)n2 - o2;
    const double ch = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
    const double h = 0.5 * ch;
    theta[i] = 2.0 * asin(h < 1.0 ? h : 1.0) * kRadToDeg;
    N[o] = n0;
    N[n + o] = n1;
    N[2 * n + o] = n2;
    const float k = kk[i];
    src[2 * i + 1] = make_float4(k * n0, k * n1, k * n2, 0.0f);
    wv = (double)w;
    cv = ch;
  }
  const double bw = block_sum(wv, lds);
  const double bc = block_sum(cv, lds);
  if (threadIdx.x == 0) {
    blk[blockIdx.x] = bw;
    blk[nblk + blockIdx.x] = bc;
  }
}

// Mean of w from the block partials (one block, fixed order).
__global__ __launch_bounds__(kRedBlock) void k_mean(const double* __restrict__ blk, int nblk, int64_t n,
                                                    double* __restrict__ out) {
  __shared__ double lds[kRedBlock / 64];
  double a = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) a += blk[i];
  const double sa = block_sum(a, lds);
  if (threadIdx.x == 0) *out = sa / (double)n;
}

// ---- Mean of the k largest angles (the convergence statistic), exact.
// Non-negative doubles order like their bits. Up to kSelRegs angles, one block holds them all in
// registers and narrows the range of the k-th largest by 2,048 bins at a time (k_stats_small).
// Above that, two histograms over all angles fix the top 28 bits of the k-th largest
// (k_sel_hist), the few angles that share them are gathered while those above are summed
// (k_sel_collect), and one block finishes (k_stats_final): 4 launches, against 19 for a
// select of 8 bits per pass. Where more angles share the 28 bits than that block holds (near convergence the
// changes of the FP32 normals are few distinct values), three more histograms over all angles fix the other 36
// bits (k_sel_collect, k_sel_deep; their launches end at once otherwise). One block going through all angles
// again took 0.8 us per 1,000 of them: 3.8 ms of an iteration of 1M tied points, 0.04 now. It still does for up
// to kSelDeepMin angles (32 for each thread). No floating-point sum depends on the order of
// an atomic: the angles that share the bits share an exponent, so theirs is an integer sum.
constexpr int kSelBlock = 1024;
constexpr int kSelPer = 16;
constexpr int kSelRegs = kSelBlock * kSelPer;
constexpr int kSelBins = 2048;
constexpr int kSelGrid = 256;              // blocks of the passes over all angles
constexpr int kTopShift = 49, kMidShift = 36;  // bits below the first and second histogram's digits
constexpr int kTopBins = 8256;             // 180 degrees and below: bits >> 49 <= 8243
constexpr int kMidBins = 1 << (kTopShift - kMidShift);
static_assert(kTopBins + kMidBins <= kSelHistLen && kSelRegs == kSelSmallMax, "workspace and rule of the selection");

// Range select over the values `visit` hands out (each call visits all of them): narrows [lo, lo +
// 2^width) to the k-th largest value. On return either the range is one value, or exactly krem
// values of the last range remain and all of them belong to the k largest. Block-wide.
struct Range {
  uint64_t lo;
  int sh;        // the range is [lo, lo + 2^sh)
  uint64_t krem; // how many of the values in the range are among the k largest
  bool whole;    // all values of the range are
};

struct SelLds {
  unsigned bins[kSelBins];
  unsigned wsum[kSelBlock / 64];
  int digit;
  unsigned above, count;
};

// The largest bin d of h[0..nb) with suffix count >= krem; above = the count of the bins over d. Bin
// loads through `load(i)`. One block of kSelBlock threads.
template <class F>
__device__ void find_bin(F load, int nb, uint64_t krem, SelLds& s) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int per = (nb + kSelBlock - 1) / kSelBlock;
  // thread t owns the bins [hi - per, hi) counted from the top
  const int hi = nb - t * per;
  unsigned sum = 0;
  for (int u = 1; u <= per; ++u) sum += hi - u >= 0 ? load(hi - u) : 0u;
  unsigned inc = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (t == 0) {
    s.digit = 0;
    s.above = 0;
    s.count = 0;
  }
  __syncthreads();
  if (lane == 63) s.wsum[wv] = inc;
  __syncthreads();
  unsigned before = inc - sum;
  for (int w = 0; w < wv; ++w) before += s.wsum[w];
  if (before < krem && before + sum >= krem) {  // exactly one thread when the total is >= krem
    unsigned c = before;
    for (int u = 1; u <= per; ++u) {
      const unsigned x = load(hi - u);
      if (c + x >= krem) {
        s.digit = hi - u;
        s.above = c;
        s.count = x;
        break;
      }
      c += x;
    }
  }
  __syncthreads();
}

template <class V>
__device__ void narrow(V visit, Range& r, SelLds& s) {
  while (r.sh > 0 && !r.whole) {
    const int step = r.sh > 11 ? r.sh - 11 : 0;
    for (int i = threadIdx.x; i < kSelBins; i += kSelBlock) s.bins[i] = 0;
    __syncthreads();
    const uint64_t lo = r.lo, last = r.lo + ((1ull << r.sh) - 1ull);
    visit([&](uint64_t b) {
      if (b >= lo && b <= last) atomicAdd(&s.bins[(b - lo) >> step], 1u);
    });
    __syncthreads();
    find_bin([&](int i) { return s.bins[i]; }, 1 << (r.sh - step), r.krem, s);
    r.lo += (uint64_t)s.digit << step;
    r.krem -= s.above;
    r.sh = step;
    r.whole = s.count == r.krem;
    __syncthreads();
  }
}

// Sums the block partials of w and the chord into stats[0] and stats[2] (block-wide).
__device__ void mean_stats(const double* blk, int nblk, int64_t n, const double* iso, double* lds, double* stats) {
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
    a += blk[i];
    b += blk[nblk + i];
  }
  const double sa = block_sum(a, lds);
  const double sb = block_sum(b, lds);
  if (threadIdx.x == 0) {
    stats[0] = iso ? *iso : sa / (double)n;
    stats[2] = sb / (double)n;
  }
}

// Sets the flag when the iteration ends with these statistics: a value that is not finite, or a
// largest angle change within eps_deg (negative: never).
__device__ __forceinline__ void set_stop(const double* stats, double eps_deg, int32_t* stop) {
  if (!stop) return;
  if (!isfinite(stats[0]) || !isfinite(stats[1]) || !isfinite(stats[2]) || stats[1] <= eps_deg) *stop = 1;
}

__global__ __launch_bounds__(kSelBlock) void k_stats_small(const double* __restrict__ theta, int n, int64_t k,
                                                           const double* __restrict__ blk, int nblk,
                                                           const double* __restrict__ iso, double* stats,
                                                           double eps_deg, int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ SelLds s;
  __shared__ double lds[kSelBlock / 64];
  __shared__ uint64_t ext[2][kSelBlock / 64];
  const int t = threadIdx.x;
  double v[kSelPer];
  uint64_t mx = 0, mn = ~0ull;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const int i = t + j * kSelBlock;
    v[j] = i < n ? theta[i] : 0.0;
    const uint64_t b = (uint64_t)__double_as_longlong(v[j]);
    if (i < n) {
      mx = b > mx ? b : mx;
      mn = b < mn ? b : mn;
    }
  }
  mean_stats(blk, nblk, n, iso, lds, stats);
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t x = __shfl_xor((unsigned long long)mx, o, 64), y = __shfl_xor((unsigned long long)mn, o, 64);
    mx = x > mx ? x : mx;
    mn = y < mn ? y : mn;
  }
  if ((t & 63) == 0) {
    ext[0][t >> 6] = mx;
    ext[1][t >> 6] = mn;
  }
  __syncthreads();
  for (int w = 0; w < kSelBlock / 64; ++w) {
    mx = ext[0][w] > mx ? ext[0][w] : mx;
    mn = ext[1][w] < mn ? ext[1][w] : mn;
  }
  Range r{mn, mx == mn ? 0 : 64 - __clzll((long long)(mx - mn)), (uint64_t)k, k == n};
  auto visit = [&](auto f) {
#pragma unroll
    for (int j = 0; j < kSelPer; ++j)
      if (t + j * kSelBlock < n) f((uint64_t)__double_as_longlong(v[j]));
  };
  narrow(visit, r, s);
  double sum = 0.0;
#pragma unroll
  for (int j = 0; j < kSelPer; ++j) {
    const uint64_t b = (uint64_t)__double_as_longlong(v[j]);
    if (t + j * kSelBlock < n && (r.whole ? b >= r.lo : b > r.lo)) sum += v[j];
  }
  const double total = block_sum(sum, lds);
  if (t == 0) {
    const double rest = r.whole ? 0.0 : (double)r.krem * __longlong_as_double((long long)r.lo);
    stats[1] = (total + rest) / (double)k;
    set_stop(stats, eps_deg, stop);
  }
}

// sel[0] = first digit, sel[1] = values among the k largest with that digit, sel[2] = gathered
// values (the rest of sel: k_sel_collect, k_sel_deep). MID = false: histogram of the first digit. MID = true:
// finds the first digit and takes the histogram of the second among the values that have it.
template <bool MID>
__global__ __launch_bounds__(kSelBlock) void k_sel_hist(const double* __restrict__ theta, int64_t n, int64_t k,
                                                        uint32_t* __restrict__ hist, uint64_t* __restrict__ sel,
                                                        const int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ SelLds s;
  __shared__ unsigned bins[MID ? kMidBins : kTopBins];
  constexpr int kBins = MID ? kMidBins : kTopBins;
  uint32_t* const top = hist;
  uint32_t* const mine = MID ? hist + kTopBins : hist;
  for (int i = threadIdx.x; i < kBins; i += kSelBlock) bins[i] = 0;
  uint64_t first = 0;
  if (MID) {
    find_bin([&](int i) { return top[i]; }, kTopBins, (uint64_t)k, s);
    first = (uint64_t)s.digit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sel[0] = first;
      sel[1] = (uint64_t)k - s.above;
      sel[2] = 0;
    }
  }
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * kSelBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSelBlock) {
    const uint64_t b = (uint64_t)__double_as_longlong(theta[i]);
    if (!MID) {
      const uint64_t d = b >> kTopShift;
      atomicAdd(&bins[d < kTopBins ? d : kTopBins - 1], 1u);
    } else if ((b >> kTopShift) == first) {
      atomicAdd(&bins[(b >> kMidShift) & (kMidBins - 1)], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kBins; i += kSelBlock)
    if (bins[i]) atomicAdd(&mine[i], bins[i]);
}

// The histograms of the other 36 bits, 12 at a time from the top: counts, and for the upper two the sums of
// the bits below the digit.
struct SelDeep {
  uint32_t* cnt[3];
  unsigned long long* sum[2];
  __device__ __forceinline__ explicit SelDeep(uint32_t* hist) {
    uint32_t* const p = hist + kSelHistLen;
    for (int l = 0; l < 3; ++l) cnt[l] = p + l * kSelDeepBins;
    for (int l = 0; l < 2; ++l) sum[l] = reinterpret_cast<unsigned long long*>(p + (3 + 2 * l) * kSelDeepBins);
  }
};
static_assert(kSelHistLen % 2 == 0 && kSelDeepBins == 1 << 12, "64-bit sums behind the counts, 12-bit digits");

struct DeepLds {
  unsigned cnt[kSelDeepBins];
  unsigned long long sum[kSelDeepBins];
};

// Histogram LEVEL of the offsets (36 bits, in their bucket) for which `take` holds.
template <int LEVEL, class F>
__device__ void deep_hist(const double* __restrict__ theta, int64_t n, uint64_t lo, F take, const SelDeep& d,
                          DeepLds& h) {
  constexpr int sh = 24 - 12 * LEVEL;
  for (int i = threadIdx.x; i < kSelDeepBins; i += kSelBlock) {
    h.cnt[i] = 0;
    h.sum[i] = 0;
  }
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * kSelBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSelBlock) {
    const uint64_t b = (uint64_t)__double_as_longlong(theta[i]), o = b - lo;
    if (b < lo || o >= (1ull << kMidShift) || !take(o)) continue;
    const int at = (int)(o >> sh) & (kSelDeepBins - 1);
    atomicAdd(&h.cnt[at], 1u);
    if (LEVEL < 2) atomicAdd(&h.sum[at], (unsigned long long)(o & ((1ull << sh) - 1ull)));
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSelDeepBins; i += kSelBlock) {
    if (!h.cnt[i]) continue;
    atomicAdd(&d.cnt[LEVEL][i], h.cnt[i]);
    if (LEVEL < 2) atomicAdd(&d.sum[LEVEL < 2 ? LEVEL : 0][i], h.sum[i]);
  }
}

// Sums, per block, the values above those with the selected 28 top bits, and gathers those that have them, or,
// where they are too many for that (and n > kSelDeepMin), counts the first 12 of their other bits. sel[3] =
// their lowest bit pattern, sel[4] = how many are among the k largest, sel[5] = how many there are.
__global__ __launch_bounds__(kSelBlock) void k_sel_collect(const double* __restrict__ theta, int64_t n,
                                                           uint32_t* __restrict__ hist,
                                                           uint64_t* __restrict__ sel, uint64_t* __restrict__ cand,
                                                           double* __restrict__ top,
                                                           const int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ SelLds s;
  __shared__ DeepLds h;
  __shared__ double lds[kSelBlock / 64];
  const uint64_t first = sel[0], krem = sel[1];
  find_bin([&](int i) { return hist[kTopBins + i]; }, kMidBins, krem, s);
  const uint64_t lo = (first << kTopShift) | ((uint64_t)s.digit << kMidShift), next = lo + (1ull << kMidShift);
  const bool deep = n > kSelDeepMin && s.count > kSelRegs;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sel[3] = lo;
    sel[4] = krem - s.above;
    sel[5] = s.count;
  }
  double v = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kSelBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kSelBlock) {
    const double x = theta[i];
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    if (b >= next) {
      v += x;
    } else if (b >= lo && !deep) {
      const uint64_t at = atomicAdd(reinterpret_cast<unsigned long long*>(&sel[2]), 1ull);
      if (at < kSelRegs) cand[at] = b;
    }
  }
  const double b = block_sum(v, lds);
  if (threadIdx.x == 0) top[blockIdx.x] = b;
  if (deep) deep_hist<0>(theta, n, lo, [](uint64_t) { return true; }, SelDeep(hist), h);
}

// LEVEL 1, 2: finds the digit of the level before and takes the histogram of the next 12 bits among the
// offsets that have it; nothing to do where the values were gathered. sel[4 + 2 LEVEL] = the digits found so far,
// sel[5 + 2 LEVEL] = values among the k largest that have them.
template <int LEVEL>
__global__ __launch_bounds__(kSelBlock) void k_sel_deep(const double* __restrict__ theta, int64_t n,
                                                        uint32_t* __restrict__ hist, uint64_t* __restrict__ sel,
                                                        const int32_t* __restrict__ stop) {
  if ((stop && *stop) || sel[5] <= kSelRegs) return;
  __shared__ SelLds s;
  __shared__ DeepLds h;
  const SelDeep d(hist);
  const uint64_t krem = LEVEL == 1 ? sel[4] : sel[7], found = LEVEL == 1 ? 0 : sel[6];
  find_bin([&](int i) { return d.cnt[LEVEL - 1][i]; }, kSelDeepBins, krem, s);
  const uint64_t digits = (found << 12) | (uint64_t)s.digit;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sel[4 + 2 * LEVEL] = digits;
    sel[5 + 2 * LEVEL] = krem - s.above;
  }
  deep_hist<LEVEL>(theta, n, sel[3], [&](uint64_t o) { return (o >> (36 - 12 * LEVEL)) == digits; }, d, h);
}

// Count and sum (minus base each) of the offsets that are among the k largest, but for those equal to the k-th:
// of the bins above the digit found, level by level. Adds this thread's share; *kth = the k-th
// largest offset, *krem = how many of its copies are among the k largest. Block-wide.
__device__ void deep_sum(const SelDeep& d, const uint64_t* __restrict__ sel, SelLds& s, uint64_t* hi, uint64_t* lo,
                         uint64_t* cnt, uint64_t* kth, uint64_t* krem) {
  const uint64_t left = sel[9], found = sel[8];
  find_bin([&](int i) { return d.cnt[2][i]; }, kSelDeepBins, left, s);
  *kth = (found << 12) | (uint64_t)s.digit;
  *krem = left - s.above;
#pragma unroll
  for (int level = 0; level < 3; ++level) {
    const int sh = 24 - 12 * level;
    const uint64_t digits = *kth >> sh, before = digits & ~(uint64_t)(kSelDeepBins - 1);
    for (int i = (int)(digits & (kSelDeepBins - 1)) + 1 + threadIdx.x; i < kSelDeepBins; i += kSelBlock) {
      const uint64_t c = d.cnt[level][i], o = (before | (uint64_t)i) << sh;
      *hi += c * (o >> 18);
      *lo += c * (o & 0x3ffffull);
      if (level < 2) {
        const uint64_t x = d.sum[level < 2 ? level : 0][i];
        *hi += x >> 18;
        *lo += x & 0x3ffffull;
      }
      *cnt += c;
    }
  }
}

__global__ __launch_bounds__(kSelBlock) void k_stats_final(const double* __restrict__ theta, int64_t n, int64_t k,
                                                           const double* __restrict__ blk, int nblk,
                                                           const double* __restrict__ iso,
                                                           uint32_t* __restrict__ hist,
                                                           const uint64_t* __restrict__ sel,
                                                           const uint64_t* __restrict__ cand,
                                                           const double* __restrict__ top, int ntop, double* stats,
                                                           double eps_deg, int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ SelLds s;
  __shared__ double lds[kSelBlock / 64];
  __shared__ unsigned long long part[2];  // integer sum of the low bits, in two halves
  __shared__ unsigned long long cnt;
  const int t = threadIdx.x;
  if (t < 2) part[t] = 0;
  if (t == 2) cnt = 0;
  mean_stats(blk, nblk, n, iso, lds, stats);
  const uint64_t base = sel[3];
  // sum of the values among the k largest but for the ones equal to the k-th: they share an exponent, so
  // value = base + (bits - base) ulp
  uint64_t hi = 0, lo = 0, c = 0;
  Range r{base, 0, 0, false};
  if (n > kSelDeepMin && sel[5] > kSelRegs) {
    deep_sum(SelDeep(hist), sel, s, &hi, &lo, &c, &r.lo, &r.krem);
    r.lo += base;
  } else {
    const uint64_t m = sel[2];
    const bool held = m <= kSelRegs;  // else (n <= kSelDeepMin, nearly all angles nearly equal) from all angles
    uint64_t v[kSelPer];
#pragma unroll
    for (int j = 0; j < kSelPer; ++j) {
      const uint64_t i = t + j * kSelBlock;
      v[j] = held && i < m ? cand[i] : ~0ull;
    }
    const uint64_t last = base + ((1ull << kMidShift) - 1ull);
    auto visit = [&](auto f) {
      if (held) {
#pragma unroll
        for (int j = 0; j < kSelPer; ++j)
          if (v[j] != ~0ull) f(v[j]);
      } else {
        for (int64_t i = t; i < n; i += kSelBlock) {
          const uint64_t b = (uint64_t)__double_as_longlong(theta[i]);
          if (b >= base && b <= last) f(b);
        }
      }
    };
    r = Range{base, kMidShift, sel[4], sel[4] == m};
    narrow(visit, r, s);
    visit([&](uint64_t b) {
      if (r.whole ? b >= r.lo : b > r.lo) {
        const uint64_t d = b - base;
        hi += d >> 18;
        lo += d & 0x3ffffull;
        ++c;
      }
    });
  }
  for (int o = 32; o > 0; o >>= 1) {
    hi += __shfl_xor((unsigned long long)hi, o, 64);
    lo += __shfl_xor((unsigned long long)lo, o, 64);
    c += __shfl_xor((unsigned long long)c, o, 64);
  }
  if ((t & 63) == 0) {
    atomicAdd(&part[0], hi);
    atomicAdd(&part[1], lo);
    atomicAdd(&cnt, c);
  }
  double above = 0.0;
  for (int i = t; i < ntop; i += kSelBlock) above += top[i];
  const double sum = block_sum(above, lds);  // its barriers publish part and cnt
  if (t == 0) {
    const int e = (int)(base >> 52);
    const double ulp = ldexp(1.0, (e > 0 ? e : 1) - 1075);
    const double in = (double)cnt * __longlong_as_double((long long)base) +
                      ((double)part[0] * 262144.0 + (double)part[1]) * ulp;
    const double rest = r.whole ? 0.0 : (double)r.krem * __longlong_as_double((long long)r.lo);
    stats[1] = (sum + in + rest) / (double)k;
    set_stop(stats, eps_deg, stop);
  }
}

// SplitMix64 output number t of the stream started at `seed` (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t t) {
  uint64_t z = seed + (t + 1ull) * 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

__global__ void k_random_normals(uint64_t seed, int64_t n, float* __restrict__ N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float u0 = (float)(splitmix64(seed, 2ull * i) >> 40) * 0x1p-24f;
  const float u1 = (float)(splitmix64(seed, 2ull * i + 1ull) >> 40) * 0x1p-24f;
  const float z = 1.0f - 2.0f * u0;                 // exact
  const float rr = sqrtf((1.0f - z) * (1.0f + z));  // one rounding before the sqrt
  float sn, cs;
  sincosf(6.28318530717958647692f * u1, &sn, &cs);
  N[i] = rr * cs;
  N[n + i] = rr * sn;
  N[2 * n + i] = z;
}

// Blocks that a launch is split into whatever that leaves per split: four rounds of the blocks
// that are resident at once (8 tiles per split at least left 4 blocks for 2,000 points and 400 for
// 20,000). 40,000 points of a sphere, gradient, plain / screened: 988 / 1275 us by the 8-tile rule, 822 / 1093
// at 2,560 blocks, 812 / 1046 at 5,120.
constexpr int64_t kSmallBlocks = 1024, kFillBlocks = 5120;
// (query block, source tile) pairs up to which a launch takes the small kernel: one tile per block
// of the other kernel is then still too few blocks. Whole calls at 500 / 2,000 / 8,000 / 12,000 points,
// screened, us: 36 / 44 / 122 / 179 against 68 / 71 / 127 / 189 with one-tile splits of the other kernel and
// 157 / 387 / 415 / 488 with the 8-tile rule; from 16,000 points on (2,016 pairs) it is slower for the
// plain kernel (219 against 210).
constexpr int64_t kSmallPairs = 1536;

bool small_launch(int64_t n_src, int64_t n_qry) { return cdiv(n_src, kTile) * cdiv(n_qry, kQBlock) <= kSmallPairs; }

template <bool SCREENED, bool KAHAN>
void launch_gwn_t(bool grad, hipStream_t st, const float* Q, int64_t m, const GwnWork& w, float kappa) {
  const int64_t nfull = w.n_src / kTile;  // tiles without padding
  const dim3 grid((unsigned)cdiv(m, kQBlock), (unsigned)w.split);
  if (small_launch(w.n_src, m)) {
    const int64_t steps = cdiv(w.n_src, kSmallStep), per = cdiv(steps, w.split);
    if (grad)
      hipLaunchKernelGGL((k_gwn_small<true, SCREENED, KAHAN>), grid, dim3(kQBlock), 0, st, Q, m, w.perm_q, w.src, steps,
                         nfull, per, w.tbox, kScaledScr, kappa, w.part, w.mpad, w.stop,
                       w.clock());
    else
      hipLaunchKernelGGL((k_gwn_small<false, SCREENED, KAHAN>), grid, dim3(kQBlock), 0, st, Q, m, w.perm_q, w.src, steps,
                         nfull, per, w.tbox, kScaledScr, kappa, w.part, w.mpad, w.stop,
                       w.clock());
    return;
  }
  const int64_t per = cdiv(w.ntiles, w.split);
  if (grad)
    hipLaunchKernelGGL((k_gwn<SCREENED, KAHAN>), grid, dim3(kBlock), 0, st, Q, m, w.perm_q, w.src, w.ntiles, nfull, per,
                       w.tbox, kScaledScr, kappa, w.part, w.mpad, w.stop,
                       w.clock());
  else
    hipLaunchKernelGGL((k_gwn_w<SCREENED, KAHAN>), grid, dim3(kBlock), 0, st, Q, m, w.perm_q, w.src, w.ntiles, nfull,
                       per, w.tbox, kScaledScr, kappa, w.part, w.mpad, w.stop,
                       w.clock());
}

}  // namespace

float position_scale(const dwg_kernel_params& kp) {
  return kp.lambda > 0.0f ? (float)(std::sqrt((double)kp.lambda) * 1.4426950408889634) : 1.0f;
}

int choose_split(int64_t n_src, int64_t n_qry, int requested) {
  const int64_t ntiles = cdiv(n_src, kTile);
  if (requested > 0) return (int)std::min<int64_t>(std::min<int64_t>(requested, kMaxSplit), ntiles);
  const int64_t qblocks = cdiv(n_qry, kQBlock);
  // Aim for >= 32768 blocks (128 per CU, ~25 rounds of resident blocks) while every split keeps
  // >= 8 tiles: blocks differ in cost (near tiles take the longer path), and the last round of
  // a launch with few rounds leaves CUs idle. Measured: 1M x 1M 2 splits 599 ms, 6 splits
  // 556 ms, 16 splits 550 ms; 100K x 100K 16 splits 6.14 ms, 48 splits 5.70 ms. The partial
  // sums (28 B per query and split) are held to kAutoSplitBytes, or 16 splits if that is more.
  int64_t s = cdiv(32768, qblocks);
  s = std::min<int64_t>(s, std::max<int64_t>(1, ntiles / 8));
  if (small_launch(n_src, n_qry))
    s = std::max<int64_t>(s, std::min<int64_t>(cdiv(kSmallBlocks, qblocks), cdiv(n_src, kSmallStep)));
  else
    s = std::max<int64_t>(s, std::min<int64_t>(cdiv(kFillBlocks, qblocks), ntiles));
  const int64_t mem_cap =
      std::max<int64_t>(16, (int64_t)(kAutoSplitBytes / ((int64_t)kNAcc * 4 * qblocks * kQBlock)));
  s = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(s, mem_cap), kMaxSplit));
  return (int)s;
}

// choose_split's rules times the blocks of queries, each by a bound that never falls as sources or queries
// grow: cdiv(B, x) x <= B - 1 + x. (`fill` takes the larger count of blocks and the finer step where the
// launch is not a small one, since launches of fewer queries can be.)
int64_t split_columns(int64_t n_src, int64_t n_qry, int requested) {
  const int64_t qblocks = cdiv(n_qry, kQBlock);
  if (requested > 0) return choose_split(n_src, n_qry, requested) * qblocks * kQBlock;
  const int64_t ntiles = cdiv(n_src, kTile);
  const int64_t rounds = std::min<int64_t>(32768 - 1 + qblocks, std::max<int64_t>(1, ntiles / 8) * qblocks);
  const int64_t fill = std::min<int64_t>((small_launch(n_src, n_qry) ? kSmallBlocks : kFillBlocks) - 1 + qblocks,
                                         cdiv(n_src, kSmallStep) * qblocks);
  const int64_t memory = std::max<int64_t>(16 * qblocks, kAutoSplitBytes / ((int64_t)kNAcc * 4 * kQBlock));
  const int64_t blocks = std::min<int64_t>(std::min<int64_t>(std::max<int64_t>(rounds, fill), memory), kMaxSplit * qblocks);
  return std::max<int64_t>(blocks, qblocks) * kQBlock;
}

size_t carve_gwn(Carver& c, int64_t n_src, int64_t n_qry, int split, int64_t columns, bool same, GwnWork* out) {
  GwnWork w{};
  w.n_src = n_src;
  w.ntiles = cdiv(n_src, kTile);
  w.npad = w.ntiles * kTile;
  w.mpad = padded_queries(n_qry);
  w.split = split;
  const size_t start = c.used;
  w.src = c.take<float4>(2 * (size_t)w.npad);
  w.part = c.take<float>((size_t)columns * kNAcc);
  w.kk = c.take<float>((size_t)w.npad);
  w.theta = c.take<double>((size_t)std::max(n_src, n_qry));
  w.blk = c.take<double>(2 * (size_t)std::max<int64_t>(cdiv(std::max(n_src, n_qry), 256), kEpiSmall / 64));
  w.stats = c.take<double>(kStatsRow * kAhead);
  w.stop = c.take<int32_t>(1);
  w.hist = c.take<uint32_t>(kSelHistLen + kSelDeepLen);
  w.sel = c.take<uint64_t>(kSelState);
  w.cand = c.take<uint64_t>(kSelSmallMax);
  w.top = c.take<double>(256);
  w.tbox = c.take<float4>(2 * (size_t)w.ntiles);
  w.perm_s = c.take<int32_t>((size_t)w.npad);
  w.perm_q = same ? w.perm_s : c.take<int32_t>((size_t)w.mpad);
  carve_sort(c, std::max(n_src, n_qry), &w.sort);
  if (out) *out = w;
  return c.used - start;
}

dwg_status launch_stage(const float* P, const float* N, const float* area, const float* delta,
                        int64_t n, float eps, float kappa, bool tiles, const GwnWork& w, hipStream_t stream) {
  hipLaunchKernelGGL(k_stage, dim3((unsigned)w.ntiles), dim3(kTile), 0, stream, P, N, area, delta, n, eps, kappa,
                     w.perm_s, w.src, w.kk, w.stop, tiles ? w.tbox : nullptr);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status launch_order(const float* P, int64_t n, const float* delta, float eps, float kappa, const float* Q,
                        int64_t m, bool same, const GwnWork& w, hipStream_t stream) {
  dwg_status s = spatial_sort(P, n, delta, eps, w.sort, w.perm_s, stream);
  if (s != DWG_OK) return s;
  if (!same) {
    s = spatial_sort(Q, m, nullptr, 0.0f, w.sort, w.perm_q, stream);
    if (s != DWG_OK) return s;
  }
  return DWG_OK;
}

dwg_status launch_gwn(const float* Q, int64_t m, const dwg_kernel_params& kp, bool grad,
                      const GwnWork& w, hipStream_t stream) {
  const bool scr = kp.lambda > 0.0f;
  const bool kah = kp.compensated != 0;
  const float kappa = position_scale(kp);
  if (scr)
    kah ? launch_gwn_t<true, true>(grad, stream, Q, m, w, kappa) : launch_gwn_t<true, false>(grad, stream, Q, m, w, kappa);
  else
    kah ? launch_gwn_t<false, true>(grad, stream, Q, m, w, kappa) : launch_gwn_t<false, false>(grad, stream, Q, m, w, kappa);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

// Which sums of partials take exact errors (see combine): gradients of octree walks, and all partials that
// are not compensated themselves. Kahan steps are enough for the others: all-pairs with compensation has 0.4 to
// 1.0 times the error of the coarser splits, octree values 0.6 to 0.97 times that of one walk.
static bool two_sum(const GwnWork& w, const dwg_kernel_params& kp, bool grad) {
  return kp.compensated == 0 || (w.walk && grad);
}

template <int QB, bool TWO>
static void combine_t(int nb, int64_t m, const dwg_kernel_params& kp, bool grad, float* wout, float* gout,
                      const GwnWork& w, hipStream_t stream) {
  hipLaunchKernelGGL((k_combine<QB, TWO>), dim3(nb), dim3(kEpiBlock), 0, stream, w.part, w.split, w.mpad, m, grad,
                     scale_of(kp), w.perm_q, wout, gout, w.blk);
}

dwg_status launch_combine(int64_t m, const dwg_kernel_params& kp, bool grad, float* wout,
                          float* gout, double* wmean, const GwnWork& w, hipStream_t stream) {
  const int qb = m <= kEpiSmall ? 64 : 256;
  const int nb = (int)cdiv(m, qb);
  const bool two = two_sum(w, kp, grad);
  auto* const run = qb == 64 ? (two ? combine_t<64, true> : combine_t<64, false>)
                             : (two ? combine_t<256, true> : combine_t<256, false>);
  run(nb, m, kp, grad, wout, gout, w, stream);
  DWG_TRY_LAUNCH();
  if (wmean) {
    hipLaunchKernelGGL(k_mean, dim3(1), dim3(kRedBlock), 0, stream, w.blk, nb, m, wmean);
    DWG_TRY_LAUNCH();
  }
  return DWG_OK;
}

template <int QB, bool TWO>
static void update_t(int nb, int64_t n, const dwg_kernel_params& kp, float* N, const GwnWork& w, hipStream_t stream) {
  hipLaunchKernelGGL((k_update<QB, TWO>), dim3(nb), dim3(kEpiBlock), 0, stream, w.part, w.split, w.mpad, n, scale_of(kp),
                     w.perm_s, w.kk, N, w.src, w.theta, w.blk, nb, w.hist, w.stop, w.clock() + 1);
}

dwg_status launch_update(int64_t n, const dwg_kernel_params& kp, float* N, const GwnWork& w, int* nblk,
                         hipStream_t stream) {
  const int qb = n <= kEpiSmall ? 64 : 256;
  const int nb = (int)cdiv(n, qb);
  const bool two = two_sum(w, kp, true);
  auto* const run = qb == 64 ? (two ? update_t<64, true> : update_t<64, false>)
                             : (two ? update_t<256, true> : update_t<256, false>);
  run(nb, n, kp, N, w, stream);
  DWG_TRY_LAUNCH();
  *nblk = nb;
  return DWG_OK;
}

static int64_t top_count(int64_t n, double top_frac) {
  int64_t k = (int64_t)std::ceil(top_frac * (double)n);
  if (k < 1) k = 1;
  if (k > n) k = n;
  return k;
}

dwg_status launch_stats(int64_t n, double top_frac, const GwnWork& w, int nblk, const double* iso,
                        double eps_deg, int32_t* stop, hipStream_t stream) {
  double* const stats = w.stats + kStatsRow * w.slot;
  const int64_t k = top_count(n, top_frac);
  if (n <= kSelSmallMax) {
    hipLaunchKernelGGL(k_stats_small, dim3(1), dim3(kSelBlock), 0, stream, w.theta, (int)n, k, w.blk, nblk, iso, stats,
                       eps_deg, stop);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  const int hb = (int)std::min<int64_t>(cdiv(n, kSelBlock), kSelGrid);
  hipLaunchKernelGGL((k_sel_hist<false>), dim3(hb), dim3(kSelBlock), 0, stream, w.theta, n, k, w.hist, w.sel, stop);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL((k_sel_hist<true>), dim3(hb), dim3(kSelBlock), 0, stream, w.theta, n, k, w.hist, w.sel, stop);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_sel_collect, dim3(hb), dim3(kSelBlock), 0, stream, w.theta, n, w.hist, w.sel, w.cand, w.top,
                     stop);
  DWG_TRY_LAUNCH();
  if (n > kSelDeepMin) {
    hipLaunchKernelGGL(k_sel_deep<1>, dim3(hb), dim3(kSelBlock), 0, stream, w.theta, n, w.hist, w.sel, stop);
    DWG_TRY_LAUNCH();
    hipLaunchKernelGGL(k_sel_deep<2>, dim3(hb), dim3(kSelBlock), 0, stream, w.theta, n, w.hist, w.sel, stop);
    DWG_TRY_LAUNCH();
  }
  hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(kSelBlock), 0, stream, w.theta, n, k, w.blk, nblk, iso, w.hist, w.sel,
                     w.cand, w.top, hb, stats, eps_deg, stop);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status launch_random_normals(uint64_t seed, int64_t n, float* N, hipStream_t stream) {
  hipLaunchKernelGGL(k_random_normals, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, stream, seed, n, N);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

}  // namespace dwg
