// The paper's own normal update (Sec. 4.3, Algorithm 1): the GWN at the nodes of a grid
// around the points, the iso-value w_bar (Eq. 6), the w_bar level set, one gradient per
// face from the cross product, and every face's gradient added to its k nearest input
// points, then normalised (Eq. 7).
//
// Grid. The octree frame (lo = bounding-box minimum, side = largest extent) cut into 2^depth
// cells per axis; a point's cell is its level-21 octree cell shifted down to `depth`. The
// evaluated cells are the cells holding points grown by `dilate` rings (inside the cube),
// in Morton order; their corners, without repetitions, are placed at
// lo + c * side / 2^depth (FP64, rounded once to FP32).
// Level set: Marching Cubes (the paper's "standard Marching Cubes"). Corner index
// x + 2y + 4z; a corner is above when w > w_bar; the case of a cube is the 8-bit mask of its
// above corners. Its triangles come from a 256-case table that this file derives at compile
// time from one face rule: every face, walked counter-clockwise as seen from outside,
// contributes a segment per run of above corners, from the cut edge where the walk enters the
// run to the cut edge where it leaves (so a face with its two above corners on a diagonal
// separates them, and two cubes sharing a face draw the same segments: the surface is
// closed); the segments chain into loops, each written from its lowest edge number (edges
// numbered by their corner pair (u, v), u < v, in lexicographic order), loops in that order,
// and cut into the fan (v0, vi, vi+1). That winding makes (q1 - q0) x (q2 - q0) point away
// from the above corners. A vertex on edge (u, v): p_u + (w_bar - w_u) / (w_v - w_u)
// (p_v - p_u), FP64. At most 5 triangles per cube.
// Option (not the paper's): marching tetrahedra, each cube cut into 6 tetrahedra around
// the diagonal from corner 0 to corner 7, one per order (a, b, c) of the axes: 0, e_a,
// e_a + e_b, 7, in the order (x,y,z), (x,z,y), (y,x,z), (y,z,x), (z,x,y), (z,y,x). One lone
// inside (or outside) vertex L: the triangle of the crossings on the edges from L to the
// other three in tetrahedron order; two inside A < B, outside C < D: the quad e(A,C), e(A,D),
// e(B,D), e(B,C) split into (e(A,C), e(A,D), e(B,D)) and (e(A,C), e(B,D), e(B,C)); each turned
// away from the tetrahedron's inside vertices (q1 and q2 swapped when turned).
// Scatter. The k nearest points of each face centroid (the uniform-grid kNN) receive the
// face vector through 64-bit fixed-point atomic adds (scale 2^40 / (3 h^2), h = the cell
// size; |components| <= 3 h^2): integer sums do not depend on the order of the atomics, so
// the result is deterministic.
#include <cmath>

#include "dwg_internal.h"
#include "dwg_morton.h"

#define DWG_PROPAGATE_INT(expr) \
  do {                          \
    dwg_status s_ = (expr);     \
    if (s_ != DWG_OK) return s_; \
  } while (0)

namespace dwg {
namespace {

using morton::compact21;

__device__ __forceinline__ uint64_t morton3(int x, int y, int z) { return morton::code3(x, y, z); }

unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, 256), 16384)); }

// Code of corner k (x + 2y + 4z) of the cell.
__device__ __forceinline__ uint64_t corner_code(uint64_t cell, int k) {
  return morton3(compact21(cell >> 2) + (k & 1), compact21(cell >> 1) + ((k >> 1) & 1),
                 compact21(cell) + ((k >> 2) & 1));
}

// Cell size = side / 2^depth, side = the largest extent of the bounding box (FP64).
__device__ __forceinline__ double cell_size(const float* __restrict__ box, int depth) {
  double side = (double)box[3] - (double)box[0];
  const double sy = (double)box[4] - (double)box[1], sz = (double)box[5] - (double)box[2];
  if (sy > side) side = sy;
  if (sz > side) side = sz;
  return side / (double)(1 << depth);
}

__device__ __forceinline__ void corner_position(uint64_t code, const double* __restrict__ frame, double h, int64_t id,
                                                int64_t ld, float* __restrict__ pos) {
  const int c[3] = {compact21(code >> 2), compact21(code >> 1), compact21(code)};
  for (int d = 0; d < 3; ++d) pos[d * ld + id] = (float)__dadd_rn(frame[d], __dmul_rn((double)c[d], h));
}

// Cell code of every point at `depth` (from the level-21 octree cell).
__global__ void k_mc_point_keys(const float* __restrict__ P, int64_t n, const double* __restrict__ frame, int depth,
                                uint64_t* __restrict__ key) {
  const int sh = morton::kDepth - depth;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c[3];
    morton::cell21(P, n, i, frame, c);
    key[i] = morton3(c[0] >> sh, c[1] >> sh, c[2] >> sh);
  }
}

// head[i] = 1 where sorted key i starts a run of equal keys below `limit`.
__global__ void k_mc_heads(const uint64_t* __restrict__ key, int64_t n, uint64_t limit, int32_t* __restrict__ head) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    head[i] = (key[i] < limit && (i == 0 || key[i] != key[i - 1])) ? 1 : 0;
}

// Compacts the run heads (off = exclusive scan of the heads).
__global__ void k_mc_compact(const uint64_t* __restrict__ key, int64_t n, uint64_t limit,
                             const int32_t* __restrict__ off, uint64_t* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if (key[i] < limit && (i == 0 || key[i] != key[i - 1])) out[off[i]] = key[i];
}

// The (2 dil + 1)^3 neighbours of every occupied cell; outside the cube (or past the count)
// a sentinel 2^(3 depth) that sorts after every cell.
__global__ void k_mc_dilate(const uint64_t* __restrict__ occ, const int32_t* __restrict__ count, int64_t cap,
                            int depth, int dil, uint64_t* __restrict__ key) {
  const int64_t o = *count;
  const int w = 2 * dil + 1, w3 = w * w * w;
  const int G = 1 << depth;
  const uint64_t sentinel = 1ull << (3 * depth);
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < cap * w3; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t c = t / w3;
    const int r = (int)(t % w3);
    uint64_t k = sentinel;
    if (c < o) {
      const uint64_t code = occ[c];
      const int x = compact21(code >> 2) + r % w - dil;
      const int y = compact21(code >> 1) + (r / w) % w - dil;
      const int z = compact21(code) + r / (w * w) - dil;
      if (x >= 0 && y >= 0 && z >= 0 && x < G && y < G && z < G) k = morton3(x, y, z);
    }
    key[t] = k;
  }
}

// ---- Sets of codes as bitmaps: bit b of word w stands for code 64 w + b, so the set bits in order
// are the distinct codes in ascending order, and a code's rank among them is the number of bits in
// the words before it (an exclusive scan of the words' counts) plus those below it in its word.
// One word is a 4 x 4 x 4 block of cells: growing by rings and the corners of the cells are shifts
// of a block and its neighbours, word by word, with no atomics but one per point. Sorting a code per
// candidate instead (27 per point, 8 per cell, most of them equal) took 265 and 175 us for 100K
// points at depth 7, 42 and 43 this way (212 and 156 for the first kernels alone when they set
// one bit at a time). Used when the words fit the arrays that the sort needs (bitmap_words): they
// are then at most as many as the codes, and scanning them costs less than one pass of the sort; a
// sparse set of a deep grid is sorted.
using Word = unsigned long long;

// An axis of a block: the bits of coordinate k are m0 << (k's shift); coordinate 1 is s0 bits up,
// 2 is s1 = 8 s0.
template <int S0>
struct Axis {
  static constexpr int S1 = 8 * S0;
  static constexpr Word mask(int k) {
    Word m = 0;
    for (int b = 0; b < 64; ++b)
      if (((b / S0) & 1) + 2 * ((b / S1) & 1) == k) m |= Word(1) << b;
    return m;
  }
  static constexpr Word M0 = mask(0), M1 = mask(1), M2 = mask(2), M3 = mask(3);
  // every cell moved by one along the axis, with what comes in from the block before / after
  static __device__ __forceinline__ Word up(Word w, Word before) {
    return ((w & (M0 | M2)) << S0) | ((w & M1) << (S1 - S0)) | ((before & M3) >> (S1 + S0));
  }
  static __device__ __forceinline__ Word down(Word w, Word after) {
    return ((w & (M1 | M3)) >> S0) | ((w & M2) >> (S1 - S0)) | ((after & M0) << (S1 + S0));
  }
  // grown by r <= 2 cells both ways
  static __device__ __forceinline__ Word grow(Word w, Word before, Word after, int r) {
    Word out = w, u = w, d = w;
    for (int k = 0; k < r; ++k) {
      u = up(u, before);
      before = up(before, 0);
      d = down(d, after);
      after = down(after, 0);
      out |= u | d;
    }
    return out;
  }
};
using AxisX = Axis<4>;
using AxisY = Axis<2>;
using AxisZ = Axis<1>;

// The word of block (x, y, z) of a cube of `side` blocks per axis; empty outside.
__device__ __forceinline__ Word block_at(const Word* __restrict__ bits, int side, int x, int y, int z) {
  if ((unsigned)x >= (unsigned)side || (unsigned)y >= (unsigned)side || (unsigned)z >= (unsigned)side) return 0;
  return bits[morton3(x, y, z)];
}
__device__ __forceinline__ int blocks_per_axis(int depth) { return depth > 2 ? 1 << (depth - 2) : 1; }

// The cells holding points.
__global__ void k_bits_occupied(const float* __restrict__ P, int64_t n, const double* __restrict__ frame, int depth,
                                Word* __restrict__ bits) {
  const int sh = morton::kDepth - depth;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    int c[3];
    morton::cell21(P, n, i, frame, c);
    const uint64_t code = morton3(c[0] >> sh, c[1] >> sh, c[2] >> sh);
    const Word b = Word(1) << (code & 63);
    if (!(bits[code >> 6] & b)) atomicOr(&bits[code >> 6], b);
  }
}

// Those cells grown by r rings inside the cube, and their number per word.
__global__ void k_bits_grow(const Word* __restrict__ occ, int64_t words, int depth, int r, Word* __restrict__ bits,
                            int32_t* __restrict__ cnt) {
  const int side = blocks_per_axis(depth);
  const Word inside = depth >= 2 ? ~Word(0) : (Word(1) << (1 << 3 * depth)) - 1;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x) {
    Word v = occ[i];
    if (r > 0) {
      const int x = compact21((uint64_t)i >> 2), y = compact21((uint64_t)i >> 1), z = compact21((uint64_t)i);
      Word plane[3];
#pragma unroll
      for (int dz = -1; dz <= 1; ++dz) {
        Word row[3];
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy)
          row[dy + 1] = AxisX::grow(block_at(occ, side, x, y + dy, z + dz), block_at(occ, side, x - 1, y + dy, z + dz),
                                    block_at(occ, side, x + 1, y + dy, z + dz), r);
        plane[dz + 1] = AxisY::grow(row[1], row[0], row[2], r);
      }
      v = AxisZ::grow(plane[1], plane[0], plane[2], r) & inside;
    }
    bits[i] = v;
    cnt[i] = __popcll(v);
  }
}

// The corners of the cells (every cell and the next one along each axis), and their number per word.
__global__ void k_bits_corners(const Word* __restrict__ cells, int depth, int64_t words, Word* __restrict__ bits,
                               int32_t* __restrict__ cnt) {
  const int side = blocks_per_axis(depth);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x) {
    const int x = compact21((uint64_t)i >> 2), y = compact21((uint64_t)i >> 1), z = compact21((uint64_t)i);
    Word v = 0;
    if (x <= side && y <= side && z <= side) {
      Word plane[2];
#pragma unroll
      for (int dz = 0; dz < 2; ++dz) {
        Word row[2];
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          const Word w = block_at(cells, side, x, y - dy, z - dz);
          row[dy] = w | AxisX::up(w, block_at(cells, side, x - 1, y - dy, z - dz));
        }
        plane[dz] = row[0] | AxisY::up(row[0], row[1]);
      }
      v = plane[0] | AxisZ::up(plane[0], plane[1]);
    }
    bits[i] = v;
    cnt[i] = __popcll(v);
  }
}

__device__ __forceinline__ int32_t bit_rank(const Word* __restrict__ bits, const int32_t* __restrict__ rank,
                                            uint64_t code) {
  return rank[code >> 6] + __popcll(bits[code >> 6] & ((Word(1) << (code & 63)) - 1));
}

// The codes in ascending order.
__global__ void k_bits_list(const Word* __restrict__ bits, int64_t words,
                            const int32_t* __restrict__ rank, uint64_t* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x) {
    int32_t at = rank[i];
    for (Word b = bits[i]; b; b &= b - 1) out[at++] = 64ull * (uint64_t)i + (uint64_t)(__ffsll(b) - 1);
  }
}

// Corner ids of every cell (the rank of the corner's code) and the corner positions.
__global__ void k_bits_corner_ids(const uint64_t* __restrict__ cells, int64_t C,
                                  const Word* __restrict__ bits, int64_t words,
                                  const int32_t* __restrict__ rank, const double* __restrict__ frame,
                                  const float* __restrict__ box, int depth, int32_t* __restrict__ cidx,
                                  float* __restrict__ pos, int64_t ld) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < 8 * C; t += step)
    cidx[t] = bit_rank(bits, rank, corner_code(cells[t >> 3], (int)(t & 7)));
  const double h = cell_size(box, depth);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += step) {
    int32_t id = rank[i];
    for (unsigned long long b = bits[i]; b; b &= b - 1ull, ++id)
      corner_position(64ull * (uint64_t)i + (uint64_t)(__ffsll(b) - 1), frame, h, id, ld, pos);
  }
}

// Corner lattice keys of every cell: key[8 cell + k] = Morton code of the corner.
__global__ void k_mc_corner_keys(const uint64_t* __restrict__ cells, int64_t C, uint64_t* __restrict__ key) {
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < 8 * C; t += (int64_t)gridDim.x * blockDim.x) {
    key[t] = corner_code(cells[t >> 3], (int)(t & 7));
  }
}

// Corner ids (rank of the distinct key), the cell-corner table and the corner positions.
__global__ void k_mc_corner_ids(const uint64_t* __restrict__ key, const int32_t* __restrict__ val, int64_t n8,
                                const int32_t* __restrict__ off, const double* __restrict__ frame,
                                const float* __restrict__ box, int depth, int32_t* __restrict__ cidx,
                                float* __restrict__ pos, int64_t ld) {
  const double h = cell_size(box, depth);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n8; i += (int64_t)gridDim.x * blockDim.x) {
    const bool head = i == 0 || key[i] != key[i - 1];
    const int32_t id = head ? off[i] : off[i] - 1;
    cidx[val[i]] = id;
    if (head) corner_position(key[i], frame, h, id, ld, pos);
  }
}

// The 6 tetrahedra of a cube (corner indices, x + 2y + 4z).
__constant__ int kTet[6][4] = {{0, 1, 3, 7}, {0, 1, 5, 7}, {0, 2, 3, 7}, {0, 2, 6, 7}, {0, 4, 5, 7}, {0, 4, 6, 7}};

struct Vec3 {
  double x, y, z;
};
__device__ __forceinline__ Vec3 lerp_cross(const Vec3& a, const Vec3& b, double wa, double wb, double iso) {
  const double t = (iso - wa) / (wb - wa);
  return Vec3{a.x + t * (b.x - a.x), a.y + t * (b.y - a.y), a.z + t * (b.z - a.z)};
}

// Triangles of one tetrahedron: returns the count (0..2) and writes them when out != null.
__device__ int tet_faces(const Vec3* p, const double* w, double iso, Vec3 (*out)[3], Vec3* vec) {
  bool in[4];
  int k = 0;
  for (int t = 0; t < 4; ++t) {
    in[t] = w[t] > iso;
    k += in[t] ? 1 : 0;
  }
  if (k == 0 || k == 4) return 0;
  if (!out) return (k == 2) ? 2 : 1;
  int nf;
  if (k == 1 || k == 3) {
    int lone = 0;
    for (int t = 0; t < 4; ++t)
      if (in[t] == (k == 1)) lone = t;
    int j = 0;
    for (int t = 0; t < 4; ++t)
      if (t != lone) out[0][j++] = lerp_cross(p[lone], p[t], w[lone], w[t], iso);
    nf = 1;
  } else {
    int ins[2], outs[2], a = 0, b = 0;
    for (int t = 0; t < 4; ++t) {
      if (in[t])
        ins[a++] = t;
      else
        outs[b++] = t;
    }
    const int A = ins[0], B = ins[1], C = outs[0], D = outs[1];
    const Vec3 eAC = lerp_cross(p[A], p[C], w[A], w[C], iso), eAD = lerp_cross(p[A], p[D], w[A], w[D], iso);
    const Vec3 eBD = lerp_cross(p[B], p[D], w[B], w[D], iso), eBC = lerp_cross(p[B], p[C], w[B], w[C], iso);
    out[0][0] = eAC, out[0][1] = eAD, out[0][2] = eBD;
    out[1][0] = eAC, out[1][1] = eBD, out[1][2] = eBC;
    nf = 2;
  }
  Vec3 cin{0, 0, 0};
  for (int t = 0; t < 4; ++t)
    if (in[t]) cin.x += p[t].x, cin.y += p[t].y, cin.z += p[t].z;
  cin.x /= k, cin.y /= k, cin.z /= k;
  for (int f = 0; f < nf; ++f) {
    const Vec3 &q0 = out[f][0], &q1 = out[f][1], &q2 = out[f][2];
    const double ux = q1.x - q0.x, uy = q1.y - q0.y, uz = q1.z - q0.z;
    const double vx = q2.x - q0.x, vy = q2.y - q0.y, vz = q2.z - q0.z;
    Vec3 c{uy * vz - uz * vy, uz * vx - ux * vz, ux * vy - uy * vx};
    const double cx = (q0.x + q1.x + q2.x) / 3.0, cy = (q0.y + q1.y + q2.y) / 3.0, cz = (q0.z + q1.z + q2.z) / 3.0;
    if (c.x * (cin.x - cx) + c.y * (cin.y - cy) + c.z * (cin.z - cz) > 0.0) {
      c = Vec3{-c.x, -c.y, -c.z};
      const Vec3 tmp = out[f][1];  // wind the triangle the way its vector points
      out[f][1] = out[f][2];
      out[f][2] = tmp;
    }
    vec[f] = c;
  }
  return nf;
}

// ---- Marching Cubes case table (built at compile time from the face rule above) ----
constexpr int kMcMaxTri = 5;
struct McTable {
  uint8_t ntri[256];
  uint8_t tri[256][3 * kMcMaxTri];  // edge numbers, three per triangle
};
// edge e joins corners kEdgeLo[e] < kEdgeHi[e]
constexpr int kEdgeLo[12] = {0, 0, 0, 1, 1, 2, 2, 3, 4, 4, 5, 6};
constexpr int kEdgeHi[12] = {1, 2, 4, 3, 5, 3, 6, 7, 5, 6, 7, 7};
// the corners of each face, counter-clockwise as seen from outside the cube
constexpr int kFaceCyc[6][4] = {{0, 4, 6, 2}, {1, 3, 7, 5}, {0, 1, 5, 4}, {2, 6, 7, 3}, {0, 2, 3, 1}, {4, 5, 7, 6}};

constexpr int mc_edge(int a, int b) {
  const int lo = a < b ? a : b, hi = a < b ? b : a;
  for (int e = 0; e < 12; ++e)
    if (kEdgeLo[e] == lo && kEdgeHi[e] == hi) return e;
  return -1;
}

constexpr McTable make_mc_table() {
  McTable t{};
  for (int c = 0; c < 256; ++c) {
    int next[12] = {-1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
    for (int f = 0; f < 6; ++f)
      for (int i = 0; i < 4; ++i) {
        const int a = kFaceCyc[f][i], b = kFaceCyc[f][(i + 1) & 3];
        if (((c >> a) & 1) || !((c >> b) & 1)) continue;  // the walk enters a run at (a, b)
        int j = (i + 1) & 3;
        while ((c >> kFaceCyc[f][(j + 1) & 3]) & 1) j = (j + 1) & 3;
        next[mc_edge(a, b)] = mc_edge(kFaceCyc[f][j], kFaceCyc[f][(j + 1) & 3]);
      }
    bool used[12] = {};
    int nt = 0;
    for (int e = 0; e < 12; ++e) {
      if (next[e] < 0 || used[e]) continue;
      int loop[12] = {}, len = 0;
      for (int x = e; !used[x]; x = next[x]) {
        used[x] = true;
        loop[len++] = x;
      }
      for (int v = 1; v + 1 < len; ++v, ++nt) {
        t.tri[c][3 * nt + 0] = (uint8_t)loop[0];
        t.tri[c][3 * nt + 1] = (uint8_t)loop[v];
        t.tri[c][3 * nt + 2] = (uint8_t)loop[v + 1];
      }
    }
    t.ntri[c] = (uint8_t)nt;
  }
  return t;
}
constexpr McTable kMcHost = make_mc_table();
static_assert(kMcHost.ntri[0] == 0 && kMcHost.ntri[255] == 0 && kMcHost.ntri[1] == 1, "table");
constexpr int mc_max_tri() {
  int m = 0;
  for (int c = 0; c < 256; ++c) m = kMcHost.ntri[c] > m ? kMcHost.ntri[c] : m;
  return m;
}
static_assert(mc_max_tri() == kMcMaxTri, "at most five triangles per cube");
__constant__ McTable kMc = kMcHost;

__device__ void load_cell(int64_t ci, const int32_t* __restrict__ cidx, const float* __restrict__ pos, int64_t ld,
                          const float* __restrict__ w, Vec3* p, double* wv) {
  for (int k = 0; k < 8; ++k) {
    const int64_t id = cidx[8 * ci + k];
    p[k] = Vec3{pos[id], pos[ld + id], pos[2 * ld + id]};
    wv[k] = w[id];
  }
}

__global__ void k_mt_count(int64_t C, const int32_t* __restrict__ cidx, const float* __restrict__ pos, int64_t ld,
                           const float* __restrict__ w, const double* __restrict__ iso_p, int32_t* __restrict__ cnt) {
  const double iso = *iso_p;
  for (int64_t ci = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; ci < C; ci += (int64_t)gridDim.x * blockDim.x) {
    Vec3 p[8];
    double wv[8];
    load_cell(ci, cidx, pos, ld, w, p, wv);
    int c = 0;
    for (int t = 0; t < 6; ++t) {
      Vec3 tp[4];
      double tw[4];
      for (int j = 0; j < 4; ++j) {
        tp[j] = p[kTet[t][j]];
        tw[j] = wv[kTet[t][j]];
      }
      c += tet_faces(tp, tw, iso, nullptr, nullptr);
    }
    cnt[ci] = c;
  }
}

// Faces of every cell at off[ci]: centroids (planar [3][ldf]), vectors, and optionally the
// triangles ([F][9]: q0, q1, q2).
__global__ void k_mt_emit(int64_t C, const int32_t* __restrict__ cidx, const float* __restrict__ pos, int64_t ld,
                          const float* __restrict__ w, const double* __restrict__ iso_p,
                          const int32_t* __restrict__ off, int64_t fcap, float* __restrict__ cen, int64_t ldf,
                          float4* __restrict__ vec, float* __restrict__ tri, int64_t tcap) {
  const double iso = *iso_p;
  for (int64_t ci = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; ci < C; ci += (int64_t)gridDim.x * blockDim.x) {
    Vec3 p[8];
    double wv[8];
    load_cell(ci, cidx, pos, ld, w, p, wv);
    int64_t f = off[ci];
    for (int t = 0; t < 6; ++t) {
      Vec3 tp[4];
      double tw[4];
      for (int j = 0; j < 4; ++j) {
        tp[j] = p[kTet[t][j]];
        tw[j] = wv[kTet[t][j]];
      }
      Vec3 out[2][3], v[2];
      const int nf = tet_faces(tp, tw, iso, out, v);
      for (int s = 0; s < nf; ++s, ++f) {
        if (f >= fcap) continue;
        if (cen) {
          cen[f] = (float)((out[s][0].x + out[s][1].x + out[s][2].x) / 3.0);
          cen[ldf + f] = (float)((out[s][0].y + out[s][1].y + out[s][2].y) / 3.0);
          cen[2 * ldf + f] = (float)((out[s][0].z + out[s][1].z + out[s][2].z) / 3.0);
        }
        if (vec) vec[f] = make_float4((float)v[s].x, (float)v[s].y, (float)v[s].z, 0.0f);
        if (tri && f < tcap)
          for (int q = 0; q < 3; ++q) {
            tri[9 * f + 3 * q + 0] = (float)out[s][q].x;
            tri[9 * f + 3 * q + 1] = (float)out[s][q].y;
            tri[9 * f + 3 * q + 2] = (float)out[s][q].z;
          }
      }
    }
  }
}

// Case of cell ci: the 8-bit mask of its corners above.
__device__ __forceinline__ int mc_case(int64_t ci, const int32_t* __restrict__ cidx, const float* __restrict__ w,
                                       double iso) {
  int c = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) c |= ((double)w[cidx[8 * ci + k]] > iso ? 1 : 0) << k;
  return c;
}

struct McEdges {
  uint8_t lo[12], hi[12];
};
constexpr McEdges make_edges() {
  McEdges e{};
  for (int i = 0; i < 12; ++i) e.lo[i] = (uint8_t)kEdgeLo[i], e.hi[i] = (uint8_t)kEdgeHi[i];
  return e;
}
__constant__ McEdges kEdges = make_edges();

// The vertex on edge e of cell ci.
__device__ __forceinline__ Vec3 mc_vertex(int e, int64_t ci, const int32_t* __restrict__ cidx,
                                          const float* __restrict__ pos, int64_t ld, const float* __restrict__ w,
                                          double iso) {
  const int64_t u = cidx[8 * ci + kEdges.lo[e]], v = cidx[8 * ci + kEdges.hi[e]];
  return lerp_cross(Vec3{pos[u], pos[ld + u], pos[2 * ld + u]}, Vec3{pos[v], pos[ld + v], pos[2 * ld + v]}, w[u], w[v],
                    iso);
}

__global__ void k_mc_count(int64_t C, const int32_t* __restrict__ cidx, const float* __restrict__ w,
                           const double* __restrict__ iso_p, int32_t* __restrict__ cnt) {
  const double iso = *iso_p;
  for (int64_t ci = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; ci < C; ci += (int64_t)gridDim.x * blockDim.x) {
    cnt[ci] = kMc.ntri[mc_case(ci, cidx, w, iso)];
  }
}

// Triangles of every cell at off[ci], in table order: centroids (planar [3][ldf]), face
// vectors (q1 - q0) x (q2 - q0), and optionally the triangles ([F][9]: q0, q1, q2). Most cells have
// none and leave after their count; the others read the corners of their cut edges where they
// lie (all eight corners of every cell in arrays, indexed by edge, went through scratch memory: 35 us for
// 100K points at depth 7; 15 now).
__global__ void k_mc_emit(int64_t C, const int32_t* __restrict__ cidx, const float* __restrict__ pos, int64_t ld,
                          const float* __restrict__ w, const double* __restrict__ iso_p,
                          const int32_t* __restrict__ off, int64_t fcap, float* __restrict__ cen, int64_t ldf,
                          float4* __restrict__ vec, float* __restrict__ tri, int64_t tcap) {
  const double iso = *iso_p;
  for (int64_t ci = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; ci < C; ci += (int64_t)gridDim.x * blockDim.x) {
    int64_t f = off[ci];
    const int nt = off[ci + 1] - off[ci];
    if (nt == 0) continue;
    const int c = mc_case(ci, cidx, w, iso);
    for (int s = 0; s < nt; ++s, ++f) {
      if (f >= fcap) continue;
      const Vec3 q0 = mc_vertex(kMc.tri[c][3 * s], ci, cidx, pos, ld, w, iso),
                 q1 = mc_vertex(kMc.tri[c][3 * s + 1], ci, cidx, pos, ld, w, iso),
                 q2 = mc_vertex(kMc.tri[c][3 * s + 2], ci, cidx, pos, ld, w, iso);
      const double ux = q1.x - q0.x, uy = q1.y - q0.y, uz = q1.z - q0.z;
      const double vx = q2.x - q0.x, vy = q2.y - q0.y, vz = q2.z - q0.z;
      if (cen) {
        cen[f] = (float)((q0.x + q1.x + q2.x) / 3.0);
        cen[ldf + f] = (float)((q0.y + q1.y + q2.y) / 3.0);
        cen[2 * ldf + f] = (float)((q0.z + q1.z + q2.z) / 3.0);
      }
      if (vec)
        vec[f] = make_float4((float)(uy * vz - uz * vy), (float)(uz * vx - ux * vz), (float)(ux * vy - uy * vx), 0.0f);
      if (tri && f < tcap) {
        const Vec3 q[3] = {q0, q1, q2};
        for (int k = 0; k < 3; ++k) {
          tri[9 * f + 3 * k + 0] = (float)q[k].x;
          tri[9 * f + 3 * k + 1] = (float)q[k].y;
          tri[9 * f + 3 * k + 2] = (float)q[k].z;
        }
      }
    }
  }
}

__device__ __forceinline__ double fixed_scale(const double* frame, int depth) {
  const double sc = frame[3];
  const double h = sc > 0.0 ? (2097152.0 / sc) / (double)(1 << depth) : 0.0;
  return h > 0.0 ? 1099511627776.0 / (3.0 * h * h) : 1.0;  // 2^40 / (3 h^2)
}

// Every face of the chunk adds its vector to its k nearest points (fixed point): a thread per
// (face, neighbour, component), so that a wavefront reads consecutive neighbours and the three
// additions to a point fall into one request. The atomics bound it. (A thread per face with 3 k
// additions one after another, the level set of 100K points at depth 7, k = 10: 106 us; 50 now.)
__global__ void k_mc_scatter(const int32_t* __restrict__ idx, int64_t m, int k, const float4* __restrict__ vec,
                             const double* __restrict__ frame, int depth, int64_t n,
                             unsigned long long* __restrict__ acc) {
  const double S = fixed_scale(frame, depth);
  const float* const v = reinterpret_cast<const float*>(vec);
  const uint32_t total = 3u * (uint32_t)(m * k);  // m <= 2^20, k <= kMaxK
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const uint32_t e = i / 3u, d = i - 3u * e, f = e / (uint32_t)k;
    const int64_t j = idx[e];
    if (j < 0 || j >= n) continue;
    atomicAdd(&acc[3 * j + d], (unsigned long long)llrint((double)v[4 * f + d] * S));
  }
}

__device__ double mc_block_sum(double v, double* lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += lds[k];
  return r;
}

// Eq. 7 with the face sums: n = normalize(sum) (kept when the sum is 0), in place at the
// point's original index; theta and the chord partials; restaged moments; cleared sums and selection histograms.
__global__ __launch_bounds__(256) void k_mc_update(const int32_t* __restrict__ perm, int64_t n,
                                                   unsigned long long* __restrict__ acc,
                                                   const double* __restrict__ frame, int depth,
                                                   const float* __restrict__ kk, float* __restrict__ N,
                                                   float4* __restrict__ src, double* __restrict__ theta,
                                                   double* __restrict__ blk, int nblk,
                                                   uint32_t* __restrict__ hist) {
  __shared__ double lds[4];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  clear_hist(hist, n);
  double cv = 0.0;
  if (i < n) {
    const int64_t o = perm[i];
    const double S = fixed_scale(frame, depth);
    const double ax = (double)(long long)acc[3 * o] / S, ay = (double)(long long)acc[3 * o + 1] / S,
                 az = (double)(long long)acc[3 * o + 2] / S;
    acc[3 * o] = acc[3 * o + 1] = acc[3 * o + 2] = 0ull;
    const float o0 = N[o], o1 = N[n + o], o2 = N[2 * n + o];
    const double l = sqrt(ax * ax + ay * ay + az * az);
    float n0 = o0, n1 = o1, n2 = o2;
    if (l > 0.0 && l <= 1.7976931348623157e308) {
      n0 = (float)(ax / l);
      n1 = (float)(ay / l);
      n2 = (float)(az / l);
    }
    const double e0 = (double)n0 - o0, e1 = (double)n1 - o1, e2 = (double)n2 - o2;
    const double ch = sqrt(e0 * e0 + e1 * e1 + e2 * e2);
    const double h = 0.5 * ch;
    theta[i] = 2.0 * asin(h < 1.0 ? h : 1.0) * 57.295779513082320876798;
    N[o] = n0;
    N[n + o] = n1;
    N[2 * n + o] = n2;
    const float k = kk[i];
    src[2 * i + 1] = make_float4(k * n0, k * n1, k * n2, 0.0f);
    cv = ch;
  }
  const double bc = mc_block_sum(cv, lds);
  if (threadIdx.x == 0) {
    blk[blockIdx.x] = 0.0;
    blk[nblk + blockIdx.x] = bc;
  }
}

// Copies the points behind the corners in the query array (columns m .. m + n).
__global__ void k_mc_append_points(const float* __restrict__ P, int64_t n, float* __restrict__ pos, int64_t ld,
                                   int64_t m) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    for (int d = 0; d < 3; ++d) pos[d * ld + m + i] = P[d * n + i];
}

// FP64 mean of w[0..n): per-block partials (fixed shuffle tree), then one block in order.
__global__ __launch_bounds__(256) void k_mc_mean_part(const float* __restrict__ w, int64_t n,
                                                      double* __restrict__ part) {
  __shared__ double lds[4];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    s += (double)w[i];
  const double b = mc_block_sum(s, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = b;
}

__global__ __launch_bounds__(256) void k_mc_mean_final(const double* __restrict__ part, int nb, int64_t n,
                                                       double* __restrict__ out) {
  __shared__ double lds[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) s += part[i];
  const double b = mc_block_sum(s, lds);
  if (threadIdx.x == 0) *out = b / (double)n;
}

__global__ void k_zero_u64(unsigned long long* __restrict__ a, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = 0ull;
}

}  // namespace

int64_t mc_key_cap(int64_t n, const McParams& mp) {
  const int64_t w = 2 * mp.dilate + 1;
  return n * w * w * w;
}

size_t carve_mc_grid(Carver& c, int64_t n, const McParams& mp, McWork* out) {
  const size_t s0 = c.used;
  McWork w{};
  w.n = n;
  w.kcap = std::max<int64_t>(mc_key_cap(n, mp), n);
  w.bpart = c.take<float>(kBboxParts);
  w.box = c.take<float>(8);
  w.frame = c.take<double>(4);
  w.key[0] = c.take<uint64_t>((size_t)w.kcap);
  w.key[1] = c.take<uint64_t>((size_t)w.kcap);
  w.work = c.take<int32_t>(radix_work_len(w.kcap));
  w.head = c.take<int32_t>((size_t)w.kcap + 1);
  w.hdsums = c.take<int32_t>(scan_sums_len(w.kcap));
  w.occ = c.take<uint64_t>((size_t)n);
  w.cells = c.take<uint64_t>((size_t)w.kcap);
  if (out) *out = w;
  return c.used - s0;
}

int mc_faces_per_cell(const McParams& mp) { return mp.tets ? 12 : kMcMaxTri; }

size_t carve_mc_faces(Carver& c, int64_t n, int64_t C, const McParams& mp, McWork* w) {
  const size_t s0 = c.used;
  const int k = mp.k;
  McWork t{};
  McWork* o = w ? w : &t;
  o->C = C;
  o->tets = mp.tets;
  o->mcap = 8 * C;
  o->fcap = mc_faces_per_cell(mp) * C;
  o->chunk = std::min<int64_t>(std::max<int64_t>(o->fcap, 1), int64_t(1) << 20);
  o->ckey[0] = c.take<uint64_t>((size_t)(8 * C));
  o->ckey[1] = c.take<uint64_t>((size_t)(8 * C));
  o->cval[0] = c.take<int32_t>((size_t)(8 * C));
  o->cval[1] = c.take<int32_t>((size_t)(8 * C));
  o->cwork = c.take<int32_t>(radix_work_len(8 * C));
  o->chead = c.take<int32_t>((size_t)(8 * C) + 1);
  o->chdsums = c.take<int32_t>(scan_sums_len(8 * C));
  o->cidx = c.take<int32_t>((size_t)(8 * C));
  o->pos = c.take<float>((size_t)(3 * (o->mcap + n)));
  o->wc = c.take<float>((size_t)(o->mcap + n));
  o->iso = c.take<double>(1);
  o->ipart = c.take<double>(256);
  o->fcnt = c.take<int32_t>((size_t)C + 1);
  o->fsums = c.take<int32_t>(scan_sums_len(C));
  o->cen = c.take<float>((size_t)(3 * o->fcap));
  o->vec = c.take<float4>((size_t)o->fcap);
  o->idx = c.take<int32_t>((size_t)(o->chunk * k));
  o->dist = c.take<float>((size_t)(o->chunk * k));
  o->acc = c.take<unsigned long long>((size_t)(3 * n));
  carve_knn(c, n, o->chunk, &o->knn);
  return c.used - s0;
}

namespace {
// Words of a bitmap over the codes of 3 x bits, when `sets` of them and a count per word fit the
// sort's arrays of `keys` keys; 0 otherwise.
int64_t bitmap_words(int bits, int sets, int64_t keys) {
  const int64_t words = int64_t(1) << std::max(0, 3 * bits - 6);
  return 3 * bits <= 48 && sets * words <= keys ? words : 0;
}

Word* cell_bits(const McWork& w, int64_t words) { return reinterpret_cast<Word*>(w.key[0]) + words; }

dwg_status read_count(const int32_t* count, int64_t* out, hipStream_t st) {
  int32_t c = 0;
  DWG_TRY_HIP(hipMemcpyAsync(&c, count, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  DWG_TRY_HIP(hipStreamSynchronize(st));
  *out = c;
  return DWG_OK;
}
}  // namespace

dwg_status mc_cells(const float* P, int64_t n, const McParams& mp, const McWork& w, int64_t* C_host,
                    hipStream_t st) {
  DWG_PROPAGATE_INT(morton_frame(P, n, w.bpart, w.box, w.frame, st));
  if (const int64_t words = bitmap_words(mp.depth, 2, mc_key_cap(n, mp))) {
    Word* const occ = reinterpret_cast<Word*>(w.key[0]);
    Word* const bits = cell_bits(w, words);
    hipLaunchKernelGGL(k_zero_u64, dim3(grid_of(words)), dim3(256), 0, st, occ, words);
    DWG_TRY_LAUNCH();
    hipLaunchKernelGGL(k_bits_occupied, dim3(grid_of(n)), dim3(256), 0, st, P, n, w.frame, mp.depth, occ);
    DWG_TRY_LAUNCH();
    hipLaunchKernelGGL(k_bits_grow, dim3(grid_of(words)), dim3(256), 0, st, occ, words, mp.depth, mp.dilate, bits,
                       w.head);
    DWG_TRY_LAUNCH();
    DWG_PROPAGATE_INT(exclusive_scan(w.head, words, w.hdsums, st));
    hipLaunchKernelGGL(k_bits_list, dim3(grid_of(words)), dim3(256), 0, st, bits, words, w.head, w.cells);
    DWG_TRY_LAUNCH();
    return read_count(w.head + words, C_host, st);
  }
  hipLaunchKernelGGL(k_mc_point_keys, dim3(grid_of(n)), dim3(256), 0, st, P, n, w.frame, mp.depth, w.key[0]);
  DWG_TRY_LAUNCH();
  int res = 0;
  DWG_PROPAGATE_INT(radix_sort_keys(w.key, n, 3 * mp.depth, w.work, &res, st));
  const uint64_t limit = 1ull << (3 * mp.depth);
  hipLaunchKernelGGL(k_mc_heads, dim3(grid_of(n)), dim3(256), 0, st, w.key[res], n, limit, w.head);
  DWG_TRY_LAUNCH();
  DWG_PROPAGATE_INT(exclusive_scan(w.head, n, w.hdsums, st));
  hipLaunchKernelGGL(k_mc_compact, dim3(grid_of(n)), dim3(256), 0, st, w.key[res], n, limit, w.head, w.occ);
  DWG_TRY_LAUNCH();
  // grow by `dilate` rings: (2 dilate + 1)^3 candidates per occupied cell, sentinel-padded
  const int64_t nk = mc_key_cap(n, mp);
  hipLaunchKernelGGL(k_mc_dilate, dim3(grid_of(nk)), dim3(256), 0, st, w.occ, w.head + n, n, mp.depth, mp.dilate,
                     w.key[0]);
  DWG_TRY_LAUNCH();
  DWG_PROPAGATE_INT(radix_sort_keys(w.key, nk, 3 * mp.depth + 1, w.work, &res, st));
  hipLaunchKernelGGL(k_mc_heads, dim3(grid_of(nk)), dim3(256), 0, st, w.key[res], nk, limit, w.head);
  DWG_TRY_LAUNCH();
  DWG_PROPAGATE_INT(exclusive_scan(w.head, nk, w.hdsums, st));
  hipLaunchKernelGGL(k_mc_compact, dim3(grid_of(nk)), dim3(256), 0, st, w.key[res], nk, limit, w.head, w.cells);
  DWG_TRY_LAUNCH();
  return read_count(w.head + nk, C_host, st);
}

dwg_status mc_corners(const McParams& mp, McWork& w, int64_t* m_host, hipStream_t st) {
  const int64_t n8 = 8 * w.C;
  const int64_t cell_words = bitmap_words(mp.depth, 2, mc_key_cap(w.n, mp));
  const int64_t words = cell_words ? bitmap_words(mp.depth + 1, 1, n8) : 0;
  if (words) {  // from the bitmap that mc_cells left
    Word* const bits = reinterpret_cast<Word*>(w.ckey[0]);
    hipLaunchKernelGGL(k_bits_corners, dim3(grid_of(words)), dim3(256), 0, st, cell_bits(w, cell_words), mp.depth, words,
                       bits, w.chead);
    DWG_TRY_LAUNCH();
    DWG_PROPAGATE_INT(exclusive_scan(w.chead, words, w.chdsums, st));
    DWG_PROPAGATE_INT(read_count(w.chead + words, m_host, st));
    w.m = *m_host;
    w.ld = w.m + (mp.iso_points ? w.n : 0);
    hipLaunchKernelGGL(k_bits_corner_ids, dim3(grid_of(std::max(n8, words))), dim3(256), 0, st, w.cells, w.C, bits,
                       words, w.chead, w.frame, w.box, mp.depth, w.cidx, w.pos, w.ld);
    DWG_TRY_LAUNCH();
    return DWG_OK;
  }
  hipLaunchKernelGGL(k_mc_corner_keys, dim3(grid_of(n8)), dim3(256), 0, st, w.cells, w.C, w.ckey[0]);
  DWG_TRY_LAUNCH();
  int res = 0;
  DWG_PROPAGATE_INT(radix_sort_pairs(w.ckey, w.cval, true, n8, 3 * (mp.depth + 1), w.cwork, &res, st));
  hipLaunchKernelGGL(k_mc_heads, dim3(grid_of(n8)), dim3(256), 0, st, w.ckey[res], n8, ~0ull, w.chead);
  DWG_TRY_LAUNCH();
  DWG_PROPAGATE_INT(exclusive_scan(w.chead, n8, w.chdsums, st));
  DWG_PROPAGATE_INT(read_count(w.chead + n8, m_host, st));
  w.m = *m_host;
  w.ld = w.m + (mp.iso_points ? w.n : 0);
  hipLaunchKernelGGL(k_mc_corner_ids, dim3(grid_of(n8)), dim3(256), 0, st, w.ckey[res], w.cval[res], n8, w.chead,
                     w.frame, w.box, mp.depth, w.cidx, w.pos, w.ld);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mc_faces(const McWork& w, float* tri, int64_t tcap, int64_t* F_host, hipStream_t st) {
  if (w.tets)
    hipLaunchKernelGGL(k_mt_count, dim3(grid_of(w.C)), dim3(256), 0, st, w.C, w.cidx, w.pos, w.ld, w.wc, w.iso,
                       w.fcnt);
  else
    hipLaunchKernelGGL(k_mc_count, dim3(grid_of(w.C)), dim3(256), 0, st, w.C, w.cidx, w.wc, w.iso, w.fcnt);
  DWG_TRY_LAUNCH();
  DWG_PROPAGATE_INT(exclusive_scan(w.fcnt, w.C, w.fsums, st));
  if (w.tets)
    hipLaunchKernelGGL(k_mt_emit, dim3(grid_of(w.C)), dim3(256), 0, st, w.C, w.cidx, w.pos, w.ld, w.wc, w.iso,
                       w.fcnt, w.fcap, w.cen, w.fcap, w.vec, tri, tcap);
  else
    hipLaunchKernelGGL(k_mc_emit, dim3(grid_of(w.C)), dim3(256), 0, st, w.C, w.cidx, w.pos, w.ld, w.wc, w.iso,
                       w.fcnt, w.fcap, w.cen, w.fcap, w.vec, tri, tcap);
  DWG_TRY_LAUNCH();
  return read_count(w.fcnt + w.C, F_host, st);
}

dwg_status mc_scatter(const McParams& mp, const McWork& w, int64_t F, hipStream_t st) {
  for (int64_t q0 = 0; q0 < F; q0 += w.chunk) {
    const int64_t m = std::min<int64_t>(w.chunk, F - q0);
    DWG_PROPAGATE_INT(knn_search(w.cen, w.fcap, q0, m, w.knn, mp.k, w.idx, w.dist, st));
    hipLaunchKernelGGL(k_mc_scatter, dim3(grid_of(3 * m * mp.k)), dim3(256), 0, st, w.idx, m, mp.k, w.vec + q0, w.frame,
                       mp.depth, w.n, w.acc);
    DWG_TRY_LAUNCH();
  }
  return DWG_OK;
}

dwg_status mc_append_points(const float* P, int64_t n, const McWork& w, hipStream_t st) {
  hipLaunchKernelGGL(k_mc_append_points, dim3(grid_of(n)), dim3(256), 0, st, P, n, w.pos, w.ld, w.m);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mc_point_iso(const McWork& w, const float* w_points, int64_t n, hipStream_t st) {
  constexpr int kParts = 256;
  hipLaunchKernelGGL(k_mc_mean_part, dim3(kParts), dim3(256), 0, st, w_points, n, w.ipart);
  DWG_TRY_LAUNCH();
  hipLaunchKernelGGL(k_mc_mean_final, dim3(1), dim3(256), 0, st, w.ipart, kParts, n, w.iso);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mc_clear(const McWork& w, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(grid_of(3 * w.n)), dim3(256), 0, st, w.acc, 3 * w.n);
  DWG_TRY_LAUNCH();
  return DWG_OK;
}

dwg_status mc_update(const McParams& mp, const McWork& w, const GwnWork& g, float* N, int* nblk, hipStream_t st) {
  const int nb = (int)cdiv(w.n, 256);
  hipLaunchKernelGGL(k_mc_update, dim3(nb), dim3(256), 0, st, g.perm_s, w.n, w.acc, w.frame, mp.depth, g.kk, N,
                     g.src, g.theta, g.blk, nb, g.hist);
  DWG_TRY_LAUNCH();
  *nblk = nb;
  return DWG_OK;
}

}  // namespace dwg
