// chamfer.hip -- Chamfer distance between two point sets on gfx950 (phi-SfT's
// evaluation metric, Sec. 4.2, Eq. 10):
//   Ch(G, M) = 1/|G| sum_g min_m |g - m|^2 + 1/|M| sum_m min_g |m - g|^2.
//
// Small sets: both nearest-neighbour searches run in one launch of k_chamfer_nn. A workgroup takes
// a block of 1024 query points (four per lane, coordinates in registers) and a tile of
// at most kChTile database points staged in LDS as three coordinate arrays (every lane reads the
// same point: an LDS broadcast), and keeps each query's smallest squared distance and
// its index; the tiles of one query block go to different workgroups, which merge their
// results with a 64-bit atomic minimum on (distance bits << 32 | index). Non-negative
// floats order like their bit patterns, so the merged value is the smallest distance
// and, among equal distances, the smallest index: the result does not depend on the
// order in which workgroups finish. Differences are formed coordinate by coordinate in
// FP32 (no |g|^2 + |m|^2 - 2 g.m expansion, whose cancellation would swamp the nearest
// distances), the means are accumulated in FP64 in a fixed order.
//
// Large sets: all pairs are bound by the vector ALUs (65536 against 40000 points: 800 us;
// sorted 126 us), and nearly all of them are far apart. Both sets are sorted into the cells of a 32^3 grid
// in Morton order (one counting sort), every 64 consecutive points get their bounding box,
// and a workgroup of four wavefronts searches for 64 sorted queries: it visits only the
// blocks whose box is no further from a query than the best point found so far. The
// bounds are formed with the operations of the distance itself, each of which rounds
// monotonically, so a skipped point's distance is larger as computed; equal distances are
// decided by the index. So both ways give the same bits, also for infinities and NaN
// (which no bound excludes and no comparison selects). The sort's order within a cell
// varies from run to run; the results do not depend on it.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "../../include/phisft_sim.h"

namespace phisft {

constexpr int kChThreads = 256;
constexpr int kChQ = 4;                          // query points per lane
constexpr int kChBlockQ = kChThreads * kChQ;     // query points per workgroup
constexpr int kChTile = 2048;                    // database points per workgroup (LDS) at most
constexpr int kChTileMin = 64;                   // and at least: 5000 by 289 points in tiles
                                                 // of 2048 kept 8 CUs busy, 196 us; now 19
constexpr int kChGrid = 1024;                    // workgroups that fill the chip

struct ChamferPass {
  const float* q;        // [3][nq] query points
  const float* db;       // [3][nd] database points
  int nq, nd;
  int qblocks;           // query blocks of this pass
  unsigned long long* best;   // [nq] packed minimum (distance bits << 32 | index)
};

// (infinity, index 0): what a search that selects nothing ends with
constexpr unsigned long long kChNone = 0x7f80000000000000ull;

__global__ void __launch_bounds__(kChThreads) k_chamfer_init(unsigned long long* best, long n,
                                                             int* bad) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) best[k] = kChNone;
  if (k == 0) *bad = 0;
}

// Sum over the 64 lanes of a wavefront, the same in every lane (each step adds the
// same two values in either order).
__device__ __forceinline__ double wave_sum64(double v) {
  for (int o = 32; o > 0; o >>= 1) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __shfl_xor(t.x, o);
    t.y = __shfl_xor(t.y, o);
    v += *reinterpret_cast<double*>(&t);
  }
  return v;
}

// Squared length, the operations and their order fixed: the sorted search compares bounds
// formed with it against distances formed with it.
__device__ __forceinline__ float dist2(float dx, float dy, float dz) {
  return fmaf(dz, dz, fmaf(dx, dx, dy * dy));
}

// Workgroups [0, nb0) serve pass 0 (queries G, database M), the rest pass 1 (M into G):
// block b of a pass covers query block b % qblocks and database tile b / qblocks.
__global__ void __launch_bounds__(kChThreads) k_chamfer_nn(ChamferPass p0, ChamferPass p1,
                                                           int nb0, int ntile, int* bad) {
  __shared__ float sx[kChTile], sy[kChTile], sz[kChTile];
  const bool second = (int)blockIdx.x >= nb0;
  const ChamferPass& p = second ? p1 : p0;
  const int b = second ? (int)blockIdx.x - nb0 : (int)blockIdx.x;
  const int qb = b % p.qblocks, tile = b / p.qblocks;
  const int d0 = tile * ntile, nloc = min(ntile, p.nd - d0);
  const int tid = threadIdx.x;
  for (int j = tid; j < nloc; j += kChThreads) {
    sx[j] = p.db[d0 + j];
    sy[j] = p.db[p.nd + d0 + j];
    sz[j] = p.db[2 * p.nd + d0 + j];
  }
  float qx[kChQ], qy[kChQ], qz[kChQ], bd[kChQ];
  int bi[kChQ];
#pragma unroll
  for (int k = 0; k < kChQ; ++k) {
    // lanes past the last query search with a copy of it and store nothing
    const int i = min(qb * kChBlockQ + k * kChThreads + tid, p.nq - 1);
    qx[k] = p.q[i];
    qy[k] = p.q[p.nq + i];
    qz[k] = p.q[2 * p.nq + i];
    bd[k] = INFINITY;
    bi[k] = 0;
  }
  // every point is a query of exactly one block of its pass (tile 0 checks it)
  if (tile == 0) {
    bool fin = true;
#pragma unroll
    for (int k = 0; k < kChQ; ++k) fin = fin && isfinite(qx[k]) && isfinite(qy[k]) && isfinite(qz[k]);
    if (!fin) atomicOr(bad, 1);
  }
  __syncthreads();
  for (int j = 0; j < nloc; ++j) {
    const float x = sx[j], y = sy[j], z = sz[j];
#pragma unroll
    for (int k = 0; k < kChQ; ++k) {
      const float d = dist2(qx[k] - x, qy[k] - y, qz[k] - z);
      if (d < bd[k]) {   // strictly smaller: the first index among equal distances stays
        bd[k] = d;
        bi[k] = j;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kChQ; ++k) {
    const int i = qb * kChBlockQ + k * kChThreads + tid;
    if (i < p.nq && nloc > 0) {
      const unsigned long long v =
          ((unsigned long long)__float_as_uint(bd[k]) << 32) | (unsigned)(d0 + bi[k]);
      atomicMin(p.best + i, v);
    }
  }
}

// Unpacks the minima of both sets (distance and index, either output optional) and sums
// the distances per workgroup in FP64 (fixed order: a butterfly per wavefront, then the
// wavefronts in order).
struct ChamferOut {
  const unsigned long long* best;
  int n;
  float* d;
  int* idx;
  double* part;
};

__global__ void __launch_bounds__(kChThreads) k_chamfer_unpack(ChamferOut og, ChamferOut om,
                                                               int nbg) {
  __shared__ double s_w[kChThreads / 64];
  const bool second = (int)blockIdx.x >= nbg;
  const ChamferOut& o = second ? om : og;
  const unsigned long long* best = o.best;
  const int n = o.n, blk = second ? (int)blockIdx.x - nbg : (int)blockIdx.x;
  float* d = o.d;
  int* idx = o.idx;
  double* part = o.part;
  const int i = blk * kChThreads + threadIdx.x;
  double v = 0.0;
  if (i < n) {
    const unsigned long long w = best[i];
    const float dist = __uint_as_float((unsigned)(w >> 32));
    if (d) d[i] = dist;
    if (idx) idx[i] = (int)(unsigned)(w & 0xffffffffu);
    v = dist;
  }
  v = wave_sum64(v);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kChThreads / 64; ++w) t += s_w[w];
    part[blk] = t;
  }
}

// Ch = (sum of G's partials) / |G| + (sum of M's partials) / |M|, one workgroup, fixed
// order; NaN when an input coordinate was not finite.
__global__ void __launch_bounds__(kChThreads) k_chamfer_sum(const double* pg, int nbg, int ng,
                                                            const double* pm, int nbm, int nm,
                                                            const int* bad, double* ch) {
  __shared__ double s_w[2][kChThreads / 64];
  double a = 0.0, c = 0.0;
  for (int k = threadIdx.x; k < nbg; k += kChThreads) a += pg[k];
  for (int k = threadIdx.x; k < nbm; k += kChThreads) c += pm[k];
  a = wave_sum64(a);
  c = wave_sum64(c);
  if ((threadIdx.x & 63) == 0) {
    s_w[0][threadIdx.x >> 6] = a;
    s_w[1][threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sa = 0.0, sc = 0.0;
    for (int w = 0; w < kChThreads / 64; ++w) {
      sa += s_w[0][w];
      sc += s_w[1][w];
    }
    *ch = *bad ? NAN : sa / ng + sc / nm;
  }
}

// ------------------------------------------------- large sets: sorted, pruned search
constexpr int kChCells = 32 * 32 * 32;
constexpr int kChPts = 64;      // points of a block
// Workgroups of the search (65536 by 40000 points: 132 us without splitting, 89 with) and
// the largest split.
constexpr int kChNearGrid = 2048, kChSplit = 16;

struct ChamferSet {
  const float* p;      // [3][n]
  int n, nblk;
  int* head;           // [kChCells] counts, then first places
  int2* where;         // [n] cell and place within it
  float4* sorted;      // [n] coordinates and original index (bits)
  float* box;          // [6][nblk] lowest, highest coordinates
  unsigned long long* best;
  int split;           // workgroups that share a block of queries
};

struct ChamferGrid {
  unsigned* lim;       // [6] keys of the highest -x, -y, -z, x, y, z; zero before
  int* bad;
};

// Order-preserving map of floats to unsigned (NaN apart); zero is below every float.
__device__ __forceinline__ unsigned float_key(float v) {
  const unsigned u = __float_as_uint(v);
  return u & 0x80000000u ? ~u : u | 0x80000000u;
}
__device__ __forceinline__ float key_float(unsigned k) {
  return __uint_as_float(k & 0x80000000u ? k & 0x7fffffffu : ~k);
}

__global__ void __launch_bounds__(256) k_chamfer_clear(ChamferSet a, ChamferSet b, ChamferGrid g) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < kChCells) {
    a.head[k] = 0;
    b.head[k] = 0;
  }
  if (k < 6) g.lim[k] = 0;
  if (k == 6) *g.bad = 0;
  for (int i = k; i < a.n; i += gridDim.x * 256) a.best[i] = kChNone;
  for (int i = k; i < b.n; i += gridDim.x * 256) b.best[i] = kChNone;
}

// Common bounding box of the finite coordinates of both sets.
__global__ void __launch_bounds__(256) k_chamfer_bounds(ChamferSet a, ChamferSet b, ChamferGrid g) {
  const int lane = threadIdx.x & 63;
  float hi[6];
  for (int q = 0; q < 6; ++q) hi[q] = -INFINITY;
  bool fin = true;
  for (long k = (long)blockIdx.x * 256 + threadIdx.x; k < (long)a.n + b.n; k += gridDim.x * 256l) {
    const ChamferSet& s = k < a.n ? a : b;
    const int i = (int)(k < a.n ? k : k - a.n);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const float v = s.p[(size_t)r * s.n + i];
      if (!isfinite(v)) {
        fin = false;
        continue;
      }
      hi[r] = fmaxf(hi[r], -v);
      hi[3 + r] = fmaxf(hi[3 + r], v);
    }
  }
#pragma unroll
  for (int q = 0; q < 6; ++q)
    for (int o = 32; o > 0; o >>= 1) hi[q] = fmaxf(hi[q], __shfl_xor(hi[q], o));
  __shared__ float s_hi[4][6];
  if (lane == 0)
    for (int q = 0; q < 6; ++q) s_hi[threadIdx.x >> 6][q] = hi[q];
  if (!__all(fin) && lane == 0) atomicOr(g.bad, 1);
  __syncthreads();
  if (threadIdx.x < 6) {
    float v = s_hi[0][threadIdx.x];
    for (int w = 1; w < 4; ++w) v = fmaxf(v, s_hi[w][threadIdx.x]);
    atomicMax(g.lim + threadIdx.x, float_key(v));
  }
}

__device__ __forceinline__ int spread3(int v) {   // 5 bits, two zeros between
  v = (v | v << 8) & 0x100f;
  v = (v | v << 4) & 0x10c3;
  return (v | v << 2) & 0x1249;
}

// A point's cell; any cell is right, near ones together are fast.
__device__ __forceinline__ int cell_of(const float* lo, float scale, float x, float y, float z) {
  const float c[3] = {x, y, z};
  int r = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    r |= spread3((int)fminf(fmaxf((c[k] - lo[k]) * scale, 0.0f), 31.0f)) << k;
  return r;
}

__global__ void __launch_bounds__(256) k_chamfer_count(ChamferSet a, ChamferSet b, ChamferGrid g) {
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k >= (long)a.n + b.n) return;
  const ChamferSet& s = k < a.n ? a : b;
  const int i = (int)(k < a.n ? k : k - a.n);
  float lo[3], ext = 0.0f;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    lo[r] = -key_float(g.lim[r]);
    ext = fmaxf(ext, key_float(g.lim[3 + r]) - lo[r]);
  }
  const float scale = ext > 0.0f ? 32.0f / ext : 0.0f;
  const int c = cell_of(lo, scale, s.p[i], s.p[(size_t)s.n + i], s.p[2 * (size_t)s.n + i]);
  s.where[i] = make_int2(c, atomicAdd(s.head + c, 1));
}

// Counts to first places, one workgroup per set.
__global__ void __launch_bounds__(1024) k_chamfer_scan(ChamferSet a, ChamferSet b) {
  __shared__ int s_w[16];
  int* head = blockIdx.x == 0 ? a.head : b.head;
  constexpr int per = kChCells / 1024;
  const int tid = threadIdx.x, lane = tid & 63;
  int4 v[per / 4];
  int sum = 0;
#pragma unroll
  for (int q = 0; q < per / 4; ++q) {
    v[q] = reinterpret_cast<const int4*>(head + per * tid)[q];
    sum += v[q].x + v[q].y + v[q].z + v[q].w;
  }
  int up = sum;   // inclusive over the wavefront
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(up, o);
    if (lane >= o) up += t;
  }
  if (lane == 63) s_w[tid >> 6] = up;
  __syncthreads();
  int at = up - sum;
  for (int w = 0; w < tid >> 6; ++w) at += s_w[w];
#pragma unroll
  for (int q = 0; q < per / 4; ++q) {
    int4 o;
    o.x = at;
    o.y = o.x + v[q].x;
    o.z = o.y + v[q].y;
    o.w = o.z + v[q].z;
    at = o.w + v[q].w;
    reinterpret_cast<int4*>(head + per * tid)[q] = o;
  }
}

__global__ void __launch_bounds__(256) k_chamfer_scatter(ChamferSet a, ChamferSet b) {
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k >= (long)a.n + b.n) return;
  const ChamferSet& s = k < a.n ? a : b;
  const int i = (int)(k < a.n ? k : k - a.n);
  const int2 w = s.where[i];
  s.sorted[s.head[w.x] + w.y] =
      make_float4(s.p[i], s.p[(size_t)s.n + i], s.p[2 * (size_t)s.n + i], __int_as_float(i));
}

// Bounding boxes of the blocks, one wavefront each (NaN coordinates are left out: such a
// point is never selected).
__global__ void __launch_bounds__(256) k_chamfer_boxes(ChamferSet a, ChamferSet b) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= a.nblk + b.nblk) return;
  const ChamferSet& s = w < a.nblk ? a : b;
  const int k = w < a.nblk ? w : w - a.nblk;
  const float4 p = s.sorted[min(k * kChPts + lane, s.n - 1)];
  float lo[3] = {p.x, p.y, p.z}, hi[3] = {p.x, p.y, p.z};
#pragma unroll
  for (int r = 0; r < 3; ++r)
    for (int o = 32; o > 0; o >>= 1) {
      lo[r] = fminf(lo[r], __shfl_xor(lo[r], o));
      hi[r] = fmaxf(hi[r], __shfl_xor(hi[r], o));
    }
  if (lane == 0)
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      s.box[r * s.nblk + k] = lo[r];
      s.box[(3 + r) * s.nblk + k] = hi[r];
    }
}

// Distance of the intervals [a0, a1] and [b0, b1] (0 when they meet).
__device__ __forceinline__ float gap(float a0, float a1, float b0, float b1) {
  return fmaxf(fmaxf(b0 - a1, a0 - b1), 0.0f);
}

__device__ __forceinline__ float lane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Nearest points of 64 sorted queries, the other set's blocks dealt in turn to the four
// wavefronts of a workgroup (of `split` workgroups, where the queries' blocks alone are too
// few to fill the chip). Each wavefront first visits the nearest of its blocks, which bounds the
// rest; the best points of all four meet in LDS after every block. Distances and indices
// are compared as one 64-bit number (distances are not negative, and NaN is above
// infinity). A block's points travel while the one before is searched.
__global__ void __launch_bounds__(256) k_chamfer_near(ChamferSet a, ChamferSet b) {
  __shared__ unsigned long long s_best[kChPts];
  __shared__ float4 s_pts[4][kChPts];
  const bool second = (int)blockIdx.x >= a.nblk * a.split;
  const ChamferSet& Q = second ? b : a;
  const ChamferSet& D = second ? a : b;
  const int part = second ? (int)blockIdx.x - a.nblk * a.split : (int)blockIdx.x;
  const int blk = part % Q.nblk, waves = 4 * Q.split;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nb = D.nblk, nd = D.n;
  const int turn = part / Q.nblk * 4 + wave;   // of this wavefront among all of the block
  const float4* sorted = D.sorted;
  const int qi = blk * kChPts + lane;
  const float4 q = Q.sorted[min(qi, Q.n - 1)];
  float qb[6];
#pragma unroll
  for (int r = 0; r < 6; ++r) qb[r] = Q.box[r * Q.nblk + blk];
  if (wave == 0) s_best[lane] = kChNone;
  __syncthreads();
  float4* pts = s_pts[wave];
  unsigned long long best = kChNone;
  float x[6];   // box of this lane's block of a chunk
  // loads it and gives its distance from the queries' box; infinity past the last
  auto bound = [&](int k) {
#pragma unroll
    for (int r = 0; r < 6; ++r) x[r] = D.box[r * nb + min(k, nb - 1)];
    const float d = dist2(gap(qb[0], qb[3], x[0], x[3]), gap(qb[1], qb[4], x[1], x[4]),
                          gap(qb[2], qb[5], x[2], x[5]));
    return k < nb ? d : INFINITY;
  };
  auto points = [&](int k) { return sorted[min(k * kChPts + lane, nd - 1)]; };
  auto visit = [&](const float4& p) {   // a copy of the set's last point may stand in
    pts[lane] = p;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll 8
    for (int j = 0; j < kChPts; ++j) {
      const float4 t = pts[j];
      const float d = dist2(q.x - t.x, q.y - t.y, q.z - t.z);
      const unsigned long long v =
          (unsigned long long)__float_as_uint(d) << 32 | __float_as_uint(t.w);
      best = v < best ? v : best;
    }
    __builtin_amdgcn_wave_barrier();
    atomicMin(&s_best[lane], best);
    best = min(best, *(volatile unsigned long long*)&s_best[lane]);
  };
  auto reach = [&] { return __uint_as_float((unsigned)(best >> 32)); };
  // the nearest of this wavefront's blocks
  float near = INFINITY;
  int first = -1;
  for (int k = turn + waves * lane; k < nb; k += waves * 64) {
    const float d = bound(k);
    if (first < 0 || d < near) {
      near = d;
      first = k;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float d = __shfl_xor(near, o);
    const int k = __shfl_xor(first, o);
    if (k >= 0 && (first < 0 || d < near || (d == near && k < first))) {
      near = d;
      first = k;
    }
  }
  first = __builtin_amdgcn_readfirstlane(first);
  if (first >= 0) visit(points(first));
  __syncthreads();
  best = min(best, s_best[lane]);
  float4 held;
  bool holds = false;
  for (int c = turn; c < nb; c += waves * 64) {
    const int k = c + waves * lane;
    const float d = bound(k);
    float far = reach();   // the worst of the queries' best
    for (int o = 32; o > 0; o >>= 1) far = fmaxf(far, __shfl_xor(far, o));
    unsigned long long todo = __ballot(k < nb && k != first && !(d > far));
    while (todo) {
      const int l = __builtin_ctzll(todo);
      todo &= todo - 1;
      // is the box within reach of any single query?
      float e[3];
      const float qc[3] = {q.x, q.y, q.z};
#pragma unroll
      for (int r = 0; r < 3; ++r) e[r] = gap(qc[r], qc[r], lane_f(x[r], l), lane_f(x[3 + r], l));
      if (__ballot(!(dist2(e[0], e[1], e[2]) > reach())) == 0) continue;
      const float4 p = points(c + waves * l);
      if (holds) visit(held);
      held = p;
      holds = true;
    }
  }
  if (holds) visit(held);
  __syncthreads();
  if (wave == 0 && qi < Q.n) {
    if (Q.split == 1) Q.best[__float_as_int(q.w)] = s_best[lane];
    else atomicMin(Q.best + __float_as_int(q.w), s_best[lane]);
  }
}

static inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

struct ChamferLayout {
  size_t best_g, best_m, part_g, part_m, bad, total;
  int nbg, nbm;
};

static ChamferLayout chamfer_layout(int ng, int nm) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  ChamferLayout L{};
  L.nbg = cdiv(ng, kChThreads);
  L.nbm = cdiv(nm, kChThreads);
  L.best_g = 0;
  L.best_m = up(8 * (size_t)ng);
  L.part_g = L.best_m + up(8 * (size_t)nm);
  L.part_m = L.part_g + up(8 * (size_t)L.nbg);
  L.bad = L.part_m + up(8 * (size_t)L.nbm);
  L.total = L.bad + 256;
  return L;
}

// What the sorted search needs besides; ends at its total.
struct ChamferSorted {
  size_t lim, head[2], where[2], sorted[2], box[2], total;
  int nblk[2];
};

static ChamferSorted chamfer_sorted(const ChamferLayout& L, int ng, int nm) {
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  ChamferSorted S{};
  size_t at = L.total;
  S.lim = at;
  at += 256;
  for (int k = 0; k < 2; ++k) {
    const size_t n = k == 0 ? ng : nm;
    S.nblk[k] = cdiv((long)n, kChPts);
    S.head[k] = at;
    at += 4 * (size_t)kChCells;
    S.where[k] = at;
    at += up(8 * n);
    S.sorted[k] = at;
    at += up(16 * n);
    S.box[k] = at;
    at += up(24 * (size_t)S.nblk[k]);
  }
  S.total = at;
  return S;
}

// Pairs from which on the sorted search is the faster one (sorted against all pairs, us:
// 1.0e8 pairs 60, 50; 65536 by 1600 75, 55; 60000 by 4000 82, 99; 2.6e8 65, 109; 9e8 87, 325;
// 65536 by 40000 139, 878).
constexpr double kChSortedPairs = 1.8e8;

static bool chamfer_wants_sorted(int ng, int nm) {
  return (double)ng * (double)nm >= kChSortedPairs;
}

}  // namespace phisft

using namespace phisft;

extern "C" {

size_t sim_chamfer_workspace_bytes(int32_t n_g, int32_t n_m) {
  if (n_g < 1 || n_m < 1) return 0;
  const ChamferLayout L = chamfer_layout(n_g, n_m);
  return chamfer_wants_sorted(n_g, n_m) ? chamfer_sorted(L, n_g, n_m).total : L.total;
}

sim_status sim_chamfer(const float* g, int32_t n_g, const float* m, int32_t n_m, double* ch,
                       float* d_g, int32_t* i_g, float* d_m, int32_t* i_m, void* workspace,
                       size_t workspace_bytes, void* stream) {
  if (!g || !m || !ch || !workspace || n_g < 1 || n_m < 1) return SIM_E_INVALID;
  const ChamferLayout L = chamfer_layout(n_g, n_m);
  if (workspace_bytes < L.total) return SIM_E_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* w = static_cast<char*>(workspace);
  auto* bg = reinterpret_cast<unsigned long long*>(w + L.best_g);
  auto* bm = reinterpret_cast<unsigned long long*>(w + L.best_m);
  auto* pg = reinterpret_cast<double*>(w + L.part_g);
  auto* pm = reinterpret_cast<double*>(w + L.part_m);
  int* bad = reinterpret_cast<int*>(w + L.bad);
  const ChamferSorted S = chamfer_sorted(L, n_g, n_m);
  if (chamfer_wants_sorted(n_g, n_m) && workspace_bytes >= S.total) {
    ChamferSet set[2];
    for (int k = 0; k < 2; ++k) {
      ChamferSet& t = set[k];
      t.p = k == 0 ? g : m;
      t.n = k == 0 ? n_g : n_m;
      t.nblk = S.nblk[k];
      t.head = reinterpret_cast<int*>(w + S.head[k]);
      t.where = reinterpret_cast<int2*>(w + S.where[k]);
      t.sorted = reinterpret_cast<float4*>(w + S.sorted[k]);
      t.box = reinterpret_cast<float*>(w + S.box[k]);
      t.best = k == 0 ? bg : bm;
      t.split = std::min(kChSplit, std::max(1, kChNearGrid / t.nblk));
    }
    const ChamferGrid gr{reinterpret_cast<unsigned*>(w + S.lim), bad};
    const ChamferSet &a = set[0], &b = set[1];
    const dim3 th(256), pts(cdiv((long)n_g + n_m, 256));
    hipLaunchKernelGGL(k_chamfer_clear, dim3(kChCells / 256), th, 0, st, a, b, gr);
    hipLaunchKernelGGL(k_chamfer_bounds, dim3(pts.x < 256 ? pts.x : 256), th, 0, st, a, b, gr);
    hipLaunchKernelGGL(k_chamfer_count, pts, th, 0, st, a, b, gr);
    hipLaunchKernelGGL(k_chamfer_scan, dim3(2), dim3(1024), 0, st, a, b);
    hipLaunchKernelGGL(k_chamfer_scatter, pts, th, 0, st, a, b);
    hipLaunchKernelGGL(k_chamfer_boxes, dim3(cdiv((long)a.nblk + b.nblk, 4)), th, 0, st, a, b);
    hipLaunchKernelGGL(k_chamfer_near, dim3(a.nblk * a.split + b.nblk * b.split), th, 0,
                       st, a, b);
  } else {
    ChamferPass p0{g, m, n_g, n_m, cdiv(n_g, kChBlockQ), bg};
    ChamferPass p1{m, g, n_m, n_g, cdiv(n_m, kChBlockQ), bm};
    // smaller tiles until there are workgroups for every CU
    int tile = kChTile;
    long nb0, nb1;
    for (;; tile /= 2) {
      nb0 = (long)p0.qblocks * cdiv(n_m, tile);
      nb1 = (long)p1.qblocks * cdiv(n_g, tile);
      if (tile == kChTileMin || nb0 + nb1 >= kChGrid) break;
    }
    if (nb0 + nb1 > 0x7fffffffL) return SIM_E_INVALID;
    // the two packed-minimum arrays are contiguous up to alignment padding, which the
    // fill covers as well (it lies inside the workspace)
    const long nfill = (long)(L.part_g - L.best_g) / 8;
    hipLaunchKernelGGL(k_chamfer_init, dim3(cdiv(nfill, kChThreads)), dim3(kChThreads), 0, st, bg,
                       nfill, bad);
    hipLaunchKernelGGL(k_chamfer_nn, dim3((unsigned)(nb0 + nb1)), dim3(kChThreads), 0, st, p0, p1,
                       (int)nb0, tile, bad);
  }
  hipLaunchKernelGGL(k_chamfer_unpack, dim3(L.nbg + L.nbm), dim3(kChThreads), 0, st,
                     ChamferOut{bg, n_g, d_g, i_g, pg}, ChamferOut{bm, n_m, d_m, i_m, pm}, L.nbg);
  hipLaunchKernelGGL(k_chamfer_sum, dim3(1), dim3(kChThreads), 0, st, pg, L.nbg, n_g, pm, L.nbm,
                     n_m, bad, ch);
  return hipGetLastError() == hipSuccess ? SIM_OK : SIM_E_HIP;
}

}  // extern "C"
