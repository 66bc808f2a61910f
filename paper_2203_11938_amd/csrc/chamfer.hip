// chamfer.hip -- Chamfer distance between two point sets on gfx950 (phi-SfT's
// evaluation metric, Sec. 4.2, Eq. 10):
//   Ch(G, M) = 1/|G| sum_g min_m |g - m|^2 + 1/|M| sum_m min_g |m - g|^2.
//
// Small sets: both nearest-neighbour searches run in one launch of k_chamfer_nn. A workgroup
// takes a block of 1024 query points (four per lane, coordinates in registers) and a tile
// of at most kChTile database points staged in LDS as three coordinate arrays (every lane
// reads the same point: an LDS broadcast), and keeps each query's smallest squared distance and
// its index; the tiles of one query block go to different workgroups, which merge their
// results with a 64-bit atomic minimum on (distance bits << 32 | index). Non-negative
// floats order like their bit patterns, so the merged value is the smallest distance
// and, among equal distances, the smallest index: the result does not depend on the
// order in which workgroups finish. Differences are formed coordinate by coordinate in
// FP32 (no |g|^2 + |m|^2 - 2 g.m expansion, whose cancellation would swamp the nearest
// distances), the means are accumulated in FP64 in a fixed order.
//
// Large sets: all pairs are bound by the vector ALUs (65536 against 40000 points: 800 us;
// sorted 121 to 138 us over seeds, 130 on average), and nearly all of them are far apart.
// Each set is sorted into the cells of a 32^3 grid of its own in Morton order (one counting
// sort), every 64 consecutive points get their bounding box, and a workgroup of four
// wavefronts searches for 64 sorted queries: it visits only the blocks whose box is no
// further from a query than the best point found so far. The bounds are formed with the
// operations of the distance itself, each of which rounds monotonically, so a skipped
// point's distance is larger as computed; equal distances are decided by the index. So both
// ways give the same bits, also for infinities and NaN (whose distances no comparison
// selects). The sort's order within a cell varies from run to run; the results do not
// depend on it.

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
constexpr int kChTilePlain = 1024;               // at most, of sets not worth sorting
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

// All pairs. Blocks [0, nb0) serve pass 0 (queries G, database M), the rest pass 1 (M into G):
// block b of a pass covers query block b % qblocks and database tile b / qblocks.
struct ChamferPairs {
  ChamferPass p[2];
  long nb0, nb;
  int ntile;        // points of a tile, at most T
};

template <int T>
__device__ __forceinline__ void all_pairs(const ChamferPairs& c, float (*s)[T], int* bad) {
  const int tid = threadIdx.x;
  for (long blk = blockIdx.x; blk < c.nb; blk += gridDim.x) {
    const bool second = blk >= c.nb0;
    const ChamferPass& p = second ? c.p[1] : c.p[0];
    const long b = second ? blk - c.nb0 : blk;
    const int qb = (int)(b % p.qblocks), tile = (int)(b / p.qblocks);
    const int d0 = tile * c.ntile, nloc = min(c.ntile, p.nd - d0);
    for (int j = tid; j < nloc; j += kChThreads) {
      s[0][j] = p.db[d0 + j];
      s[1][j] = p.db[p.nd + d0 + j];
      s[2][j] = p.db[2 * p.nd + d0 + j];
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
      const float x = s[0][j], y = s[1][j], z = s[2][j];
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
    __syncthreads();   // the tile is read, the next one may come
  }
}

__global__ void __launch_bounds__(kChThreads) k_chamfer_nn(ChamferPairs c, int* bad) {
  __shared__ float s[3][kChTile];
  all_pairs<kChTile>(c, s, bad);
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

// Grid of a set: lowest corner and cells per length. plain: its points are so concentrated
// that sorting cannot tell them apart; all pairs are then looked at instead.
struct ChamferGrid {
  float lo[3], scale;
  int plain;
};

__device__ __forceinline__ bool use_all_pairs(const ChamferGrid* g) { return g[0].plain || g[1].plain; }

__device__ __forceinline__ int spread3(int v) {   // 5 bits, two zeros between
  v = (v | v << 8) & 0x100f;
  v = (v | v << 4) & 0x10c3;
  return (v | v << 2) & 0x1249;
}

// A point's cell; any cell is right, near ones together are fast.
__device__ __forceinline__ int cell_of(const ChamferGrid& g, float x, float y, float z) {
  const float c[3] = {x, y, z};
  int r = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    r |= spread3((int)fminf(fmaxf((c[k] - g.lo[k]) * g.scale, 0.0f), 31.0f)) << k;
  return r;
}

// Median of 64 values, one a lane of a wavefront (NaN last), the same in every lane: sorted
// by a bitonic network.
__device__ __forceinline__ float median64(float v, int lane) {
  v = v == v ? v : INFINITY;
#pragma unroll
  for (int size = 2; size <= 64; size *= 2)
#pragma unroll
    for (int o = size / 2; o > 0; o /= 2) {
      const float w = __shfl_xor(v, o);
      const bool low = ((lane & o) == 0) == ((lane & size) == 0);
      v = low ? fminf(v, w) : fmaxf(v, w);
    }
  return __shfl(v, 32);
}

// First launch: the last two workgroups find the sets' grids, the others clear. A grid
// spans the bulk of 1024 of the set's points: of every 16 the lowest and highest
// coordinates, and of those the medians (about the outer 4 % at each end, so a set may
// hold a few outliers, which end up in the outermost cells), widened by a thirty-second. With a
// grid over all points one outlier far away put the rest into one cell: 65536 against
// 40000 points took 2284 us, all pairs 825, this way 134. Cells of a sixteenth of the
// grid's length then count how often two of the points meet: surfaces about 1 time in 200,
// lines 1 in 16; from 1 in 6 on the set is searched plainly (half of it in one place: 1 in 4).
constexpr int kChSample = 1024;
__global__ void __launch_bounds__(kChSample) k_chamfer_start(ChamferSet a, ChamferSet b,
                                                             ChamferGrid* grid, int* bad) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nclear = gridDim.x - 2;
  if ((int)blockIdx.x < nclear) {
    const int k = blockIdx.x * kChSample + tid, stride = nclear * kChSample;
    for (int i = k; i < kChCells; i += stride) a.head[i] = b.head[i] = 0;
    for (long i = k; i < a.n; i += stride) a.best[i] = kChNone;
    for (long i = k; i < b.n; i += stride) b.best[i] = kChNone;
    if (k == 0) *bad = 0;
    return;
  }
  __shared__ float s_end[6][64];   // lowest and highest of every 16 points
  __shared__ float s_med[6];
  __shared__ int s_cell[16 * 16 * 16], s_met;
  const int which = blockIdx.x - nclear;
  const ChamferSet& s = which == 0 ? a : b;
  // golden-ratio steps: even strides would meet the same columns of an ordered grid
  const int i = (int)((unsigned long long)(tid * 2654435769u) * (unsigned)s.n >> 32);
  float c[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    c[r] = s.p[(size_t)r * s.n + i];
    float lo = c[r], hi = c[r];
    for (int o = 8; o > 0; o >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, o));
      hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if ((lane & 15) == 0) {
      s_end[r][tid >> 4] = lo;
      s_end[3 + r][tid >> 4] = hi;
    }
  }
  for (int k = tid; k < 16 * 16 * 16; k += kChSample) s_cell[k] = 0;
  if (tid == 0) s_met = 0;
  __syncthreads();
  if (wave < 6) {
    const float m = median64(s_end[wave][lane], lane);
    if (lane == 0) s_med[wave] = m;
  }
  __syncthreads();
  ChamferGrid g;
  float ext = 0.0f;
#pragma unroll
  for (int r = 0; r < 3; ++r) ext = fmaxf(ext, s_med[3 + r] - s_med[r]);
  const bool some = ext > 0.0f && isfinite(ext);
#pragma unroll
  for (int r = 0; r < 3; ++r) g.lo[r] = some ? s_med[r] - 0.03125f * ext : 0.0f;
  g.scale = some ? 32.0f / (1.0625f * ext) : 0.0f;
  // Morton order: the upper four bits of each coordinate are the upper twelve of the cell
  const int met = atomicAdd(&s_cell[cell_of(g, c[0], c[1], c[2]) >> 3], 1);
  int sum = met;
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == 0) atomicAdd(&s_met, sum);
  __syncthreads();
  if (tid == 0) {
    g.plain = s_met > kChSample * kChSample / 2 / 6;
    grid[which] = g;
  }
}

// Cells and places within them. Points of a wavefront that share a cell take their places
// together: with an atomic addition each, 65536 points in one cell took 0.7 ms.
__global__ void __launch_bounds__(256) k_chamfer_count(ChamferSet a, ChamferSet b,
                                                       const ChamferGrid* grid, int nba, int* bad) {
  if (use_all_pairs(grid)) return;
  const bool second = (int)blockIdx.x >= nba;
  const ChamferSet& s = second ? b : a;
  const int lane = threadIdx.x & 63;
  const long k = ((long)blockIdx.x - (second ? nba : 0)) * 256 + threadIdx.x;
  const bool live = k < s.n;
  const int i = (int)(live ? k : s.n - 1);
  const float x = s.p[i], y = s.p[(size_t)s.n + i], z = s.p[2 * (size_t)s.n + i];
  if (!__all(isfinite(x) && isfinite(y) && isfinite(z)) && lane == 0) atomicOr(bad, 1);
  const int c = cell_of(grid[second ? 1 : 0], x, y, z);
  int leader = lane, place = 0, count = 1;
  unsigned long long todo = __ballot(live);
  for (int turn = 0; turn < 8 && todo; ++turn) {   // the rest has cells of few points each
    const int l = __builtin_ctzll(todo);
    const unsigned long long same = __ballot(live && c == __builtin_amdgcn_readlane(c, l));
    if (live && same >> lane & 1) {
      leader = l;
      place = __popcll(same & ((1ull << lane) - 1));
      count = __popcll(same);
    }
    todo &= ~same;
  }
  int first = 0;
  if (live && lane == leader) first = atomicAdd(s.head + c, count);
  first = __shfl(first, leader);
  if (live) s.where[i] = make_int2(c, first + place);
}

// Counts to first places, one workgroup per set, in 8 chunks of 16 bytes a thread (with 128
// contiguous bytes a thread, whose loads touch 64 lines a wavefront, 9.7 us).
__global__ void __launch_bounds__(1024) k_chamfer_scan(ChamferSet a, ChamferSet b,
                                                       const ChamferGrid* grid) {
  if (use_all_pairs(grid)) return;
  constexpr int kChunks = kChCells / 4096;
  __shared__ int s_w[16 * kChunks];   // [chunk][wavefront]
  int4* head = reinterpret_cast<int4*>(blockIdx.x == 0 ? a.head : b.head);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int4 v[kChunks];
  int up[kChunks];   // inclusive over the wavefront
#pragma unroll
  for (int q = 0; q < kChunks; ++q) v[q] = head[1024 * q + tid];
#pragma unroll
  for (int q = 0; q < kChunks; ++q) {
    up[q] = v[q].x + v[q].y + v[q].z + v[q].w;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(up[q], o);
      if (lane >= o) up[q] += t;
    }
    if (lane == 63) s_w[16 * q + wave] = up[q];
  }
  __syncthreads();
  int before = 0;   // of this thread's entry of s_w
  if (tid < 16 * kChunks)
    for (int k = 0; k < tid; ++k) before += s_w[k];
  __syncthreads();
  if (tid < 16 * kChunks) s_w[tid] = before;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kChunks; ++q) {
    int4 o;
    o.x = s_w[16 * q + wave] + up[q] - (v[q].x + v[q].y + v[q].z + v[q].w);
    o.y = o.x + v[q].x;
    o.z = o.y + v[q].y;
    o.w = o.z + v[q].z;
    head[1024 * q + tid] = o;
  }
}

__global__ void __launch_bounds__(256) k_chamfer_scatter(ChamferSet a, ChamferSet b,
                                                         const ChamferGrid* grid) {
  if (use_all_pairs(grid)) return;
  const long k = (long)blockIdx.x * 256 + threadIdx.x;
  if (k >= (long)a.n + b.n) return;
  const ChamferSet& s = k < a.n ? a : b;
  const int i = (int)(k < a.n ? k : k - a.n);
  const int2 w = s.where[i];
  s.sorted[s.head[w.x] + w.y] =
      make_float4(s.p[i], s.p[(size_t)s.n + i], s.p[2 * (size_t)s.n + i], __int_as_float(i));
}

__device__ __forceinline__ bool finite3(const float4& p) {
  return isfinite(p.x) && isfinite(p.y) && isfinite(p.z);
}

// Bounding boxes of the blocks, one wavefront each. A point with a coordinate that is not finite
// is left out: its distance is NaN or infinite, and neither is ever selected.
__global__ void __launch_bounds__(256) k_chamfer_boxes(ChamferSet a, ChamferSet b,
                                                       const ChamferGrid* grid) {
  if (use_all_pairs(grid)) return;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= a.nblk + b.nblk) return;
  const ChamferSet& s = w < a.nblk ? a : b;
  const int k = w < a.nblk ? w : w - a.nblk;
  const float4 p = s.sorted[min(k * kChPts + lane, s.n - 1)];
  const bool fin = finite3(p);
  float lo[3] = {p.x, p.y, p.z}, hi[3] = {p.x, p.y, p.z};
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    if (!fin) {
      lo[r] = INFINITY;
      hi[r] = -INFINITY;
    }
    for (int o = 32; o > 0; o >>= 1) {
      lo[r] = fminf(lo[r], __shfl_xor(lo[r], o));
      hi[r] = fmaxf(hi[r], __shfl_xor(hi[r], o));
    }
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
// Sets that are not worth sorting are searched plainly in the same launch, their tiles in the
// same LDS (13505 by 13440 equal points: 84 us, with k_chamfer_nn alone 74).
__global__ void __launch_bounds__(256) k_chamfer_near(ChamferSet a, ChamferSet b, ChamferPairs pairs,
                                                      const ChamferGrid* grid, int* bad) {
  __shared__ __align__(16) float s_tile[3][kChTilePlain];
  if (use_all_pairs(grid)) {
    all_pairs<kChTilePlain>(pairs, s_tile, bad);
    return;
  }
  float4 (*s_pts)[kChPts] = reinterpret_cast<float4 (*)[kChPts]>(&s_tile[0][0]);   // [4]
  unsigned long long* s_best = reinterpret_cast<unsigned long long*>(s_pts + 4);   // [kChPts]
  static_assert(sizeof(s_tile) >= 4 * kChPts * sizeof(float4) + kChPts * 8, "both in one tile");
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
  // a query that is not finite finds nothing, and needs no block
  const bool fin = finite3(q);
  auto reach = [&] { return fin ? __uint_as_float((unsigned)(best >> 32)) : -1.0f; };
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

// Pairs from which on the sorted search is the faster one (sorted against all pairs, us, with
// the calls' gaps: 1.0e8 pairs 60, 50; 65536 by 1600 75, 55; 65536 by 2753 80, 83; 13505 by
// 13440 62, 83; 30000 by 30000 86, 333; 65536 by 40000 134, 900).
constexpr double kChSortedPairs = 1.8e8;

// The sort takes time with the points, so the smaller set must not be too small either (2
// million by 100: sorted 858, all pairs 474; 500000 by 1000 264, 190; 300000 by 2000 196, 241).
constexpr double kChSortedMean = 1400.0;

static bool chamfer_wants_sorted(int ng, int nm) {
  const double pairs = (double)ng * (double)nm;
  return pairs >= kChSortedPairs && pairs >= kChSortedMean * ((double)ng + (double)nm);
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
  ChamferPairs pairs{{{g, m, n_g, n_m, cdiv(n_g, kChBlockQ), bg}, {m, g, n_m, n_g, cdiv(n_m, kChBlockQ), bm}},
                     0, 0, 0};
  auto split = [&](int tile) {   // smaller tiles until there are workgroups for every CU
    for (;; tile /= 2) {
      pairs.ntile = tile;
      pairs.nb0 = (long)pairs.p[0].qblocks * cdiv(n_m, tile);
      pairs.nb = pairs.nb0 + (long)pairs.p[1].qblocks * cdiv(n_g, tile);
      if (tile == kChTileMin || pairs.nb >= kChGrid) break;
    }
  };
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
    const ChamferSet &a = set[0], &b = set[1];
    const dim3 th(256), pts(cdiv((long)n_g + n_m, 256));
    ChamferGrid* grid = reinterpret_cast<ChamferGrid*>(w + S.lim);
    split(kChTilePlain);
    const int nclear = std::min(std::max(pts.x / 16, 32u), 512u);
    hipLaunchKernelGGL(k_chamfer_start, dim3(nclear + 2), dim3(kChSample), 0, st, a, b, grid, bad);
    hipLaunchKernelGGL(k_chamfer_count, dim3(L.nbg + L.nbm), th, 0, st, a, b, grid, L.nbg, bad);
    hipLaunchKernelGGL(k_chamfer_scan, dim3(2), dim3(1024), 0, st, a, b, grid);
    hipLaunchKernelGGL(k_chamfer_scatter, pts, th, 0, st, a, b, grid);
    hipLaunchKernelGGL(k_chamfer_boxes, dim3(cdiv((long)a.nblk + b.nblk, 4)), th, 0, st, a, b, grid);
    hipLaunchKernelGGL(k_chamfer_near, dim3(a.nblk * a.split + b.nblk * b.split), th, 0,
                       st, a, b, pairs, grid, bad);
  } else {
    split(kChTile);
    if (pairs.nb > 0x7fffffffL) return SIM_E_INVALID;
    // the two packed-minimum arrays are contiguous up to alignment padding, which the
    // fill covers as well (it lies inside the workspace)
    const long nfill = (long)(L.part_g - L.best_g) / 8;
    hipLaunchKernelGGL(k_chamfer_init, dim3(cdiv(nfill, kChThreads)), dim3(kChThreads), 0, st, bg,
                       nfill, bad);
    hipLaunchKernelGGL(k_chamfer_nn, dim3((unsigned)pairs.nb), dim3(kChThreads), 0, st, pairs, bad);
  }
  hipLaunchKernelGGL(k_chamfer_unpack, dim3(L.nbg + L.nbm), dim3(kChThreads), 0, st,
                     ChamferOut{bg, n_g, d_g, i_g, pg}, ChamferOut{bm, n_m, d_m, i_m, pm}, L.nbg);
  hipLaunchKernelGGL(k_chamfer_sum, dim3(1), dim3(kChThreads), 0, st, pg, L.nbg, n_g, pm, L.nbm,
                     n_m, bad, ch);
  return hipGetLastError() == hipSuccess ? SIM_OK : SIM_E_HIP;
}

}  // extern "C"
