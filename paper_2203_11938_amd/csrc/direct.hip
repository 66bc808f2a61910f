// direct.hip -- direct solution of the step matrix A on gfx950: a multifrontal
// factorisation over the elimination plan of direct_prep.cpp and its two triangular
// passes, all in FP64, in one launch of k_ds_run.
//
// Work is cut into tasks of one front each. With F_pp and F_bp the front's pivot and
// border blocks (both from A plus the children's updates):
//   pivot     X = F_pp^-1              symmetric block sweep in registers
//   border    W = F_bp X               32 border rows
//   Schur     S = (children) - W F_bp^T    a 64x64 tile of the lower triangle
//   forward   t = b_p + (children), g = (children) - W t    64 border rows
//   backward  x_p = X t - W^T x_b      32 pivot unknowns, top down
// Keeping the inverse of every pivot block instead of its triangular factor is what lets
// both passes run as matrix-vector products without a serial substitution inside a front;
// pivot blocks are at most 96 wide, and a solve is accepted only on its true residual
// (k_ds_resid). A later solve with the same factor runs the forward and backward tasks
// alone.
//
// What bounds it: the chain of fronts from a leaf to the root (13 of a 64x64 sheet), each
// a pivot sweep and three hand-offs between workgroups, not the arithmetic (1.3 GFLOP).
// A forward and adjoint of 60 steps on that sheet took 140 ms with the iterative solver
// (100 to 300 iterations of 5 to 12 us a solve) and take 45 ms with this one; 40 steps of a
// 17x17 sheet 66 and 10.8 ms, 30 forward and adjoint steps of a 200x200 sheet 440 and 211 ms.
// Workgroups take the tasks in a topological order and wait on per-front counters, so the
// only tasks ever waited for have been taken by workgroups that run (one of each queue is
// enough: the order within every queue is part of one order of all tasks, and a workgroup
// changes queues empty-handed), and a launch per level and kind (65 launches of at least
// 4 us each on that sheet) is saved. Every array that one task writes and another reads
// is written once per launch, on cache lines of its own, with write-through stores, and
// read only after its counter, so ordinary cached loads see it. All waits are bounded: a
// time-out ends the launch, the residual test fails and the iterative solver takes over.
// Every sum has a fixed order, so results do not depend on which workgroup ran what, nor, in
// a handle that is solved directly, on the other sheets of its batch (whether it is, is
// decided for all its sheets together: by their memory, and by the time either solver takes).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "direct.h"
#include "direct_kernels.h"

namespace phisft {
namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kSide = 3 * kDsMaxPiv / kDsTile;   // tiles of the largest pivot block
constexpr int kLd = 3 * kDsMaxPiv + 2;           // LDS row stride of the blocks
constexpr int kLdT = 18;                         // LDS row stride of a 16x16 tile
constexpr int kLdK = 50;                         // LDS row stride of a Schur operand's half
constexpr int kLds = 3 * kDsMaxPiv * kLd;        // doubles of dynamic LDS
constexpr int kSpinLimit = 1 << 22;              // polls of a wait (seconds)
static_assert(kDsMaxBorder + 3 * kDsMaxPiv + 16 * 33 <= kLds, "backward task's vectors");
static_assert(2 * kDsSchurTile * kLdK <= kLds, "Schur operands");
static_assert((3 * kSide + 3) * 16 * kLdT <= kLds, "pivot sweep panels and diagonal");

__device__ __forceinline__ dbl4 mfma4(double a, double b, dbl4 c) {
  // A operand: lane l holds row l % 16, column l / 16; B: row l / 16, column l % 16;
  // C/D: register q holds row 4 q + l / 16, column l % 16
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const int2 t = *reinterpret_cast<const int2*>(&v);
  int2 r;
  r.x = __builtin_amdgcn_readlane(t.x, lane);
  r.y = __builtin_amdgcn_readlane(t.y, lane);
  return *reinterpret_cast<double*>(&r);
}

// Reciprocal from the hardware estimate x and its error e = 1 - a x: x (1 + e + e^2),
// which leaves e^3 (1 / a = x / (1 - e)).
__device__ __forceinline__ double recip(double a) {
  const double x = __builtin_amdgcn_rcp(a);
  const double e = fma(-a, x, 1.0);
  return fma(x, fma(e, e, e), x);
}

// Symmetric sweep of a symmetric 16x16 tile in the matrix cores' C layout on one
// wavefront, four pivots at a time: with Q the inverse of the 4x4 pivot block and R the
// four pivot rows (register kb),
//   M_ij -= R_i^T Q R_j,  M_kj = Q R_j,  M_ik = R_i^T Q,  M_kk = -Q,
// which after all pivots leaves -M^-1. By symmetry the pivot rows in C layout are at once
// the A operand (R^T) and the B operand of a rank-4 update, so each step is two matrix
// instructions; the pivot columns come out of the same update with -Q in their place of
// the B operand and zero in the accumulator (nothing cancels). The 4x4 block is inverted
// in 2x2 blocks from lane broadcasts (two reciprocals in a row instead of four: 860
// cycles a step where elimination column by column took 970), the determinants with the
// products' rounding errors included. False if a pivot is not positive.
__device__ __forceinline__ double det2(double a, double b, double c) {
  const double bb = b * b;
  return fma(a, c, -bb) - fma(b, b, -bb);
}
__device__ __forceinline__ bool sweep16(dbl4& d, int lane) {
  const int g = lane >> 4, c = lane & 15, c4 = c & 3;
  bool good = true;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const double R = d[kb];
    const double a = lane_value(R, 4 * kb), b = lane_value(R, 16 + 4 * kb),
                 e = lane_value(R, 16 + 4 * kb + 1);
    const double m00 = lane_value(R, 32 + 4 * kb), m01 = lane_value(R, 32 + 4 * kb + 1),
                 m10 = lane_value(R, 48 + 4 * kb), m11 = lane_value(R, 48 + 4 * kb + 1);
    const double s00 = lane_value(R, 32 + 4 * kb + 2), s10 = lane_value(R, 48 + 4 * kb + 2),
                 s11 = lane_value(R, 48 + 4 * kb + 3);
    // I = [a b; b e]^-1, L = [m] I, J = ([s] - L [m]^T)^-1
    const double da = det2(a, b, e), ra = recip(da);
    const double i00 = e * ra, i01 = -b * ra, i11 = a * ra;
    const double l00 = fma(m00, i00, m01 * i01), l01 = fma(m00, i01, m01 * i11);
    const double l10 = fma(m10, i00, m11 * i01), l11 = fma(m10, i01, m11 * i11);
    const double t00 = s00 - fma(l00, m00, l01 * m01);
    const double t10 = s10 - fma(l10, m00, l11 * m01);
    const double t11 = s11 - fma(l10, m10, l11 * m11);
    const double dt = det2(t00, t10, t11), rt = recip(dt);
    const double j00 = t11 * rt, j01 = -t10 * rt, j11 = t00 * rt;
    good = good && a > 0.0 && da > 0.0 && t00 > 0.0 && dt > 0.0;
    // Q = [I + L^T K, -K^T; -K, J], K = J L
    const double k00 = fma(j00, l00, j01 * l10), k01 = fma(j00, l01, j01 * l11);
    const double k10 = fma(j01, l00, j11 * l10), k11 = fma(j01, l01, j11 * l11);
    const double q00 = fma(l00, k00, fma(l10, k10, i00)), q01 = fma(l00, k01, fma(l10, k11, i01)),
                 q11 = fma(l01, k01, fma(l11, k11, i11));
    // this lane's entry Q[c % 4][g]
    const bool g1 = g & 1, c1 = c & 1;
    const double qi = c1 ? (g1 ? q11 : q01) : (g1 ? q01 : q00);
    const double qj = c1 ? (g1 ? j11 : j01) : (g1 ? j01 : j00);
    const int row = g < 2 ? c4 : g, col = g < 2 ? g : c4;   // below the diagonal blocks
    const double qk = (row & 1) ? ((col & 1) ? k11 : k10) : ((col & 1) ? k01 : k00);
    const double sel = (g < 2) == (c4 < 2) ? (g < 2 ? qi : qj) : -qk;
    const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
    const dbl4 v = mfma4(c < 4 ? sel : 0.0, R, zero);  // rows 0..3: Q R
    const bool piv = (c >> 2) == kb;
    const double V = piv ? -sel : v[0];
    dbl4 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = piv ? 0.0 : d[q];
    d = mfma4(-R, V, acc);
    d[kb] = V;
  }
  return good;
}

// Sum over the 16 lanes of a DPP row, the same in each.
__device__ __forceinline__ double row_sum(double v) {
#define PHISFT_ROW_STEP(ctrl)                                                        \
  {                                                                                  \
    int2 t = *reinterpret_cast<int2*>(&v);                                           \
    t.x = __builtin_amdgcn_update_dpp(0, t.x, ctrl, 0xf, 0xf, false);                \
    t.y = __builtin_amdgcn_update_dpp(0, t.y, ctrl, 0xf, 0xf, false);                \
    v += *reinterpret_cast<double*>(&t);                                             \
  }
  PHISFT_ROW_STEP(0x140)   // row mirror
  PHISFT_ROW_STEP(0x141)   // half mirror
  PHISFT_ROW_STEP(0x4E)    // quad_perm [2,3,0,1]
  PHISFT_ROW_STEP(0xB1)    // quad_perm [1,0,3,2]
#undef PHISFT_ROW_STEP
  return v;
}

// Stores that reach memory, for data other workgroups of the launch read.
__device__ __forceinline__ void put(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroup's barrier. The wait for this wavefront's own LDS accesses is written out:
// hipcc leaves it away at the head of the task loop, where the access in flight is on the
// loop's back edge (a wavefront then reads the last task's number and does that again).
__device__ __forceinline__ void sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
}

// Buffer accesses: a uniform base and size in scalar registers, one 32-bit byte offset per
// lane, and no test of bounds in the code: a load past the size gives zero, a store past
// it does nothing. Tasks are short and bound by their instructions, so this counts.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kNowhere = 0x40000000;   // an offset past every size, also added to another
constexpr int kSc1 = 16;               // write through the caches
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const double* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ double load1(__amdgpu_buffer_rsrc_t b, int at) {
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, at, 0, 0);
  return *reinterpret_cast<const double*>(&v);
}
__device__ __forceinline__ double2 load2(__amdgpu_buffer_rsrc_t b, int at) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, at, 0, 0);
  return *reinterpret_cast<const double2*>(&v);
}
__device__ __forceinline__ void put1(__amdgpu_buffer_rsrc_t b, int at, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const u32x2*>(&v), b, at, 0, kSc1);
}
__device__ __forceinline__ void put2(__amdgpu_buffer_rsrc_t b, int at, double2 v) {
  __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(&v), b, at, 0, kSc1);
}

// Rows of an LDS block (stride kLd, np columns) to memory, 16 threads a row.
__device__ __forceinline__ void put_rows(double* p, const double* l, int rows, int np, int tid) {
  const __amdgpu_buffer_rsrc_t b = buffer(p, rows * np * 8);
#pragma unroll
  for (int i = 0; i < 3 * kDsMaxPiv; i += kThreads / 16) {
    if (i >= rows) break;
    const int r = i + (tid >> 4), c = 2 * (tid & 15);
#pragma unroll
    for (int k = 0; k < 3 * kDsMaxPiv; k += 32)
      if (k + c < np)
        put2(b, (r * np + k + c) * 8, *reinterpret_cast<const double2*>(l + r * kLd + k + c));
  }
}

__device__ __forceinline__ double2 get2(const double* p) {
  return *reinterpret_cast<const double2*>(p);
}

// Tables that no task writes, read at uniform addresses through the scalar cache.
template <class T>
using Table = const __attribute__((address_space(4))) T*;

template <class T>
__device__ __forceinline__ Table<T> table(const T* p) {
  return (Table<T>)reinterpret_cast<uintptr_t>(p);
}

struct Shared {
  int go[kDsGoWords], bad;
  int next[2];     // >= 0: rec holds a task
  DsTask rec[2];   // this task's and the next one's record, in turn
};

// What wavefront 0 holds of the next task while this one runs.
struct Next {
  const DsTask* tasks;
  int list;        // of DsArgs::q0
  int queue;       // the queue this workgroup takes from,
  int base, count; // its first task and their number
  int slot;        // of Shared::rec for the next task
  int turn;        // of Shared::go for the next wait; the same in every thread
  int number;      // in its queue; -1: the queue is empty, -2: all are
  unsigned long long rec;   // 8 bytes of its record per lane
};

// The thread's number, opaque to the optimiser: what each task derives from it would
// otherwise be moved out of the task loop and stay in registers across all tasks.
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v) {
  const int lo = uni((int)v), hi = uni((int)(v >> 32));
  return (long long)hi << 32 | (unsigned)lo;
}

// Waits (bounded) until every lane's counter of wavefront 0 reaches the lane's target (0:
// nothing to wait for). Every thread calls. 0 when the launch is to end, else 1, or 3 when
// the counters have also reached `want`. Also a barrier of the workgroup. Thread 0 hands the
// outcome over in two words in turn, for waits may follow each other without another
// barrier: it writes a word again only past the next wait's barrier, which every
// wavefront enters after it has read this wait's outcome. With one word a wavefront that
// reads late would take the next wait's outcome for this one's.
__device__ __forceinline__ int wait_lanes(Table<DsArgs> a, int c, int target, int want, Next& nx,
                                          Shared& sh) {
  int& word = sh.go[nx.turn];
  nx.turn = ds_next_word(nx.turn);
  if (threadIdx.x < 64) {
    int go = 1;
    for (int spins = 0;;) {
      int v = 0;
      if (target > 0 || want > 0)
        v = __hip_atomic_load(a->count + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__all(v >= target)) {
        if (__all(v >= want)) go = 3;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      if ((++spins & 255) == 0) {
        if (spins > kSpinLimit)
          __hip_atomic_store(a->abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__hip_atomic_load(a->abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
          go = 0;
          break;
        }
      }
    }
    if (threadIdx.x == 0) word = go;
  }
  sync();
  return uni(word);
}

__device__ __forceinline__ bool wait_one(Table<DsArgs> a, int c, int target, Next& nx, Shared& sh) {
  return wait_lanes(a, c, threadIdx.x == 0 ? target : 0, 0, nx, sh) != 0;
}

// Waits for the children's counters `which` (and looks whether the counters c2 of lanes 2
// and up have reached their `want`): as wait_lanes.
__device__ __forceinline__ int wait_children(Table<DsArgs> a, const DsTask& tk, int which, int c2,
                                             int want, Next& nx, Shared& sh) {
  const int lane = thread_id();
  int c = c2, target = 0;
  if (lane < 2) {
    c = tk.f.kcnt[lane] + which;
    target = which == kDsHeadDone ? tk.f.khead[lane] : which == kDsSchurDone ? tk.f.kschur[lane]
                                                                             : tk.f.kfwd[lane];
  }
  const int nc = uni(tk.f.nc);
  int go = wait_lanes(a, c, target, lane < 2 ? target : want, nx, sh);
  for (int base = 2; go && base < nc; base += 64) {   // rare: more than two children
    target = 0;
    if (lane < 64 && base + lane < nc) {
      const DsChild& K = a->kid[tk.f.c0 + base + lane];
      c = K.cnt + which;
      target = which == kDsHeadDone ? K.nhead : which == kDsSchurDone ? K.nschur : K.nfwd;
    }
    go = wait_lanes(a, c, target, 0, nx, sh) ? 1 : 0;
  }
  return go;
}

__device__ __forceinline__ void claim(Table<DsArgs> a, Next& nx) {
  if (threadIdx.x == 0)
    nx.number = __hip_atomic_fetch_add(a->queue + kDsLine * nx.queue, 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void load_record(Next& nx) {
  nx.rec = reinterpret_cast<const unsigned long long*>(nx.tasks + nx.base + nx.number)[threadIdx.x];
}

// Starts the load of the next task's record; some time into the task, when the next one's
// number has come back from the queue.
__device__ __forceinline__ void fetch_next(Next& nx) {
  if (threadIdx.x >= 64) return;
  nx.number = uni(nx.number);
  if (nx.number >= nx.count) nx.number = -1;
  else load_record(nx);
}

// Takes a task from the first queue that has one, its own first. Only when no task is
// held: a task of another queue may come before the one being run, and waiting for it
// behind that one could be waiting for itself.
__device__ __forceinline__ void find_task(Table<DsArgs> a, Next& nx, bool first, Shared& sh) {
  if (threadIdx.x < 64) {
    const Table<int> q0 = a->q0[nx.list];
    for (;;) {
      const int q = (nx.queue + threadIdx.x) % kDsQueues;
      int head = 0;
      if (!first && threadIdx.x < kDsQueues)
        head = __hip_atomic_load(a->queue + kDsLine * q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool some = threadIdx.x < kDsQueues && head < q0[q + 1] - q0[q];
      first = false;
      const unsigned long long m = __ballot(some);
      nx.number = -2;
      if (m == 0) break;
      nx.queue = (nx.queue + __builtin_ctzll(m)) % kDsQueues;
      nx.base = q0[nx.queue];
      nx.count = q0[nx.queue + 1] - nx.base;
      claim(a, nx);
      nx.number = uni(nx.number);
      if (nx.number < nx.count) {
        load_record(nx);
        reinterpret_cast<unsigned long long*>(&sh.rec[nx.slot])[threadIdx.x] = nx.rec;
        break;
      }
    }
    if (threadIdx.x == 0) sh.next[nx.slot] = nx.number;
  }
  sync();
}

// Counts a task as done once every wavefront's stores have completed (put() writes
// through, so completion is visibility), and hands over to the next task.
__device__ __forceinline__ void signal(Table<DsArgs> a, int c, int c2, const Next& nx, Shared& sh) {
  if (threadIdx.x < 64) reinterpret_cast<unsigned long long*>(&sh.rec[nx.slot])[threadIdx.x] = nx.rec;
  if (threadIdx.x == 0) sh.next[nx.slot] = nx.number;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  sync();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(a->count + c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (c2 >= 0) __hip_atomic_fetch_add(a->count + c2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Local unknown of unknown u of child ch's border (u < 3 q).
__device__ __forceinline__ int local_of(Table<DsArgs> a, const DsTask& tk, int ch, int u) {
  const int v = ch < 2 ? tk.col[ch][u / 3] : a->tab[a->kid[tk.f.c0 + ch].map + u / 3];
  return 3 * v + u % 3;
}

// X = F_pp^-1. The lower triangle of F_pp is gathered into LDS (A's entries, then the
// children's updates in order), then held as 16x16 tiles by wavefronts 1 to 7, three
// each at most; wavefront 0 carries the chain. Per tile row k, phase A: wavefront 0
// applies step k - 1 to tile (k, k) and sweeps it, publishing -Q (Q its inverse); the
// others apply step k - 1 to their tiles and publish the old row k, R (the part right of
// the diagonal transposed), and tile (k + 1, k + 1). Phase B: V = Q R is formed, a column
// tile per wavefront; wavefront 0 takes column k + 1, the one it goes on with, from and
// into registers. So the chain per step is one 16x16 sweep, eight matrix instructions and
// two barriers, and everything else runs beside the sweep: a 96x96 block takes 13.6 us
// where updating the diagonal tiles on wavefront 0 as well took 19.0 us.
// A front whose sweep meets a non-positive pivot stores NaN: its solution fails the
// residual test.
__device__ __forceinline__ bool task_pivot(Table<DsArgs> a, const DsTask& tk, Next& nx, double* fac,
                                           double* lds, Shared& sh) {
  const int tid = thread_id(), lane = tid & 63, wave = uni(tid >> 6);
  const int np = uni(tk.f.np), T = np / kDsTile, n3 = 3 * uni(tk.f.p), nc = uni(tk.f.nc);
  const int cnt = uni(tk.f.cnt);
  if (tid == 0) sh.bad = 0;
  for (int e = tid; e < np * kLd; e += kThreads) lds[e] = 0.0;
  sync();
  if (tid < np && tid >= n3) lds[tid * kLd + tid] = 1.0;
  const int nalist = uni(tk.f.nalist);
  const int2* alist = reinterpret_cast<const int2*>(a->tab + uni(tk.f.alist));
  for (int e = tid; e < nalist; e += kThreads) {
    const int2 en = alist[e];
    const int l = en.y >> 16, i = en.y & 0xffff;
    double x[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) x[q] = a->A[en.x + (size_t)q * a->nv];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (l == i && c < r) continue;
        lds[(3 * l + c) * kLd + 3 * i + r] = x[3 * r + c];
      }
  }
  if (!wait_children(a, tk, kDsHeadDone, 0, 0, nx, sh)) return false;
  // A lane takes columns lane and lane + 64 of every eighth row (at most 96); the loads of
  // the first two children are all in flight before the first is used.
  constexpr int NR = 3 * kDsMaxPiv / kWaves, N0 = 64 / kWaves, N1 = NR - N0;
  auto gather = [&](const double* S, int nq, int nb, double (&s0)[NR], double (&s1)[N1]) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int r = wave + kWaves * q;
      s0[q] = r < nq && lane <= r ? S[(size_t)r * nb + lane] : 0.0;
      if (q >= N0) s1[q - N0] = r < nq && lane + 64 <= r ? S[(size_t)r * nb + lane + 64] : 0.0;
    }
  };
  auto add = [&](int ch, int nq, const double (&s0)[NR], const double (&s1)[N1]) {
    const int m0 = lane < nq ? local_of(a, tk, ch, lane) : 0;
    const int m1 = lane + 64 < nq ? local_of(a, tk, ch, lane + 64) : 0;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int r = wave + kWaves * q;
      if (r >= nq) continue;
      double* row = lds + __builtin_amdgcn_readlane(q < N0 ? m0 : m1, r & 63) * kLd;
      if (lane <= r) row[m0] += s0[q];
      if (q >= N0 && lane + 64 <= r) row[m1] += s1[q - N0];
    }
  };
  {
    double s0[2][NR], s1[2][N1];
    int nq[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      nq[ch] = ch < nc ? 3 * uni(tk.kid[ch].q) : 0;
      gather(a->ws + (ch < nc ? uni(tk.kid[ch].so) : 0), nq[ch], uni(tk.kid[ch].nb), s0[ch], s1[ch]);
    }
    add(0, nq[0], s0[0], s1[0]);
    if (nc > 1) {
      sync();
      add(1, nq[1], s0[1], s1[1]);
    }
  }
  for (int ch = 2; ch < nc; ++ch) {   // rare
    const DsChild& K = a->kid[uni(tk.f.c0) + ch];
    double s0[NR], s1[N1];
    gather(a->ws + K.so, 3 * K.q, K.nb, s0, s1);
    sync();
    add(ch, 3 * K.q, s0, s1);
  }
  fetch_next(nx);
  sync();
  const int g = lane >> 4, c16 = lane & 15;
  constexpr int NS = (kSide * (kSide + 1) / 2 + kWaves - 2) / (kWaves - 1);
  constexpr int TL = 16 * kLdT;            // a tile in LDS
  dbl4 d[NS];
  int ti[NS], tj[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int e = (wave - 1) + (kWaves - 1) * s;
    const bool own = wave > 0 && e < T * (T + 1) / 2;
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= e) ++i;
    ti[s] = own ? i : -1;
    tj[s] = own ? e - i * (i + 1) / 2 : -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * ti[s] + 4 * q + g, c = 16 * tj[s] + c16;
      d[s][q] = own ? lds[max(r, c) * kLd + min(r, c)] : 0.0;
    }
  }
  dbl4 v = {0.0, 0.0, 0.0, 0.0}, vr = v, vv = v;   // wavefront 0: tile (k, k), R and V of column k
  if (wave == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 4 * q + g;
      v[q] = lds[max(r, c16) * kLd + min(r, c16)];
    }
  }
  sync();
  double* Rl = lds;                        // [2][T] old rows
  double* Vl = Rl + 2 * kSide * TL;        // [T] scaled rows
  double* Pl = Vl + kSide * TL;            // [2] -Q
  double* Dl = Pl + 2 * TL;                // the next diagonal tile
  const int at = g * kLdT + c16;
  auto load = [&](const double* t) {
    dbl4 x;
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = t[4 * q * kLdT + at];
    return x;
  };
  auto store = [&](double* t, const dbl4& x) {
#pragma unroll
    for (int q = 0; q < 4; ++q) t[4 * q * kLdT + at] = x[q];
  };
  // this wavefront's tile s after step k
  auto step = [&](int s, int k) {
    if (ti[s] == k) {
      d[s] = load(tj[s] == k ? Pl + (k & 1) * TL : Vl + tj[s] * TL);
      return;
    }
    const dbl4 r = load(Rl + ((k & 1) * kSide + ti[s]) * TL);
    const dbl4 x = load(tj[s] == k ? Pl + (k & 1) * TL : Vl + tj[s] * TL);
    if (tj[s] == k) d[s] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q) d[s] = mfma4(-r[q], x[q], d[s]);
  };
#pragma unroll 1
  for (int k = 0; k < T; ++k) {
    double* Rk = Rl + (k & 1) * kSide * TL;
    double* Pk = Pl + (k & 1) * TL;
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      if (k > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v = mfma4(-vr[q], vv[q], v);
      }
      if (!sweep16(v, lane) && lane == 0) sh.bad = 1;
      store(Pk, v);
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (ti[s] < 0) continue;
        if (k > 0) step(s, k - 1);
        if (ti[s] == k && tj[s] < k) store(Rk + tj[s] * TL, d[s]);
        if (tj[s] == k && ti[s] > k) {
#pragma unroll
          for (int q = 0; q < 4; ++q) Rk[ti[s] * TL + c16 * kLdT + 4 * q + g] = d[s][q];
        }
        if (ti[s] == k + 1 && tj[s] == k + 1) store(Dl, d[s]);
      }
    }
    sync();
    if (wave == 0) {
      if (k + 1 < T) {
        vr = load(Rk + (k + 1) * TL);
        vv = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) vv = mfma4(-v[q], vr[q], vv);
        v = load(Dl);
        store(Vl + (k + 1) * TL, vv);
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (wave <= T && wave - 1 != k && wave - 1 != k + 1) {
      const dbl4 p = load(Pk), r = load(Rk + (wave - 1) * TL);
      dbl4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q) x = mfma4(-p[q], r[q], x);
      store(Vl + (wave - 1) * TL, x);
    }
    sync();
  }
  const bool bad = sh.bad != 0;
  if (wave > 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (ti[s] >= 0) step(s, T - 1);
  }
  sync();
  // X = -M by way of LDS, both triangles, then rows of it with 16-byte stores
  if (wave > 0) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (ti[s] < 0) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 16 * ti[s] + 4 * q + g, c = 16 * tj[s] + c16;
        const double x = bad ? NAN : -d[s][q];
        lds[r * kLd + c] = x;
        if (ti[s] != tj[s]) lds[c * kLd + r] = x;
      }
    }
  }
  sync();
  put_rows(fac + uni(tk.f.xo), lds, np, np, tid);
  signal(a, cnt + kDsPivotDone, -1, nx, sh);
  return true;
}

// W rows of a border tile: wavefront j forms column tile j of both row tiles. The lanes'
// part of X (symmetric: read along its rows, lane groups taking contiguous quarters of
// the inner dimension) is loaded at once.
template <int T>
__device__ __forceinline__ void border_product(const double* __restrict__ X, const double* Fl,
                                               double* W, int rows, int wave, int lane) {
  constexpr int np = 16 * T, kq = np / 4;
  if (wave >= T) return;
  const int g = lane >> 4, c16 = lane & 15;
  const double2* xr = reinterpret_cast<const double2*>(X + (size_t)(16 * wave + c16) * np + g * kq);
  double2 x[kq / 2];
#pragma unroll
  for (int s = 0; s < kq / 2; ++s) x[s] = get2(reinterpret_cast<const double*>(xr + s));
  dbl4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  const double2* f0 = reinterpret_cast<const double2*>(Fl + c16 * kLd + g * kq);
  const double2* f1 = reinterpret_cast<const double2*>(Fl + (16 + c16) * kLd + g * kq);
#pragma unroll
  for (int s = 0; s < kq / 2; ++s) {
    const double2 u = f0[s], v = f1[s];
    acc[0] = mfma4(u.x, x[s].x, acc[0]);
    acc[1] = mfma4(v.x, x[s].x, acc[1]);
    acc[0] = mfma4(u.y, x[s].y, acc[0]);
    acc[1] = mfma4(v.y, x[s].y, acc[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (16 * i < rows) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        put(W + (size_t)(16 * i + 4 * q + g) * np + 16 * wave + c16, acc[i][q]);
    }
}

// F_bp and W = F_bp X of 32 border rows; F_bp is gathered into LDS like the pivot block.
__device__ __forceinline__ bool task_border(Table<DsArgs> a, const DsTask& tk, Next& nx,
                                            double* fac, double* lds, Shared& sh) {
  constexpr int NR = kDsRowTile / kWaves;
  double* Fl = lds;
  const int tid = thread_id(), lane = tid & 63, wave = uni(tid >> 6);
  const int tile = uni(tk.a), np = uni(tk.f.np), nc = uni(tk.f.nc), p = uni(tk.f.p);
  const int cnt = uni(tk.f.cnt), r0 = tile * kDsRowTile, rows = min(kDsRowTile, uni(tk.f.nb) - r0);
  const int lo = uni(tk.lo), hi = uni(tk.hi);
  for (int e = tid; e < kDsRowTile * kLd; e += kThreads) Fl[e] = 0.0;
  sync();
  for (int e = lo + tid; e < hi; e += kThreads) {
    const int2 en = reinterpret_cast<const int2*>(a->tab)[e];
    const int l = (en.y >> 16) - p, i = en.y & 0xffff;
    double x[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) x[q] = a->A[en.x + (size_t)q * a->nv];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int row = 3 * l + c - r0;
      if (row < 0 || row >= kDsRowTile) continue;
#pragma unroll
      for (int r = 0; r < 3; ++r) Fl[row * kLd + 3 * i + r] = x[3 * r + c];
    }
  }
  const int go = wait_children(a, tk, kDsSchurDone, cnt + kDsPivotDone, lane == 2 ? 1 : 0, nx, sh);
  if (!go) return false;
  // a lane takes pivot columns lane and lane + 64 of this wavefront's rows of a child
  auto gather = [&](int ch, const double* S0, int nq, int ld, double (&s0)[NR], double (&s1)[NR]) {
    const int c0 = lane < nq ? 8 * lane : kNowhere, c1 = lane + 64 < nq ? 8 * (lane + 64) : kNowhere;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int br = r0 + wave + kWaves * q;
      int v = -1;
      if (ch < 2) v = uni((int)tk.row[ch & 1][br / 3 - r0 / 3]);
      else if (br < 3 * tk.f.b) v = a->tab[a->kid[tk.f.c0 + ch].inv + p + br / 3];
      const __amdgpu_buffer_rsrc_t S =
          buffer(S0 + (size_t)(3 * max(v, 0) + br % 3) * ld, v >= 0 ? 8 * nq : 0);
      s0[q] = load1(S, c0);
      s1[q] = load1(S, c1);
    }
  };
  auto add = [&](int ch, int nq, const double (&s0)[NR], const double (&s1)[NR]) {
    if (lane < nq) {
      double* x = Fl + wave * kLd + local_of(a, tk, ch, lane);
#pragma unroll
      for (int q = 0; q < NR; ++q) x[kWaves * q * kLd] += s0[q];
    }
    if (lane + 64 < nq) {
      double* x = Fl + wave * kLd + local_of(a, tk, ch, lane + 64);
#pragma unroll
      for (int q = 0; q < NR; ++q) x[kWaves * q * kLd] += s1[q];
    }
  };
  {
    // both children's loads are in flight before the first is used; a row is this
    // wavefront's alone, so the sums need no barrier
    double s0[2][NR], s1[2][NR];
    int nq[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      nq[ch] = ch < nc ? 3 * uni(tk.kid[ch].q) : 0;
      gather(ch, a->ws + (ch < nc ? uni(tk.kid[ch].so) : 0), nq[ch], uni(tk.kid[ch].nb), s0[ch],
             s1[ch]);
    }
    add(0, nq[0], s0[0], s1[0]);
    add(1, nq[1], s0[1], s1[1]);
  }
  for (int ch = 2; ch < nc; ++ch) {   // rare
    const DsChild& K = a->kid[tk.f.c0 + ch];
    double s0[NR], s1[NR];
    gather(ch, a->ws + K.so, 3 * K.q, K.nb, s0, s1);
    add(ch, 3 * K.q, s0, s1);
  }
  sync();
  put_rows(a->ws + uni(tk.f.bo) + (size_t)r0 * np, Fl, rows, np, tid);
  fetch_next(nx);
  if (go == 1 && !wait_one(a, cnt + kDsPivotDone, 1, nx, sh)) return false;
  const double* X = fac + uni(tk.f.xo);
  double* W = fac + uni(tk.f.wo) + (size_t)r0 * np;
  switch (np / kDsTile) {
    case 1: border_product<1>(X, Fl, W, rows, wave, lane); break;
    case 2: border_product<2>(X, Fl, W, rows, wave, lane); break;
    case 3: border_product<3>(X, Fl, W, rows, wave, lane); break;
    case 4: border_product<4>(X, Fl, W, rows, wave, lane); break;
    case 5: border_product<5>(X, Fl, W, rows, wave, lane); break;
    default: border_product<6>(X, Fl, W, rows, wave, lane); break;
  }
  signal(a, cnt + kDsRowsDone + tile / (kDsSchurTile / kDsRowTile), -1, nx, sh);
  return true;
}

// acc += (rows of W) (rows of B)^T over kc (a multiple of 16) staged columns: a 32x16 block
// per wavefront, lane groups taking quarters of the columns.
__device__ __forceinline__ void schur_product(const double* w0, const double* b0, int kc, int g,
                                              dbl4 (&acc)[2]) {
  const int kq = kc / 4, o = g * kq;
  for (int s = 0; s < kq; s += 4) {
    const double2 x0 = *reinterpret_cast<const double2*>(w0 + o + s);
    const double2 x1 = *reinterpret_cast<const double2*>(w0 + o + s + 2);
    const double2 y0 = *reinterpret_cast<const double2*>(w0 + 16 * kLdK + o + s);
    const double2 y1 = *reinterpret_cast<const double2*>(w0 + 16 * kLdK + o + s + 2);
    const double2 z0 = *reinterpret_cast<const double2*>(b0 + o + s);
    const double2 z1 = *reinterpret_cast<const double2*>(b0 + o + s + 2);
    acc[0] = mfma4(x0.x, z0.x, acc[0]);
    acc[1] = mfma4(y0.x, z0.x, acc[1]);
    acc[0] = mfma4(x0.y, z0.y, acc[0]);
    acc[1] = mfma4(y0.y, z0.y, acc[1]);
    acc[0] = mfma4(x1.x, z1.x, acc[0]);
    acc[1] = mfma4(y1.x, z1.x, acc[1]);
    acc[0] = mfma4(x1.y, z1.y, acc[0]);
    acc[1] = mfma4(y1.y, z1.y, acc[1]);
  }
}

// S = (children) - W F_bp^T, one lower 64x64 tile: each wavefront forms a 32x16 block. The
// children's parts travel while the border rows are waited for; the operands pass through
// LDS in halves of the inner dimension.
__device__ __forceinline__ bool task_schur(Table<DsArgs> a, const DsTask& tk, Next& nx, double* fac,
                                           double* lds, Shared& sh) {
  double* Wl = lds;
  double* Bl = lds + kDsSchurTile * kLdK;
  const int tid = thread_id(), lane = tid & 63, wave = uni(tid >> 6);
  const int g = lane >> 4, c16 = lane & 15;
  const int np = uni(tk.f.np), nb = uni(tk.f.nb), nc = uni(tk.f.nc), cnt = uni(tk.f.cnt);
  const int ij = uni(tk.a);
  const int I = ij >> 16, J = ij & 0xffff, I0 = I * kDsSchurTile, J0 = J * kDsSchurTile;
  const int i0 = I0 + 32 * (wave >> 2), col = J0 + 16 * (wave & 3) + c16;
  // byte offsets of the tile's rows and columns in the first children's updates
  unsigned* places = reinterpret_cast<unsigned*>(lds + 2 * kDsSchurTile * kLdK);   // [child][row, col][64]
  if (tid < 4 * kDsSchurTile) {
    const int ch = tid >> 7, u = tid & 63, base = tid & 64 ? J0 : I0, x = (base + u) / 3;
    const int k = x - base / 3, ld = tk.kid[ch].nb;
    const int v = ch < nc ? (tid & 64 ? tk.col[ch][k] : tk.row[ch][k]) : -1;
    const int e = 8 * (3 * v + base + u - 3 * x);
    places[tid] = v < 0 ? kNowhere : tid & 64 ? e : e * ld;
  }
  constexpr int per = kDsSchurTile / kDsRowTile;
  const int group = lane == 2 ? I : J, rows_cnt = cnt + kDsRowsDone + group;
  const int rows_of = lane == 2 || lane == 3
                          ? min(per, (nb + kDsRowTile - 1) / kDsRowTile - per * group) : 0;
  const int go = wait_children(a, tk, kDsSchurDone, rows_cnt, rows_of, nx, sh);
  if (!go) return false;
  double x[2][8];
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    const int ld = ch < nc ? uni(tk.kid[ch].nb) : 0;
    const __amdgpu_buffer_rsrc_t S = buffer(a->ws + (ch < nc ? uni(tk.kid[ch].so) : 0), 8 * ld * ld);
    const unsigned* rows = places + 128 * ch + 32 * (wave >> 2) + g;
    const unsigned c = places[128 * ch + 64 + 16 * (wave & 3) + c16];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[ch][q] = load1(S, (int)(rows[4 * q] + c));
  }
  if (go == 1 && !wait_lanes(a, rows_cnt, rows_of, 0, nx, sh)) return false;
  // Halves of at most 48 columns, 16, 32 or 48: eight threads a row, up to three 16-byte
  // pieces each; the second half travels during the first's products.
  const __amdgpu_buffer_rsrc_t W = buffer(fac + uni(tk.f.wo), 8 * nb * np);
  const __amdgpu_buffer_rsrc_t B = buffer(a->ws + uni(tk.f.bo), 8 * nb * np);
  const int k1 = min(np, 48), k2 = np - k1;
  const int sr = tid >> 3, sc = 2 * (tid & 7);
  const int wat = 8 * ((I0 + sr) * np + sc), bat = 8 * ((J0 + sr) * np + sc);
  double2 wv[3], bv[3];
  auto fetch = [&](int k0, int k) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (16 * q < k) {
        wv[q] = load2(W, wat + 8 * k0 + 128 * q);
        bv[q] = load2(B, bat + 8 * k0 + 128 * q);
      }
  };
  auto stage = [&](int k) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (16 * q < k) {
        *reinterpret_cast<double2*>(Wl + sr * kLdK + sc + 16 * q) = wv[q];
        *reinterpret_cast<double2*>(Bl + sr * kLdK + sc + 16 * q) = bv[q];
      }
  };
  fetch(0, k1);
  dbl4 acc[2];
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q >> 2][q & 3] = -(x[0][q] + x[1][q]);
  stage(k1);
  if (k2 > 0) fetch(48, k2);
  fetch_next(nx);
  sync();
  const double* w0 = Wl + (32 * (wave >> 2) + c16) * kLdK;
  const double* b0 = Bl + (16 * (wave & 3) + c16) * kLdK;
  schur_product(w0, b0, k1, g, acc);
  if (k2 > 0) {
    sync();
    stage(k2);
    sync();
    schur_product(w0, b0, k2, g, acc);
  }
  for (int ch = 2; ch < nc; ++ch) {   // rare
    const DsChild& K = a->kid[tk.f.c0 + ch];
    const int b3 = 3 * uni(tk.f.b);
    const int* inv = a->tab + K.inv + tk.f.p;
    const int v = col < b3 ? inv[col / 3] : -1;
    if (v < 0) continue;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int row = i0 + 4 * q + g;
      const int w = row < b3 && col <= row ? inv[row / 3] : -1;
      if (w >= 0)
        acc[q >> 2][q & 3] -= a->ws[K.so + (size_t)(3 * w + row % 3) * K.nb + 3 * v + col % 3];
    }
  }
  const __amdgpu_buffer_rsrc_t S = buffer(a->ws + uni(tk.f.so), 8 * nb * nb);
  const int sat = col < nb ? 8 * ((i0 + g) * nb + col) : kNowhere;
#pragma unroll
  for (int q = 0; q < 8; ++q) put1(S, sat + 32 * nb * q, -acc[q >> 2][q & 3]);
  signal(a, cnt + kDsSchurDone, I < 2 ? cnt + kDsHeadDone : -1, nx, sh);
  return true;
}

// t = b_p + (children), g = (children) - W t of 64 border rows, 16 lanes a row. Every
// workgroup of a front gathers t itself; W travels while the children are waited for.
__device__ __forceinline__ bool task_forward(Table<DsArgs> a, const DsTask& tk, Next& nx, bool factor,
                                             double* fac, double* lds, Shared& sh) {
  constexpr int NP = kDsFwdRows * 16 / kThreads;   // rows of a thread
  static_assert(kDsFwdRows == kDsSchurTile, "a chunk is a group of row tiles");
  double* t = lds;
  const int tid = thread_id(), lane = tid & 63, l16 = tid & 15;
  const int chunk = uni(tk.a), np = uni(tk.f.np), nb = uni(tk.f.nb), nc = uni(tk.f.nc);
  const int cnt = uni(tk.f.cnt), p = uni(tk.f.p), n3 = 3 * uni(tk.f.b), r0 = chunk * kDsFwdRows;
  // W belongs to this launch only when it factorises too
  int go = 1;
  if (factor) {
    constexpr int per = kDsSchurTile / kDsRowTile;
    const int all = (nb + kDsRowTile - 1) / kDsRowTile;
    int c = cnt + kDsRowsDone + chunk, target = lane == 0 && nb > 0 ? min(per, all - per * chunk) : 0;
    int want = target;
    if (lane == 1 || lane == 2) {
      c = tk.f.kcnt[lane - 1] + kDsForwardDone;
      want = tk.f.kfwd[lane - 1];
    }
    go = wait_lanes(a, c, target, want, nx, sh);
    if (!go) return false;
    if (nc > 2) go = 1;
  }
  const __amdgpu_buffer_rsrc_t W = buffer(fac + uni(tk.f.wo), 8 * nb * np);
  double w[NP][kSide];
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int at = 8 * ((r0 + (kThreads / 16) * q + (tid >> 4)) * np + l16);
#pragma unroll
    for (int k = 0; k < kSide; ++k)
      if (16 * k < np) w[q][k] = load1(W, at + 128 * k);
  }
  double v = 0.0;
  if (tid < 3 * p) v = a->rhs[(size_t)(tid % 3) * a->nv + a->tab[tk.f.verts + tid / 3]];
  if (go == 1 && !wait_children(a, tk, kDsForwardDone, 0, 0, nx, sh)) return false;
  double h[NP], e[2];
#pragma unroll
  for (int ch = 0; ch < 2; ++ch) {
    const int x = ch < nc && tid < 3 * p ? tk.col[ch][tid / 3] : -1;
    e[ch] = x >= 0 ? a->ws[tk.kid[ch].g + 3 * x + tid % 3] : 0.0;
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int r = r0 + (kThreads / 16) * q + (tid >> 4);
    double x[2];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
      const int s = ch < nc && l16 == 0 && r < n3 ? tk.row[ch][r / 3 - r0 / 3] : -1;
      x[ch] = s >= 0 ? a->ws[tk.kid[ch].g + 3 * s + r % 3] : 0.0;
    }
    h[q] = x[0] + x[1];
    if (l16 == 0 && r < n3)
      for (int ch = 2; ch < nc; ++ch) {
        const int s = a->tab[tk.f.gsrc + ch * (p + n3 / 3) + p + r / 3];
        if (s >= 0) h[q] += a->ws[s + r % 3];
      }
  }
  if (tid < np) {
    v += e[0] + e[1];
    if (tid < 3 * p)
      for (int ch = 2; ch < nc; ++ch) {
        const int s = a->tab[tk.f.gsrc + ch * (p + n3 / 3) + tid / 3];
        if (s >= 0) v += a->ws[s + tid % 3];
      }
    t[tid] = v;
    if (chunk == 0) put(a->ws + tk.f.t + tid, v);
  }
  fetch_next(nx);
  sync();
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const int r = r0 + (kThreads / 16) * q + (tid >> 4);
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kSide; ++k)
      if (16 * k < np) s += w[q][k] * t[16 * k + l16];
    s = row_sum(s);
    if (l16 == 0 && r < n3) put(a->ws + tk.f.g + r, h[q] - s);
  }
  signal(a, cnt + kDsForwardDone, -1, nx, sh);
  return true;
}

// x_p = X t - W^T x_b of 32 pivot unknowns, the border rows spread over 16 groups of
// threads; X, the first rows of W and the places of x_b travel while the parent is
// waited for.
__device__ __forceinline__ bool task_backward(Table<DsArgs> a, const DsTask& tk, Next& nx, bool factor,
                                              double* fac, double* lds, Shared& sh) {
  constexpr int G = kThreads / kDsBwdCols, NW = 20, NX = 3 * kDsMaxPiv / G, NB = 2;
  double* xb = lds;
  double* t = xb + kDsMaxBorder;
  double* part = t + 3 * kDsMaxPiv;          // [G][33]
  const int tid = thread_id(), lane = tid & 63;
  const int np = uni(tk.f.np), n3 = 3 * uni(tk.f.b), cnt = uni(tk.f.cnt);
  const int cl = tid % kDsBwdCols, rg = tid / kDsBwdCols;
  const int c = uni(tk.a) * kDsBwdCols + cl;
  // the parent's solution, or at a root its own right-hand side
  const int pcnt = uni(tk.f.pcnt), nfwd = uni(tk.f.nfwd);
  const int last = pcnt < 0 ? cnt + kDsForwardDone : pcnt + kDsBackwardDone;
  const int nlast = pcnt < 0 ? nfwd : uni(tk.f.pbwd);
  int go = 1;
  if (factor) {   // X and W are complete: the forward pass read all rows of W
    const int cw = lane == 0 ? cnt + kDsPivotDone : lane == 1 ? cnt + kDsForwardDone : last;
    const int target = lane == 0 ? 1 : lane == 1 ? nfwd : 0;
    go = wait_lanes(a, cw, target, lane == 2 ? nlast : target, nx, sh);
    if (!go) return false;
  }
  const int nb = uni(tk.f.nb);
  const __amdgpu_buffer_rsrc_t X = buffer(fac + uni(tk.f.xo), 8 * np * np);
  const __amdgpu_buffer_rsrc_t W = buffer(fac + uni(tk.f.wo), 8 * nb * np);
  const int at = c < np ? 8 * (rg * np + c) : kNowhere;
  const int* xsrc = a->tab + uni(tk.f.xsrc);
  double w[NW], x[NX];
  int xs[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int r = tid + kThreads * q;
    xs[q] = r < n3 ? xsrc[r / 3] + r % 3 : -1;
  }
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    if (G * q < nb) w[q] = load1(W, at + 8 * G * np * q);
  }
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    if (G * q < np) x[q] = load1(X, at + 8 * G * np * q);
  }
  if (go == 1 && !wait_one(a, last, nlast, nx, sh)) return false;
  // zero on the padding rows, whose W is zero
#pragma unroll
  for (int q = 0; q < NB; ++q)
    if (tid + kThreads * q < nb) xb[tid + kThreads * q] = xs[q] >= 0 ? a->ws[xs[q]] : 0.0;
  for (int r = tid + kThreads * NB; r < nb; r += kThreads)
    xb[r] = r < n3 ? a->ws[xsrc[r / 3] + r % 3] : 0.0;
  if (tid < np) t[tid] = a->ws[tk.f.t + tid];
  fetch_next(nx);
  sync();
  double s = 0.0, u = 0.0;
#pragma unroll
  for (int q = 0; q < NX; ++q)
    if (G * q < np) s += x[q] * t[rg + G * q];
#pragma unroll
  for (int q = 0; q < NW; ++q)
    if (G * q < nb) u += w[q] * xb[rg + G * q];
#pragma unroll 8
  for (int r = G * NW; r < nb; r += G) u += load1(W, at + 8 * r * np) * xb[rg + r];
  part[rg * 33 + cl] = s - u;
  sync();
  if (tid < kDsBwdCols && c < np) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < G; ++q) v += part[q * 33 + cl];
    put(a->ws + tk.f.x + c, v);
    if (c < 3 * tk.f.p) a->sol[(size_t)(c % 3) * a->nv + a->tab[tk.f.verts + c / 3]] = v;
  }
  signal(a, cnt + kDsBackwardDone, -1, nx, sh);
  return true;
}

// The tables come through a device copy of DsArgs that every task reads anew: as kernel
// arguments their pointers would stay in scalar registers across the task loop, whose
// spills then cost vector registers in every task. (fac is not restrict: what it points to
// is written by other workgroups during the launch.)
__global__ void __launch_bounds__(kThreads, 4) k_ds_run(const DsArgs* __restrict__ args,
                                                        double* fac,
                                                        const DsTask* __restrict__ tasks,
                                                        int factor,
                                                        const int* __restrict__ left) {
  if (left) {   // a correction: nothing to do when every sheet is solved
    if (*left == 0) return;
  } else if (blockIdx.x == 0 && threadIdx.x < 2) {
    args->left[threadIdx.x] = 0;
  }
  extern __shared__ __align__(16) double lds[];
  __shared__ Shared sh;
  Next nx{tasks, factor, (int)blockIdx.x % kDsQueues, 0, 0, 0, 0, 0, 0};
  find_task(table(args), nx, true, sh);
#pragma unroll 1
  for (;;) {
    if (uni(sh.next[nx.slot]) < 0) {
      sync();
      find_task(table(args), nx, false, sh);
      if (uni(sh.next[nx.slot]) < 0) return;
    }
    const DsTask& tk = sh.rec[nx.slot];
    nx.slot ^= 1;
    const DsArgs* ap = args;
    asm volatile("" : "+s"(ap));
    const Table<DsArgs> a = table(ap);
    claim(a, nx);   // the next task's number travels while this one runs
    const int kind = uni(tk.kind);
    bool go = true;
    if (kind == kDsPivot) go = task_pivot(a, tk, nx, fac, lds, sh);
    else if (kind == kDsBorder) go = task_border(a, tk, nx, fac, lds, sh);
    else if (kind == kDsSchur) go = task_schur(a, tk, nx, fac, lds, sh);
    else if (kind == kDsForward) go = task_forward(a, tk, nx, factor != 0, fac, lds, sh);
    else go = task_backward(a, tk, nx, factor != 0, fac, lds, sh);
    if (!go) return;
  }
}

// x += dx of the sheets not accepted yet.
__global__ void __launch_bounds__(256) k_ds_add(DsArgs a, DsAccept o, const double* __restrict__ dx,
                                                const int* __restrict__ vert_inst) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= a.nv || o.done[vert_inst[i]]) return;
#pragma unroll
  for (int r = 0; r < 3; ++r) a.sol[(size_t)r * a.nv + i] += dx[(size_t)r * a.nv + i];
}

// True residual of the solution, 64 rows per workgroup (the four wavefronts take every
// fourth slot of the rows); the last workgroup of a sheet to finish adds the partial
// sums in order and accepts the solve when |b - A x| <= tol |b|. With o.again only the
// sheets not accepted before are looked at.
__global__ void __launch_bounds__(256) k_ds_resid(DsArgs a, DsAccept o,
                                                  const DsRows* __restrict__ tasks) {
  __shared__ double part[4][3][kDsResRows];
  __shared__ int s_last;
  const DsRows tk = tasks[blockIdx.x];
  const int inst = tk.sheet, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the next solve's counters, queue and abort flag start at zero
  for (int e = blockIdx.x * 256 + tid; e < o.clear_ints; e += gridDim.x * 256) a.count[e] = 0;
  if (o.again && o.done[inst]) return;   // every workgroup of the sheet
  const int end = o.inst_voff[inst] + o.inst_nv[inst];
  const int i = tk.row0 + lane, nv = a.nv;
  double y[3] = {0.0, 0.0, 0.0};
  if (i < end)
    for (int k = wave; k < a.maxnz; k += 4) {
      const int j = o.ell_col[k * nv + i];
      if (j < 0) continue;
      const double x0 = a.sol[j], x1 = a.sol[nv + j], x2 = a.sol[2 * nv + j];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double* A = a.A + (size_t)(k * 9 + 3 * r) * nv + i;
        y[r] += A[0] * x0 + A[nv] * x1 + A[2 * (size_t)nv] * x2;
      }
    }
#pragma unroll
  for (int r = 0; r < 3; ++r) part[wave][r][lane] = y[r];
  __syncthreads();
  const int w0 = o.inst_res0[inst], nw = o.inst_res0[inst + 1] - w0;
  if (wave == 0) {
    double rr = 0.0, bb = 0.0;
    if (i < end) {
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double b = a.rhs[(size_t)r * nv + i];
        const double e = b - (part[0][r][lane] + part[1][r][lane] + part[2][r][lane] +
                              part[3][r][lane]);
        if (o.res) o.res[(size_t)r * nv + i] = e;
        rr += e * e;
        bb += b * b;
      }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
      rr += __shfl_xor(rr, s);
      bb += __shfl_xor(bb, s);
    }
    if (lane == 0) {
      __hip_atomic_store(o.part + 2 * blockIdx.x, rr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(o.part + 2 * blockIdx.x + 1, bb, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      const int n = __hip_atomic_fetch_add(o.arrived + inst, 1, __ATOMIC_ACQ_REL,
                                           __HIP_MEMORY_SCOPE_AGENT);
      s_last = n == nw - 1;
    }
  }
  __syncthreads();
  if (!s_last || wave != 0) return;
  double rr = 0.0, bb = 0.0;
  for (int w = lane; w < nw; w += 64) {
    rr += __hip_atomic_load(o.part + 2 * (w0 + w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bb += __hip_atomic_load(o.part + 2 * (w0 + w) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    rr += __shfl_xor(rr, s);
    bb += __shfl_xor(bb, s);
  }
  if (lane != 0) return;
  __hip_atomic_store(o.arrived + inst, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool ok = isfinite(bb) && rr <= o.tol * o.tol * bb;   // NaN: false
  o.done[inst] = ok ? 1 : 0;
  if (!ok) __hip_atomic_fetch_add(o.left, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (ok) {
    if (o.iters) o.iters[inst] = bb > 0.0 ? 1 : 0;
    if (o.resid) o.resid[inst] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
  }
}

}  // namespace

hipError_t ds_prepare(int* blocks_per_cu) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ds_run),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           kLds * (int)sizeof(double));
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(
      blocks_per_cu, reinterpret_cast<const void*>(&k_ds_run), kThreads, kLds * sizeof(double));
}

void launch_ds_run(const DsArgs* args, double* fac, const DsTask* tasks, int ntasks, bool factor,
                   int grid, const int* left, hipStream_t st) {
  hipLaunchKernelGGL(k_ds_run, dim3(std::min(grid, ntasks)), dim3(kThreads), kLds * sizeof(double),
                     st, args, fac, tasks, factor ? 1 : 0, left);
}

void launch_ds_add(const DsArgs& a, const DsAccept& o, const double* dx, const int* vert_inst,
                   hipStream_t st) {
  hipLaunchKernelGGL(k_ds_add, dim3((a.nv + 255) / 256), dim3(256), 0, st, a, o, dx, vert_inst);
}

void launch_ds_resid(const DsArgs& a, const DsAccept& o, const DsRows* tasks, int ntasks,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_ds_resid, dim3(ntasks), dim3(256), 0, st, a, o, tasks);
}

}  // namespace phisft
