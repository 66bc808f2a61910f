// direct.h -- the direct solver of the step matrix: elimination plan (host) and its
// device tables. See direct_prep.cpp (plan) and direct.hip (kernels).
#pragma once

#include <vector>

namespace phisft {

constexpr int kDsTile = 16;      // matrix-core tile: unknowns are padded to it
constexpr int kDsMaxPiv = 32;    // pivot vertices of a front at most (96 unknowns)
// A piece of at most this many vertices is not cut further, in sheets of at most
// kDsSmallSheet vertices and in larger ones. Small sheets are bound by the pivot sweeps on
// the chain, which small leaves shorten (48 against 24: 10x10 +6 %, 20x20 +3 %, 29x29 the
// same); large ones gain from fewer fronts (32x32 -3 %, 64x64 -6 to -9 %, 200x200 -2 %;
// 64 and more lose again there).
constexpr int kDsLeafSmall = 24, kDsLeaf = 48, kDsSmallSheet = 900;
constexpr int kDsMaxBorder = 4096;  // border unknowns of a front at most (LDS vectors)
constexpr int kDsSchurTile = 64;    // tile of the border update
constexpr int kDsRowTile = 32;      // border rows per task of W = B X
constexpr int kDsFwdRows = 64;      // border rows per task of the forward pass
constexpr int kDsBwdCols = 32;      // pivot columns per task of the backward pass
constexpr int kDsQueues = 8;        // task queues, one per die (XCD)
constexpr int kDsOneQueue = 512;     // with fewer factorisation tasks all are in one
constexpr int kDsResRows = 64;      // rows per workgroup of the residual

// One front: p pivot vertices eliminated together and the b later vertices they couple
// to (the border). Unknown 3 l + c is component c of local vertex l; local vertices are
// the pivots, then the border in elimination order. np, nb: 3 p and 3 b rounded up to 16,
// which also keeps every array of a front on cache lines of its own. Index tables are
// offsets into one int array (tab), vectors offsets into one workspace.
struct DsFront {
  int np, nb, p, b;
  int verts;                 // tab: vertex ids of the local vertices
  int nc, c0;                // children at kids[c0 .. c0 + nc)
  int kcnt[2];               // counters of the first two children
  int khead[2], kschur[2], kfwd[2];   // and their numbers of tasks
  int cnt;                   // the front's counters (kDs*Done)
  int pcnt, pbwd;            // the parent's counters (or -1) and number of backward tasks
  int nfwd;
  int gsrc;                  // tab: [k (p + b) + l] where local vertex l's part of child
                             // k's border vector starts, or -1
  int xsrc;                  // tab: where border vertex u's solution starts
  int alist, nalist;         // tab: entries of A in the pivot block: pairs (offset of the
                             // 3x3 block in A, column l << 16 | row i), i <= l < p
  int blist;                 // tab: per row tile r its entries (p <= l) are the pairs from
                             // tab[blist + r] up to tab[blist + r + 1]
  int t, g, x;               // pivot, border and solution vectors
  long long xo, wo;          // X [np][np] and W [nb][np] in the step's factor
  long long so, bo;          // Schur update [nb][nb] and border block [nb][np]
};

// A child of a front: tab[inv + l] is the child's border index of the front's local vertex
// l (or -1), tab[map + u] the front's local index of the child's border vertex u
// (increasing); the first q border vertices of the child are pivots of the front.
struct DsChild {
  int cnt, nhead, nschur, nfwd;   // the child's counters and numbers of tasks
  int q, inv, map;
  int nb;
  int g;                          // the child's border vector
  long long so;
};

// One unit of work of a front. a: row tile, chunk, or I << 16 | J. The record holds
// all that a task looks up before its first data (the front, its first two children and
// the index lists of its rows), so that a workgroup can fetch it during the task before:
// the chain of lookups task, front, child, list took 4 us of a Schur task's 12 us.
enum DsKind { kDsPivot = 0, kDsBorder, kDsSchur, kDsForward, kDsBackward };
struct alignas(16) DsTask {
  int kind, front, a;
  int lo, hi;            // border: entries of A, pairs tab[2 lo .. 2 hi)
  int pad[3];
  DsFront f;
  DsChild kid[2];
  // border indices in children 0 and 1 of the vertices of the task's rows (from vertex
  // row0 / 3 on; border, Schur, forward) and ...
  short row[2][24];
  // ... of its columns (Schur) or the pivots (forward), -1: none; pivot and border: the
  // local indices of the child's first border vertices (its q pivots of the front)
  short col[2][32];
  int pad2[4];
};
static_assert(sizeof(DsTask) == 512, "fetched by one wavefront, 8 bytes a lane");

// Residual rows of a sheet: from row0 on.
struct DsRows {
  int sheet, row0;
};

// Completion counters of a front: Schur tiles that hold a parent's pivots (tile rows 0 and
// 1: the "head"), all Schur tiles, pivot, forward and backward tasks, then the border row
// tiles of each group of kDsSchurTile rows.
enum DsCounter {
  kDsHeadDone = 0, kDsSchurDone, kDsPivotDone, kDsForwardDone, kDsBackwardDone, kDsRowsDone
};

// Words in which a workgroup's consecutive waits hand over their outcomes, in turn.
constexpr int kDsGoWords = 2;
constexpr int ds_next_word(int word) { return (word + 1) % kDsGoWords; }

// Elimination plan of all sheets of a handle. Fronts are sorted by level: a front's
// children are all on lower levels.
struct DsPlan {
  bool ok = false;
  std::vector<DsFront> fronts;
  std::vector<DsChild> kids;
  std::vector<int> tab;
  std::vector<int> level0;   // [levels + 1] front ranges
  // tasks in an order in which every task comes after those it waits for: factorisation
  // with both passes of one right-hand side, and the two passes alone
  std::vector<DsTask> factor_tasks, solve_tasks;
  // queue of each task: of the workgroups of one die, whose cache then holds what the
  // tasks of a subtree share
  std::vector<unsigned char> factor_queue, solve_queue;
  std::vector<DsRows> res_tasks;   // of the residual
  std::vector<int> res0;           // [sheets + 1]
  long long factor_doubles = 0, work_doubles = 0;
  int counters = 0;
  int max_np = 0, max_nb = 0;
  int levels() const { return (int)level0.size() - 1; }
  // Frees the lists and tables (512 bytes a task: 52 MB of a 200x200 sheet).
  void drop_tables() {
    const long long f = factor_doubles, w = work_doubles;
    *this = DsPlan{};
    ok = true;
    factor_doubles = f;
    work_doubles = w;
  }
};

// xr: rest positions [nv][3] in the internal vertex order; ell_col, inst_voff and inst_nv
// as in HostLayout. plan.ok is false when a front's border exceeds kDsMaxBorder,
// or when workspace and one factor exceed max_doubles (0: no limit; found before the tables
// and tasks are built).
void build_direct_plan(int nv, int maxnz, const std::vector<int>& ell_col,
                       const std::vector<int>& inst_voff, const std::vector<int>& inst_nv,
                       const std::vector<double>& xr, DsPlan& plan,
                       double max_doubles = 0.0);

}  // namespace phisft
