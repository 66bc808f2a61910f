// direct_kernels.h -- launchers of the direct solver (definitions in direct.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "direct.h"

namespace phisft {

// Device tables, workspace and operands of one factorisation or solve.
struct DsArgs {
  const DsChild* kid;
  const int* tab;
  int nv, maxnz;
  const double* A;     // [maxnz][9][nv] step matrix
  double* ws;          // vectors, Schur updates and border blocks
  const double* rhs;   // [3][nv]
  double* sol;         // [3][nv]
  int* count;          // counters, queue and abort flag; zero before a launch
  int* queue;          // [kDsQueues] heads, kDsLine ints apart
  int* abort_flag;
  int* left;           // [2] set to zero by a launch that is not a correction
  int q0[2][kDsQueues + 1];   // the queues' tasks in the lists: passes alone, factorisation
};

constexpr int kDsLine = 32;   // ints of a cache line

// Acceptance of a solve per sheet: done[inst] = 1 when |b - A x| <= tol |b| (with one
// iteration recorded), else 0: the iterative solver then takes the sheet. The counters of
// the next launch are cleared on the way.
struct DsAccept {
  const int* ell_col;
  const int* inst_voff;
  const int* inst_nv;
  const int* inst_res0;   // [sheets + 1] residual workgroups of each sheet
  double tol;
  double* part;           // [workgroups][2]
  int* arrived;           // [sheets], zero between launches
  int clear_ints;         // ints from DsArgs::count
  int* done;              // [sheets]
  int* left;              // counts the sheets not accepted; zero before
  double* res;            // [3][nv] receives b - A x, or nullptr
  int again;              // 1: leave the sheets accepted before alone
  int* iters;             // [sheets] or nullptr
  double* resid;          // [sheets] or nullptr
};

hipError_t ds_prepare(int* blocks_per_cu);
// Runs a list of ntasks tasks, queue after queue, on at most `grid` workgroups; args:
// device copy of DsArgs; fac: X and W of every front; factor: the list factorises. With
// `left` it is a correction: nothing runs when that word is zero.
void launch_ds_run(const DsArgs* args, double* fac, const DsTask* tasks, int ntasks, bool factor,
                   int grid, const int* left, hipStream_t st);
void launch_ds_add(const DsArgs& a, const DsAccept& o, const double* dx, const int* vert_inst,
                   hipStream_t st);
void launch_ds_resid(const DsArgs& a, const DsAccept& o, const DsRows* tasks, int ntasks,
                     hipStream_t st);

}  // namespace phisft
