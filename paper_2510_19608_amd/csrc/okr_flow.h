// Load flow by prefix sums over depth-first labels: host tables and launches
// (kernels in okr_flow.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace okr {

// Where a tree's tables lie in an int array; form 0: the tree is too large.
struct FlowPlan {
  int n = 0, form = 0;     // 1: a node per thread, 2: phase by phase
  size_t end = 0, tour = 0;  // form 1: ends of the labels' subtrees; the tour
  size_t lab[3] = {}, ende[3] = {}, ptour[3] = {}, idx = 0;  // form 2, by phase: labels << 3 | phases, ends, tour; entries [3][n]
  int cnt[3] = {};           // nodes that have the phase
};

struct FlowArgs {
  const int* tab;         // the int array on the device
  const uint8_t* phase;   // by label
  const double2* z;       // [n][9] branch impedances, zero on absent phases
  const double2* Sload;   // [S][n][3] by the caller's ids
  double2 v0[3];
  double tol, vmin, vmax;
  int maxit;
  double2 *V, *J, *A;     // [S][n][3] by label (J: scratch of the second form)
  double* absV;
  int *iters, *status;
  const int* ext;         // label -> the caller's node id
  double2* Vext;          // voltages by the caller's ids, or null
  // the cumulative impedances, by one more block (levels of the tree)
  const int *parent, *lvl_off, *lvl_nodes;
  int nlev;
  double2* Zroot;
};

// An assignment to evaluate, by label: members of every cluster (CSR), every
// node's super-node; err [S].
struct FlowEval {
  const int *moff, *mem, *sup;
  double* err;
};

// Appends the tables of a tree given by label (subtree ends, phases).
FlowPlan flow_tables(int n, const int* end, const uint8_t* phase, std::vector<int>& out);
// Kernel attributes (before any capture).
hipError_t flow_prepare(const FlowPlan& p);
// Load flow of S snapshots and the cumulative impedances (form 1 or 2).
void flow_launch(const FlowPlan& p, const FlowArgs& a, int S, hipStream_t st);
// Load flow, fixed-current solve of the clusters' currents and largest errors
// (form 1; of a's outputs only the status and absV are written).
void flow_eval_launch(const FlowPlan& p, const FlowArgs& a, const FlowEval& e, int S, hipStream_t st);
// Voltages of the fixed currents I [S][n][3] by label (form 1 or 2).
void flow_fixed_launch(const FlowPlan& p, const int* tab, const uint8_t* phase, const double2* z, const double2* v0,
                       const double2* I, double2* J, double2* V, int S, hipStream_t st);

// Cumulative series impedance from the root, Zroot(v) = Zroot(parent) + z(v)
// (3x3 blocks, zero on absent phases), level by level; the impedance of the
// path between an ancestor s and r is Zroot(r) - Zroot(s).  One block.
__device__ __forceinline__ void zroot_block(int n, const int* __restrict__ parent, const int* __restrict__ lvl_off,
                                            const int* __restrict__ lvl_nodes, int nlev,
                                            const double2* __restrict__ z, double2* Zroot) {
  for (int e = threadIdx.x; e < 9; e += blockDim.x) Zroot[e] = make_double2(0.0, 0.0);  // node 0, level 0
  __syncthreads();
  for (int L = 1; L < nlev; ++L) {
    const int a = lvl_off[L], b = lvl_off[L + 1];
    for (int t = a * 9 + threadIdx.x; t < b * 9; t += blockDim.x) {
      const int v = lvl_nodes[t / 9], e = t % 9;
      const double2 up = Zroot[(size_t)parent[v] * 9 + e], zv = z[(size_t)v * 9 + e];
      Zroot[(size_t)v * 9 + e] = make_double2(up.x + zv.x, up.y + zv.y);
    }
    __threadfence_block();
    __syncthreads();
  }
}

}  // namespace okr
