// Greedy single-move reduction search (Algorithm 1, Section IV) and the
// evaluation of a fixed reduction over many scenarios (Section VI), on
// gfx950: kernels and the C ABI of include/okr_greedy.h.
//
// Design.  The full network is radial with the slack as source, so with the
// currents fixed its solution is V = V0 - sum_j Zcp(., j) I_j, where Zcp(y, j)
// is the series impedance of the common part of the root paths of y and j,
// i.e. Zroot(lca(y, j)).  Moving the aggregated load current J of super-node
// r to super-node s therefore changes node y's voltage by
//     dV_y = (Zroot(lca(y, r)) - Zroot(lca(y, s))) J,
// which is nonzero exactly on the subtrees of w = lca(r, s)'s children
// towards r and towards s.
// Nodes are labelled by their position in a depth-first order, so a subtree is
// an interval of labels and the lowest common ancestor of u < v is the
// smallest parent over (u, v]: one lookup in a sparse table.
// A cluster enters only through the smallest and largest |V^| of its members
// per phase and scenario: its largest member error against magnitude m is
// max(hi - m, m - lo), the same number as the maximum over the members
// (rounding is monotone and |a - b| symmetric), so no kernel walks members and
// merging two clusters takes their extremes.  The super-nodes are kept as a
// dense list in label order, with every label's rank in it: an interval of
// labels is an interval of the list, and the work of a move shrinks with the
// clusters that are left.
// Every move is two launches: k_greedy_score scores all candidates (both
// directions of the edge above one cluster together), k_greedy_apply settles
// the move in every block alike and writes the next list, voltages and errors.
// A search starts from the exact fixed-current solve, which also serves the
// evaluation of a given assignment.

#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/okr_greedy.h"
#include "okr_device.h"
#include "okr_flow.h"
#include "okr_internal.h"

namespace okr {

__global__ void k_branch_z(int, int, const uint8_t*, const int*, const int*, const int*, const double2*, const double2*,
                           double2*, int*, State);
__global__ void k_powerflow(int, const int*, const uint8_t*, const int*, const int*, int, const int*, const int*,
                            const double2*, const double2*, double2, double2, double2, double, int, double, double,
                            double2*, double2*, double2*, double*, int*, int*, const int*, double2*);
__global__ void k_from_vhat(int, int, const uint8_t*, const double2*, const double2*, double, double, double2*,
                            double*, int*, const int*, double2*);
__global__ void k_zroot(int, const int*, const int*, const int*, int, const double2*, double2*);

struct GState {
  int iter;  // moves applied
  int done;  // no feasible candidate left
  int s;     // the last move's super-node and the labels whose voltages it changed
  int a0, a1, b0, b1;
};

struct GStep {  // layout of okr_greedy_step
  int cand, s, r, ambiguous, n_cand, n_feasible;
  double smice, emax;
};

constexpr int kGreedyThreads = 256;
constexpr int kGreedyPickThreads = 1024;
constexpr int kGreedyMaxS = 64;      // scenarios of a search (moved currents staged in LDS)
constexpr int kGreedyMaxN = 12288;   // nodes that an incremental search accepts (its counts' 20 bits would hold 2^19)
constexpr int kGreedyFullSN = 6144;  // S x n up to which every candidate sums every cluster ...
constexpr int kGreedyFullSNL = 7680;  // ... and S x n + 3 x levels

// Lowest common ancestors of labels (depth-first positions): the smallest
// (parent, last position) over power-of-two runs of labels, level k at
// st[k * n].  Every label in (u, v] lies below lca(u, v), and the child of it
// that leads to v is the last of them whose parent it is.
struct LcaTab {
  const unsigned long long* st;
  int n;
  __device__ __forceinline__ unsigned long long key(int lo, int hi) const {  // over (lo, hi], lo < hi
    const int k = 31 - __clz(hi - lo);
    const unsigned long long x = st[(size_t)k * n + lo + 1], y = st[(size_t)k * n + hi - (1 << k) + 1];
    return x < y ? x : y;
  }
  static __device__ __forceinline__ int parent_of(unsigned long long k) { return (int)(k >> 32); }
  static __device__ __forceinline__ int child_of(unsigned long long k) { return (int)(0xffffffffu - (unsigned)k); }
  __device__ __forceinline__ int lca(int u, int v) const { return u == v ? u : parent_of(key(min(u, v), max(u, v))); }
};

// A cluster of the list: its super-node, its topmost node, the super-node of
// the cluster above it, and the phases of the two super-nodes (u's in bits
// 0-2, b's in bits 8-10).
struct GClus {
  int u, top, b, ph;
};

// The candidate pair of the edge above a cluster: super-nodes a (below) and b
// (above), w = lca(a, b), and the label intervals of the subtrees of w's
// children towards a and towards b (the latter empty when b is w).
struct GEdge {
  int a, b, w, ja, jb;  // ja, jb: ranks of a and b
  int a0, a1, b0, b1;
  int ea, eb;  // ends of a's and b's own subtrees
};

// Rescored clusters of a candidate pair: their old errors, their new errors
// and the largest one per direction (0: the cluster below moves up, 1: the one
// above moves down).
struct GPart {
  double olds, n0, n1, e0, e1;
};

// Scoring results of one block of candidates.
struct GBlk {
  double mn, snd;          // smallest SMICE, and the smallest of the others
  unsigned long long key;  // mn's candidate: id << 32 | 2 * rank + direction
  unsigned long long cnt;  // candidates, feasible ones << 20, ones with an error within amb of e_bar << 40
};

// State of the search.  Arrays with two copies are written for the next
// iteration while the current one is read (iteration parity).
struct GreedyState {
  GState* gs[2];
  GClus* cl[2];       // [n] the list of clusters, by label of the super-node
  int2* rank[2];      // [n] super-nodes below a label, and below the end of its subtree
  double* mice[2];    // [S][n] every cluster's largest error, by rank
  double* arr[2];     // [n] its maximum over scenarios
  double* bmax[2];    // maxima of arr over runs of 64 ranks
  double* bsum[2];    // sums of mice over runs of 64 ranks and all scenarios
  double* ext;        // [S][n][6] by label: smallest and largest |V^| of the cluster's members, 3 phases each
  GEdge* edge;        // [n] by rank
  GPart* part;        // [n] by label of the cluster below the edge
  double *sm, *em;    // [2n] SMICE and largest error, by rank and direction
  GBlk* blk;          // [n]
  int* sup;           // [n]
  double2 *V, *I;     // [S][n][3] voltages (current at super-nodes) and aggregated currents
};

// Largest error of a cluster against magnitude m on one phase: the members'
// largest |a - m| (the extremes are +inf and -inf where no member has the
// phase, which never wins).
__device__ __forceinline__ double ext_err(double e, double lo, double hi, double m) {
  return fmax(e, fmax(hi - m, m - lo));
}

// Impedance change of an affected super-node: Zroot(a) - Zroot(b).
struct MoveDelta {
  double2 dZ[9];
  __device__ __forceinline__ void between(const double2* Zr, int a, int b) {
    const double2* Za = Zr + (size_t)a * 9;
    const double2* Zb = Zr + (size_t)b * 9;
#pragma unroll
    for (int q = 0; q < 9; ++q) dZ[q] = csub(Za[q], Zb[q]);
  }
  __device__ __forceinline__ double2 dv(int p, const double2* J) const {
    return cadd(cadd(cmul(dZ[p * 3], J[0]), cmul(dZ[p * 3 + 1], J[1])), cmul(dZ[p * 3 + 2], J[2]));
  }
};

// Fixed-current solve of one scenario on the radial network: branch currents
// by subtree sums of the load currents I (deepest level first), then
// V(x) = V(parent) - z_x Ib(x) level by level from the slack (V0).  One block.
__device__ void sweep_block(int n, const int* parent, const uint8_t* phase, const int* lvl_off,
                            const int* lvl_nodes, int nlev, const int* ch_off, const int* ch, const double2* z,
                            const double2 (&v0)[3], const double2* I, double2* Ib, double2* V) {
  for (int q = threadIdx.x; q < n * 3; q += blockDim.x) Ib[q] = I[q];
  __syncthreads();
  for (int lev = nlev - 2; lev >= 0; --lev) {
    for (int q = lvl_off[lev] + threadIdx.x; q < lvl_off[lev + 1]; q += blockDim.x) {
      const int i = lvl_nodes[q];
      double2 s0 = Ib[i * 3], s1 = Ib[i * 3 + 1], s2 = Ib[i * 3 + 2];
      for (int e = ch_off[i]; e < ch_off[i + 1]; ++e) {
        const int c = ch[e];
        s0 = cadd(s0, Ib[c * 3]);
        s1 = cadd(s1, Ib[c * 3 + 1]);
        s2 = cadd(s2, Ib[c * 3 + 2]);
      }
      Ib[i * 3] = s0;
      Ib[i * 3 + 1] = s1;
      Ib[i * 3 + 2] = s2;
    }
    __syncthreads();
  }
  if (threadIdx.x < 3) V[threadIdx.x] = (phase[0] >> threadIdx.x & 1u) ? v0[threadIdx.x] : make_double2(0.0, 0.0);
  __syncthreads();
  for (int lev = 1; lev < nlev; ++lev) {
    for (int q = lvl_off[lev] + threadIdx.x; q < lvl_off[lev + 1]; q += blockDim.x) {
      const int i = lvl_nodes[q], pv = parent[i];
      const double2* zi = z + (size_t)i * 9;
      const double2 j0 = Ib[i * 3], j1 = Ib[i * 3 + 1], j2 = Ib[i * 3 + 2];
      for (int p = 0; p < 3; ++p) {
        double2 v = make_double2(0.0, 0.0);
        if (phase[i] >> p & 1u) {
          const double2 d = cadd(cadd(cmul(zi[p * 3], j0), cmul(zi[p * 3 + 1], j1)), cmul(zi[p * 3 + 2], j2));
          v = csub(V[pv * 3 + p], d);
        }
        V[i * 3 + p] = v;
      }
    }
    __syncthreads();
  }
}

// Start of the search: every node its own super-node, I = the load currents.
__global__ void k_greedy_init(int n, int S, const double2* __restrict__ A, double2* __restrict__ Iagg,
                              int* __restrict__ sup, GState* __restrict__ gs) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < (size_t)S * n * 3) Iagg[t] = A[t];
  if (t < (size_t)n) sup[t] = (int)t;
  if (t == 0) *gs = GState{0, 0, 0, 0, n, 0, 0};  // (every candidate is still to be scored)
}

// Fixed-current solve of every scenario (one block each) from Iagg.
__global__ __launch_bounds__(kGreedyThreads) void k_greedy_sweep(
    int n, const int* __restrict__ parent, const uint8_t* __restrict__ phase, const int* __restrict__ lvl_off,
    const int* __restrict__ lvl_nodes, int nlev, const int* __restrict__ ch_off, const int* __restrict__ ch,
    const double2* __restrict__ z, double2 v0a, double2 v0b, double2 v0c, const double2* __restrict__ Iagg,
    double2* __restrict__ Ib, double2* __restrict__ V) {
  const size_t base = (size_t)blockIdx.x * n * 3;
  const double2 v0[3] = {v0a, v0b, v0c};
  sweep_block(n, parent, phase, lvl_off, lvl_nodes, nlev, ch_off, ch, z, v0, Iagg + base, Ib + base, V + base);
}

// Maxima and sums over a wave's run of 64 ranks (summed in a fixed tree).
__device__ __forceinline__ void run_totals(double mx, double sum, double* bmax, double* bsum) {
  for (int o = 32; o > 0; o >>= 1) {
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    sum += __shfl_xor(sum, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    *bmax = mx;
    *bsum = sum;
  }
}

// The search's starting point: every node a cluster (one thread per node).
__global__ __launch_bounds__(kGreedyThreads) void k_greedy_prep(int n, int S, const int* __restrict__ parent,
                                                                const int* __restrict__ end,
                                                                const uint8_t* __restrict__ phase,
                                                                const double* __restrict__ absV, GreedyState G) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) G.rank[0][t] = make_int2(t, end[t]);
  double mx = 0.0, sum = 0.0;
  if (t < n) {
    const int b = t > 0 ? parent[t] : 0;
    const unsigned ph = phase[t];
    G.cl[0][t] = GClus{t, t, b, (int)(ph | (unsigned)phase[b] << 8)};
    for (int l = 0; l < S; ++l) {
      const size_t at = (size_t)l * n + t;
      double e = 0.0;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const bool on = ph >> p & 1u;
        const double a = absV[at * 3 + p], lo = on ? a : INFINITY, hi = on ? a : -INFINITY;
        G.ext[at * 6 + p] = lo;
        G.ext[at * 6 + 3 + p] = hi;
        e = ext_err(e, lo, hi, sqrt(cabs2(G.V[at * 3 + p])));
      }
      G.mice[0][at] = e;
      mx = fmax(mx, e);
      sum += e;
    }
    G.arr[0][t] = mx;
  }
  if (t - (int)(threadIdx.x & 63) < n) run_totals(mx, sum, G.bmax[0] + (t >> 6), G.bsum[0] + (t >> 6));
}

// Scores of every candidate: SMICE (+inf when infeasible) and the largest error
// (-1 when the direction is not a candidate), by rank of the cluster below the
// edge and direction.  With w = lca(a, b), voltages change exactly on the
// subtrees of w's children towards a and b, so only the clusters whose
// super-node lies there and the merged cluster (a's or b's) have a new error;
// their sums stay as they are until a move reaches those subtrees, a or b, and
// only then are they formed again.  In a's (b's) own subtree the voltage change
// is the same everywhere and stands in LDS for up to kGreedyDv scenarios.
// FULL: a block of 4 waves per edge adds every other cluster's present error.
// Otherwise SMICE = (total - old errors of the changed clusters) + their new
// ones, and the largest error takes the unchanged clusters from the maxima of
// runs of 64 ranks and from the positions of the runs that hold an end of an
// interval, a or b; a block of 8 waves takes 8 edges, one per wave, and waves
// share those with more than kGreedyWaveL clusters to score again.  Edges near
// the root have the long intervals and neighbouring ranks: a block's 8 edges
// lie a grid's width apart, which also leaves one edge per block when few are
// left.
// Bound by latency: eight dependent loads, the rounds over the longest interval
// and instruction fetch, so the rescoring stands in the code once.  Per launch,
// 2 scenarios: 5591 nodes 168 us as one block per candidate that walked nodes
// and members; 33 with cluster extremes, the list and both directions of an
// edge together; 20 (28 at the first moves, 12 at the last) with the sums that
// stand and the common voltage changes.  1000 nodes, FULL: 22, 11, 9.5.
// 4 edges per block 22 us, 16 24; one wave alone up to 32, 128 or 256 clusters
// within 4%.
constexpr int kGreedyEdges = 8;   // edges per block (incremental form)
constexpr int kGreedyWaveL = 64;  // clusters that one wave scores alone
constexpr int kGreedyDv = 8;       // scenarios whose common voltage changes are kept in LDS

template <bool FULL>
__global__ __launch_bounds__(FULL ? kGreedyThreads : kGreedyEdges * 64) void k_greedy_score(
    int n, int S, int cur, LcaTab T, const int* __restrict__ end, const int* __restrict__ label_id,
    const double2* __restrict__ Zr, double e_bar, double amb, GreedyState G) {
  constexpr int NW = FULL ? kGreedyThreads / 64 : kGreedyEdges, NE = FULL ? 1 : kGreedyEdges;
  __shared__ GEdge s_edge[NE];
  __shared__ int4 s_rank[NE];
  __shared__ int s_todo[NE];
  __shared__ GPart s_part[NE][NW];
  __shared__ double2 s_dv[NE][2][kGreedyDv][2][3];  // side, scenario, direction, phase
  __shared__ double s_out[NW], s_um[NW];
  __shared__ double s_v[2 * NE];
  __shared__ unsigned long long s_key[2 * NE], s_cnt[2 * NE];
  const GClus* __restrict__ cl = G.cl[cur];
  const double* __restrict__ mice = G.mice[cur];
  const double* __restrict__ ext = G.ext;
  const double2* __restrict__ V = G.V;
  const double2* __restrict__ I = G.I;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int me = FULL ? 0 : wv, j = 1 + me * (int)gridDim.x + (int)blockIdx.x;
  const GState st = *G.gs[cur];
  const GClus c = cl[j < n ? j : 0];
  const int m = n - st.iter;
  if (st.done || (int)blockIdx.x >= m - 1) return;
  GEdge E{};
  int4 R = make_int4(0, 0, 0, 0);  // the intervals' ranks
  bool d0 = false, d1 = false;
  unsigned id = 0;
  int todo = 0;  // 1: this wave scores the edge alone, 2: every wave, 3: its sums stand
  if (j < m) {
    const unsigned pa = c.ph & 7u, pb = (unsigned)c.ph >> 8;
    d0 = !(pa & ~pb);
    d1 = c.b != 0 && !(pb & ~pa);
  }
  const bool on = d0 || d1;
  if (on) {
    const int2* __restrict__ rank = G.rank[cur];
    id = 2u * (unsigned)label_id[c.top];
    E.a = c.u;
    E.b = c.b;
    E.ja = j;
    E.jb = rank[E.b].x;
    E.ea = end[E.a];
    E.eb = end[E.b];
    const int near = min(E.a, E.b);
    const unsigned long long k = T.key(near, max(E.a, E.b));
    E.w = LcaTab::parent_of(k);
    const int far = LcaTab::child_of(k);
    // a lies strictly below w; b may be w
    const int other = near != E.w ? LcaTab::child_of(T.key(E.w, near)) : -1;
    E.a0 = E.a > E.b ? far : other;
    E.b0 = E.a > E.b ? other : far;
    const int2 ra = rank[E.a0];
    E.a1 = end[E.a0];
    R.x = ra.x;
    R.y = ra.y;
    if (E.b0 >= 0) {
      const int2 rb = rank[E.b0];
      E.b1 = end[E.b0];
      R.z = rb.x;
      R.w = rb.y;
    } else {
      E.b0 = 0;
    }
    const bool hit = (E.a0 < st.a1 && st.a0 < E.a1) || (E.a0 < st.b1 && st.b0 < E.a1) ||
                     (E.b0 < st.a1 && st.a0 < E.b1) || (E.b0 < st.b1 && st.b0 < E.b1);
    todo = !hit && E.a != st.s && E.b != st.s ? 3 : FULL || (R.y - R.x) + (R.w - R.z) > kGreedyWaveL ? 2 : 1;
    if (todo != 3 && S <= kGreedyDv)
      for (int q = FULL ? tid : lane; q < 12 * S; q += FULL ? kGreedyThreads : 64) {
        const int p = q % 3, d = q / 3 & 1, l = (q / 6) % S, b = q / (6 * S);
        const double2* Za = Zr + (size_t)(b ? E.w : E.a) * 9 + p * 3;
        const double2* Zb = Zr + (size_t)(b ? E.b : E.w) * 9 + p * 3;
        const double2* J = I + ((size_t)l * n + (d ? E.b : E.a)) * 3;
        s_dv[me][b][l][d][p] = cadd(cadd(cmul(csub(Za[0], Zb[0]), J[0]), cmul(csub(Za[1], Zb[1]), J[1])),
                                    cmul(csub(Za[2], Zb[2]), J[2]));
      }
  }
  // the unchanged clusters: FULL their sum, else the total to take the changed
  // ones' old errors from, and their largest error
  double um = 0.0, out = 0.0;
  if (on && FULL) {
    int l = tid / m, q = tid - l * m;
    const int dl = kGreedyThreads / m, dq = kGreedyThreads - dl * m;
    while (l < S) {
      if (!(R.x <= q && q < R.y) && !(R.z <= q && q < R.w) && q != E.jb) {
        const double e = mice[(size_t)l * n + q];
        out += e;
        um = fmax(um, e);
      }
      l += dl;
      q += dq;
      if (q >= m) {
        q -= m;
        ++l;
      }
    }
  } else if (on) {
    const int nruns = (m + 63) >> 6;
    for (int k = lane; k < nruns; k += 64) {
      const int lo = k * 64, hi = lo + 64;
      const bool touch = (lo <= E.ja && E.ja < hi) || (lo <= E.jb && E.jb < hi) || (lo < R.y && R.x < hi) ||
                         (lo < R.w && R.z < hi);
      if (!touch) um = fmax(um, G.bmax[cur][k]);
      out += G.bsum[cur][k];
    }
    // a touched run holds a, b or an end of an interval, or lies wholly inside
    // one (a run named twice gives the same maximum)
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const int at = k == 0 ? E.ja : k == 1 ? E.jb : k == 2 ? R.x : k == 3 ? R.y - 1 : k == 4 ? R.z : R.w - 1;
      const int q = (at & ~63) + lane;
      if (at >= 0 && q < m && q != E.ja && q != E.jb && !(R.x <= q && q < R.y) && !(R.z <= q && q < R.w))
        um = fmax(um, G.arr[cur][q]);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    out += __shfl_xor(out, o, 64);
    um = fmax(um, __shfl_xor(um, o, 64));
  }
  if (lane == 0) {
    if (FULL) {
      s_out[wv] = out;
      s_um[wv] = um;
    }
    if (!FULL || wv == 0) {
      s_edge[me] = E;
      s_rank[me] = R;
      s_todo[me] = todo;
    }
  }
  __syncthreads();
  // round -1: the wave's own edge; round h: edge h by every wave
  for (int h = FULL ? 0 : -1; h < NE; ++h) {
    const int x = h < 0 ? me : h;
    if (__builtin_amdgcn_readfirstlane(s_todo[x]) != (h < 0 ? 1 : 2)) continue;
    const GEdge F = s_edge[x];
    const int4 r = s_rank[x];
    const int stride = h < 0 ? 64 : NW * 64, first = h < 0 ? lane : tid;
    // clusters of the two intervals, and b's when it is w; an item per cluster and scenario
    const int L1 = r.y - r.x, L2 = r.w - r.z, L = L1 + max(L2, 1);
    GPart P{0.0, 0.0, 0.0, 0.0, 0.0};
    int l = first / L, q = first - l * L;
    const int dl = stride / L, dq = stride - dl * L;
    while (l < S) {
      const bool inA = q < L1;
      const int k = inA ? r.x + q : L2 > 0 ? r.z + (q - L1) : F.jb;
      const int u = cl[k].u;
      const size_t at = (size_t)l * n + u;
      const bool isA = k == F.ja, isB = k == F.jb;
      const size_t mt = (size_t)l * n + (isA ? F.b : isB ? F.a : u);  // the cluster merged with u's
      double2 v[3], v0[3], v1[3];
      double lo[3], hi[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        v[p] = V[at * 3 + p];
        lo[p] = fmin(ext[at * 6 + p], ext[mt * 6 + p]);
        hi[p] = fmax(ext[at * 6 + 3 + p], ext[mt * 6 + 3 + p]);
      }
      P.olds += mice[(size_t)l * n + k];
      if (S <= kGreedyDv && (inA ? F.a <= u && u < F.ea : F.b <= u && u < F.eb)) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          v0[p] = s_dv[x][!inA][l][0][p];
          v1[p] = s_dv[x][!inA][l][1][p];
        }
      } else {
        // towards a, lca(u, b) = w; towards b, lca(u, a) = w
        const int y = T.lca(u, inA ? F.a : F.b);
        MoveDelta md;
        md.between(Zr, inA ? y : F.w, inA ? F.w : y);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          v0[p] = md.dv(p, I + ((size_t)l * n + F.a) * 3);
          v1[p] = md.dv(p, I + ((size_t)l * n + F.b) * 3);
        }
      }
      double x0 = 0.0, x1 = 0.0;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        x0 = ext_err(x0, lo[p], hi[p], sqrt(cabs2(cadd(v[p], v0[p]))));
        x1 = ext_err(x1, lo[p], hi[p], sqrt(cabs2(csub(v[p], v1[p]))));
      }
      // a's cluster is gone when it moves up, b's when it moves down
      if (isA) x0 = 0.0;
      if (isB) x1 = 0.0;
      P.n0 += x0;
      P.n1 += x1;
      P.e0 = fmax(P.e0, x0);
      P.e1 = fmax(P.e1, x1);
      l += dl;
      q += dq;
      if (q >= L) {
        q -= L;
        ++l;
      }
    }
    for (int o = 32; o > 0; o >>= 1) {
      P.olds += __shfl_xor(P.olds, o, 64);
      P.n0 += __shfl_xor(P.n0, o, 64);
      P.n1 += __shfl_xor(P.n1, o, 64);
      P.e0 = fmax(P.e0, __shfl_xor(P.e0, o, 64));
      P.e1 = fmax(P.e1, __shfl_xor(P.e1, o, 64));
    }
    if (lane == 0) s_part[x][h < 0 ? 0 : wv] = P;
  }
  __syncthreads();
  if (wv < NE && lane == 0) {
    double v0 = INFINITY, v1 = INFINITY;
    unsigned near = 0;
    if (on) {
      GPart P = todo == 3 ? G.part[E.a] : s_part[me][0];
      if (todo == 2)  // the waves' parts, in order
        for (int k = 1; k < NW; ++k) {
          const GPart Q = s_part[me][k];
          P.olds += Q.olds;
          P.n0 += Q.n0;
          P.n1 += Q.n1;
          P.e0 = fmax(P.e0, Q.e0);
          P.e1 = fmax(P.e1, Q.e1);
        }
      if (todo != 3) G.part[E.a] = P;
      if (FULL) {
        for (int k = 1; k < NW; ++k) {
          out += s_out[k];
          um = fmax(um, s_um[k]);
        }
      } else {
        out -= P.olds;
      }
      P.e0 = fmax(P.e0, um);
      P.e1 = fmax(P.e1, um);
      if (d0 && P.e0 <= e_bar) v0 = out + P.n0;
      if (d1 && P.e1 <= e_bar) v1 = out + P.n1;
      near = (d0 && fabs(P.e0 - e_bar) <= amb) + (d1 && fabs(P.e1 - e_bar) <= amb);
      G.em[2 * j] = d0 ? P.e0 : -1.0;
      G.em[2 * j + 1] = d1 ? P.e1 : -1.0;
      G.edge[j] = E;
    }
    if (j < m) {
      G.sm[2 * j] = v0;
      G.sm[2 * j + 1] = v1;
    }
    s_v[2 * me] = v0;
    s_v[2 * me + 1] = v1;
    s_key[2 * me] = (unsigned long long)id << 32 | (unsigned)(2 * j);
    s_key[2 * me + 1] = (unsigned long long)(id + 1) << 32 | (unsigned)(2 * j + 1);
    s_cnt[2 * me] = (unsigned)d0 + (unsigned)d1;
    s_cnt[2 * me + 1] = (unsigned long long)((v0 < INFINITY) + (v1 < INFINITY)) << 20 | (unsigned long long)near << 40;
  }
  __syncthreads();
  if (wv == 0) {
    const int k = min(lane, 2 * NE - 1);
    double mn = s_v[k], snd = INFINITY;
    unsigned long long key = s_key[k], cnt = lane < 2 * NE ? s_cnt[k] : 0ull;
    for (int o = NE; o > 0; o >>= 1) {
      const double om = __shfl_xor(mn, o, 64), os = __shfl_xor(snd, o, 64);
      const unsigned long long ok = __shfl_xor(key, o, 64);
      snd = fmin(fmin(snd, os), fmax(mn, om));
      if (om < mn || (om == mn && ok < key)) key = ok;
      mn = fmin(mn, om);
      cnt += __shfl_xor(cnt, o, 64);
    }
    if (lane == 0) G.blk[blockIdx.x] = GBlk{mn, snd, key, cnt};
  }
}

// The iteration's move: the smallest SMICE among feasible candidates, ties
// within tie_tol to the lowest id.  Every block settles it alike from the
// scoring blocks' records (a record's candidates are opened only when its
// second value reaches the tie threshold); then one thread per remaining
// cluster writes the next list, moves its super-node's voltage when the move
// reaches it (the expression the scoring evaluated) and its error.  What other
// blocks still read is never written: the list, ranks and errors have two
// copies, r's current is left as it is (r is no super-node any more).  With no
// feasible candidate the search is marked done.
// Bound by latency; what does not depend on the move is loaded before it is
// settled.  5591 nodes 8.9 us, 1000 nodes 8.6 (79 and 14.9 as one block that
// walked every node and rebuilt every cluster's members).
__global__ __launch_bounds__(kGreedyPickThreads) void k_greedy_apply(
    int n, int S, int cur, int edges, LcaTab T, const int* __restrict__ end, const int* __restrict__ label_id,
    const double2* __restrict__ Zr, double tie, double amb, GStep* __restrict__ steps, GreedyState G) {
  constexpr int NW = kGreedyPickThreads / 64;
  __shared__ double s_mn[NW];
  __shared__ unsigned long long s_cnt[NW], s_win[NW];
  __shared__ double2 J[kGreedyMaxS * 3];
  const int nxt = 1 - cur, tid = threadIdx.x, lane = tid & 63, t = blockIdx.x * kGreedyPickThreads + tid;
  const int grid = (n - 2) / edges + 1;  // scoring blocks
  const GState st = *G.gs[cur];
  const int tc = min(t, n - 1), t1 = min(t + 1, n - 1);
  const int2 rk = G.rank[cur][tc];
  const int te = end[tc], sup = G.sup[tc];
  const GClus c0 = G.cl[cur][tc], c1 = G.cl[cur][t1];
  if (st.done) {
    if (t == 0) *G.gs[nxt] = GState{st.iter, 1, 0, 0, 0, 0, 0};
    return;
  }
  const int m = n - st.iter, nb = min(grid, m - 1);
  double mn = INFINITY;
  unsigned long long cnt = 0;
  GBlk B{INFINITY, INFINITY, 0, 0};
  for (int b = tid; b < nb; b += kGreedyPickThreads) {
    B = G.blk[b];
    mn = fmin(mn, B.mn);
    cnt += B.cnt;
  }
  for (int o = 32; o > 0; o >>= 1) {
    mn = fmin(mn, __shfl_xor(mn, o, 64));
    cnt += __shfl_xor(cnt, o, 64);
  }
  if (lane == 0) {
    s_mn[tid >> 6] = mn;
    s_cnt[tid >> 6] = cnt;
  }
  __syncthreads();
  mn = s_mn[lane & (NW - 1)];
  cnt = s_cnt[lane & (NW - 1)];
  for (int o = NW / 2; o > 0; o >>= 1) {
    mn = fmin(mn, __shfl_xor(mn, o, 64));
    cnt += __shfl_xor(cnt, o, 64);
  }
  if (!(mn < INFINITY)) {
    if (t == 0) *G.gs[nxt] = GState{st.iter, 1, 0, 0, 0, 0, 0};
    return;
  }
  const double thr = mn + tie;
  unsigned long long win = ~0ull;  // smallest key
  bool near = false;
  for (int b = tid; b < nb; b += kGreedyPickThreads) {
    if (nb > kGreedyPickThreads) B = G.blk[b];
    if (!(B.mn <= thr + 2.0 * amb)) continue;
    near |= fabs(B.mn - thr) <= amb;
    if (B.mn <= thr && B.key < win) win = B.key;
    if (!(B.snd <= thr + 2.0 * amb)) continue;
    for (int k = 0; k < edges; ++k) {
      const int j = 1 + k * grid + b;
      if (j >= m) break;
      for (int d = 0; d < 2; ++d) {
        const double v = G.sm[2 * j + d];
        if (!(v < INFINITY)) continue;
        near |= fabs(v - thr) <= amb;
        if (v <= thr) {
          const unsigned id = 2u * (unsigned)label_id[G.cl[cur][j].top] + d;
          const unsigned long long key = (unsigned long long)id << 32 | (unsigned)(2 * j + d);
          win = key < win ? key : win;
        }
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long x = __shfl_xor(win, o, 64);
    win = x < win ? x : win;
  }
  if (lane == 0) s_win[tid >> 6] = win;
  const int fl = __syncthreads_or(near) || (cnt >> 40) ? 1 : 0;
  win = s_win[lane & (NW - 1)];
  for (int o = NW / 2; o > 0; o >>= 1) {
    const unsigned long long x = __shfl_xor(win, o, 64);
    win = x < win ? x : win;
  }
  const int wc = __builtin_amdgcn_readfirstlane((int)(unsigned)win), wj = wc >> 1, dir = wc & 1;
  const GEdge E = G.edge[wj];
  const int r = dir ? E.b : E.a, s = dir ? E.a : E.b, jr = dir ? E.jb : E.ja;
  for (int q = tid; q < S * 3; q += kGreedyPickThreads) J[q] = G.I[((size_t)(q / 3) * n + r) * 3 + q % 3];
  const GClus cr = G.cl[cur][jr], cs = G.cl[cur][dir ? E.ja : E.jb];
  __syncthreads();
  if (blockIdx.x == 0) {
    if (tid == 0) {
      GStep sp;
      sp.cand = (int)(win >> 32);
      sp.s = label_id[s];
      sp.r = label_id[r];
      sp.ambiguous = fl;
      sp.n_cand = (int)(cnt & 0xfffffu);
      sp.n_feasible = (int)(cnt >> 20 & 0xfffffu);
      sp.smice = G.sm[wc];
      sp.emax = G.em[wc];
      steps[st.iter] = sp;
      *G.gs[nxt] = GState{st.iter + 1, 0, s, E.a0, E.a1, E.b0, E.b1};
    }
    for (int q = tid; q < S * 3; q += kGreedyPickThreads) {
      const size_t ls = ((size_t)(q / 3) * n + s) * 3 + q % 3;
      G.I[ls] = cadd(G.I[ls], J[q]);
    }
  }
  if (t < n) {
    G.rank[nxt][t] = make_int2(rk.x - (t > r), rk.y - (te > r));
    if (sup == r) G.sup[t] = s;
  }
  if (t - lane >= m - 1) return;
  double mx = 0.0, sum = 0.0;
  if (t < m - 1) {
    const int jo = t + (t >= jr);
    GClus c = t >= jr ? c1 : c0;
    const bool inA = E.a0 <= c.u && c.u < E.a1, in = inA || (E.b0 <= c.u && c.u < E.b1);
    if (in || c.u == s) {
      const int x = T.lca(c.u, inA ? E.a : E.b);
      const bool up = inA != (dir != 0);  // r's side
      MoveDelta md;
      md.between(Zr, up ? x : E.w, up ? E.w : x);
      for (int l = 0; l < S; ++l) {
        const size_t at = (size_t)l * n + c.u, ar = (size_t)l * n + (c.u == s ? r : c.u);
        double e = 0.0;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          double2 v = G.V[at * 3 + p];
          if (in) {
            v = cadd(v, md.dv(p, J + l * 3));
            G.V[at * 3 + p] = v;
          }
          const double lo = fmin(G.ext[at * 6 + p], G.ext[ar * 6 + p]);
          const double hi = fmax(G.ext[at * 6 + 3 + p], G.ext[ar * 6 + 3 + p]);
          if (c.u == s) {
            G.ext[at * 6 + p] = lo;
            G.ext[at * 6 + 3 + p] = hi;
          }
          e = ext_err(e, lo, hi, sqrt(cabs2(v)));
        }
        G.mice[nxt][(size_t)l * n + t] = e;
        mx = fmax(mx, e);
        sum += e;
      }
    } else {
      for (int l = 0; l < S; ++l) {
        const double e = G.mice[cur][(size_t)l * n + jo];
        G.mice[nxt][(size_t)l * n + t] = e;
        mx = fmax(mx, e);
        sum += e;
      }
    }
    if (c.b == r && c.u != s) {
      c.b = s;
      c.ph = (c.ph & 7) | (cs.ph & 7) << 8;
    }
    if (c.u == s && dir) {  // s takes r's place under the cluster above r's
      c.top = cr.top;
      c.b = cr.b;
      c.ph = (c.ph & 7) | (cr.ph & ~7);
    }
    G.cl[nxt][t] = c;
    G.arr[nxt][t] = mx;
  }
  run_totals(mx, sum, G.bmax[nxt] + (t >> 6), G.bsum[nxt] + (t >> 6));
}

// ---- radialization (Section V) --------------------------------------------

// Critical nodes of a kept set (one block, level by level): a node that is
// not kept is critical when three or more of its tree directions reach a
// kept node through nodes that are not kept (its degree in the sub-tree that
// spans the kept nodes of its Kron clique).  Writes the radialized kept set
// and, for both kept sets, every node's nearest kept proper ancestor (-1 at
// the slack).  Scratch: down, up, cnt (n ints each).
__global__ __launch_bounds__(kGreedyPickThreads) void k_radialize(
    int n, const int* __restrict__ parent, const int* __restrict__ ch_off, const int* __restrict__ ch,
    const int* __restrict__ lvl_off, const int* __restrict__ lvl_nodes, int nlev, const int* __restrict__ sup,
    int* __restrict__ down, int* __restrict__ up, int* __restrict__ cnt, uint8_t* __restrict__ kept_rad,
    int* __restrict__ kp_rad, int* __restrict__ kp_mesh, int* __restrict__ ncrit) {
  __shared__ int shi[kGreedyPickThreads / 64];
  // down[x]: x is kept, or a kept node lies below x through non-kept nodes;
  // cnt[x]: children c with down[c]
  for (int lev = nlev - 1; lev >= 0; --lev) {
    for (int q = lvl_off[lev] + threadIdx.x; q < lvl_off[lev + 1]; q += blockDim.x) {
      const int x = lvl_nodes[q];
      int c = 0;
      for (int e = ch_off[x]; e < ch_off[x + 1]; ++e) c += down[ch[e]];
      cnt[x] = c;
      down[x] = (sup[x] == x || c > 0) ? 1 : 0;
    }
    __syncthreads();
  }
  // up[x]: the direction towards the parent reaches a kept node
  for (int lev = 0; lev < nlev; ++lev) {
    for (int q = lvl_off[lev] + threadIdx.x; q < lvl_off[lev + 1]; q += blockDim.x) {
      const int x = lvl_nodes[q];
      if (x == 0) {
        up[x] = 0;
        continue;
      }
      const int p = parent[x];
      up[x] = (sup[p] == p || up[p] || cnt[p] - down[x] > 0) ? 1 : 0;
    }
    __syncthreads();
  }
  int nc = 0;
  for (int x = threadIdx.x; x < n; x += blockDim.x) {
    const bool kept = sup[x] == x;
    const bool crit = !kept && up[x] + cnt[x] >= 3;
    nc += crit;
    kept_rad[x] = (kept || crit) ? 1 : 0;
  }
  nc = block_reduce(nc, [](int a, int b) { return a + b; }, shi);
  if (threadIdx.x == 0) *ncrit = nc;
  __syncthreads();
  for (int lev = 0; lev < nlev; ++lev) {
    for (int q = lvl_off[lev] + threadIdx.x; q < lvl_off[lev + 1]; q += blockDim.x) {
      const int x = lvl_nodes[q];
      if (x == 0) {
        kp_rad[x] = kp_mesh[x] = -1;
        continue;
      }
      const int p = parent[x];
      kp_rad[x] = kept_rad[p] ? p : kp_rad[p];
      kp_mesh[x] = sup[p] == p ? p : kp_mesh[p];
    }
    __syncthreads();
  }
}

// Voltage check of a radial reduced network (one thread per node and
// scenario): for every kept node x, the voltage of the radial network whose
// edges join each kept node to its nearest kept proper ancestor kp, with the
// aggregated load currents, is V0 - sum_j Zroot(a(lca(x, j))) I_j, a(v) = v
// when v is kept, else kp[v]; its largest distance from the full network's
// voltage V goes to *dv (bit pattern of a non-negative double).  Zero when
// every kept pair's lowest common ancestor is kept, i.e. when the network is
// radial with the same voltages.
__global__ __launch_bounds__(kGreedyThreads) void k_radial_check(
    int n, int S, const uint8_t* __restrict__ phase, const int* __restrict__ pos, LcaTab T,
    const double2* __restrict__ Zr, const int* __restrict__ sup, const uint8_t* __restrict__ kept_rad, const int* __restrict__ kp, int use_rad,
    const double2* __restrict__ Iagg, const double2* __restrict__ V, double2 v0a, double2 v0b, double2 v0c,
    unsigned long long* __restrict__ dv) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  double e = 0.0;
  if (t < n * S) {
    const int x = t % n, l = t / n;
    const bool kx = use_rad ? kept_rad[x] != 0 : sup[x] == x;
    if (kx) {
      const double2 v0[3] = {v0a, v0b, v0c};
      double2 acc[3] = {v0[0], v0[1], v0[2]};
      for (int k = 1; k < n; ++k) {  // in the caller's node order
        const int j = pos[k];
        if (sup[j] != j) continue;  // only super-nodes carry current
        int a = T.lca(x, j);
        const bool ka = use_rad ? kept_rad[a] != 0 : sup[a] == a;
        if (!ka) a = kp[a];
        const double2* Za = Zr + (size_t)a * 9;
        const double2* Ij = Iagg + ((size_t)l * n + j) * 3;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          acc[p] = csub(acc[p], cadd(cadd(cmul(Za[p * 3], Ij[0]), cmul(Za[p * 3 + 1], Ij[1])), cmul(Za[p * 3 + 2], Ij[2])));
      }
      const double2* Vx = V + ((size_t)l * n + x) * 3;
#pragma unroll
      for (int p = 0; p < 3; ++p)
        if (phase[x] >> p & 1u) e = fmax(e, sqrt(cabs2(csub(acc[p], Vx[p]))));
    }
  }
  for (int o = 32; o > 0; o >>= 1) e = fmax(e, __shfl_xor(e, o, 64));
  if ((threadIdx.x & 63) == 0 && e > 0.0) atomicMax(dv, (unsigned long long)__double_as_longlong(e));
}

// I = A I^ for a given assignment: one thread per (scenario, node, phase)
// adds its cluster's members' currents in node order (members of super-node
// y: mem[moff[y] .. moff[y + 1]); zero for nodes that are not super-nodes).
__global__ void k_greedy_aggregate(int n, int S, const int* __restrict__ moff, const int* __restrict__ mem,
                                   const double2* __restrict__ A, double2* __restrict__ Iagg) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (size_t)S * n * 3) return;
  const int p = (int)(t % 3), y = (int)((t / 3) % n);
  const size_t base = (t / 3 / n) * n * 3;
  double2 acc = make_double2(0.0, 0.0);
  for (int q = moff[y]; q < moff[y + 1]; ++q) acc = cadd(acc, A[base + (size_t)mem[q] * 3 + p]);
  Iagg[t] = acc;
}

// Largest error of the current state per scenario (one block each): every
// node against its super-node's voltage.
__global__ __launch_bounds__(kGreedyThreads) void k_greedy_err(int n, const uint8_t* __restrict__ phase,
                                                               const int* __restrict__ sup,
                                                               const double2* __restrict__ V,
                                                               const double* __restrict__ absV,
                                                               double* __restrict__ err) {
  __shared__ double shd[16];
  const size_t base = (size_t)blockIdx.x * n * 3;
  double e = 0.0;
  for (int x = threadIdx.x; x < n; x += blockDim.x)
    for (int p = 0; p < 3; ++p)
      if (phase[x] >> p & 1u) e = fmax(e, fabs(absV[base + x * 3 + p] - sqrt(cabs2(V[base + sup[x] * 3 + p]))));
  e = block_reduce(e, [](double a, double b) { return fmax(a, b); }, shd);
  if (threadIdx.x == 0) err[blockIdx.x] = e;
}

}  // namespace okr

using namespace okr;

struct okr_greedy {
  hipStream_t stream = nullptr;
  std::string err;
  bool planned = false;
  int n = 0, S = 0, nlev = 0;
  std::vector<int> parent, pos, pre;  // by the caller's id: parent, label; by label: the caller's id
  std::vector<uint8_t> phase, lphase;  // by the caller's id, by label
  // workspace layout (byte offsets)
  size_t o_topo = 0, o_z = 0, o_Zr = 0, o_A = 0, o_absV = 0, o_Vhat = 0, o_I = 0, o_V = 0, o_Ib = 0,
         o_sup = 0, o_sm = 0, o_em = 0, o_steps = 0, o_iters = 0, total = 0;
  // packed int arrays over labels: parent, end of the subtree, level offsets,
  // level nodes, children; the caller's id and its inverse; the load flow's
  // tables; phases (bytes); the status word (4 ints, cleared by the upload) and,
  // read back with it, the errors per scenario; then (64-bit) the lca table,
  // which only a search and the radialization read
  size_t t_parent = 0, t_end = 0, t_lvl_off = 0, t_lvl_nodes = 0, t_ch_off = 0, t_ch = 0, t_pre = 0, t_pos = 0,
         t_phase = 0, t_status = 0, t_lca = 0;
  // state of the search (two copies of what each iteration rewrites)
  size_t o_gs[2] = {}, o_cl[2] = {}, o_rank[2] = {}, o_mice[2] = {}, o_arr[2] = {}, o_bmax[2] = {}, o_bsum[2] = {};
  size_t o_ext = 0, o_edge = 0, o_part = 0, o_blk = 0;
  // radialization: 5 int arrays of n, kept flags, counter, two maxima
  size_t o_rad = 0, o_radk = 0, o_radx = 0;
  FlowPlan flow;
  std::vector<int> topo_host;
};

#define OKRG_FAIL(g, code, ...)            \
  do {                                     \
    char _b[512];                          \
    snprintf(_b, sizeof _b, __VA_ARGS__);  \
    (g)->err = _b;                         \
    return code;                           \
  } while (0)

#define OKRG_HIP(g, call)                                                                   \
  do {                                                                                      \
    hipError_t _e = (call);                                                                 \
    if (_e != hipSuccess) OKRG_FAIL(g, OKR_E_HIP, "%s: %s", #call, hipGetErrorString(_e)); \
  } while (0)

extern "C" int okr_greedy_create(okr_greedy** g, void* hip_stream) {
  if (!g) return OKR_E_ARG;
  okr_greedy* G = new (std::nothrow) okr_greedy();
  if (!G) return OKR_E_ARG;
  G->stream = static_cast<hipStream_t>(hip_stream);
  *g = G;
  return OKR_OK;
}

extern "C" int okr_greedy_destroy(okr_greedy* g) {
  if (!g) return OKR_E_ARG;
  delete g;
  return OKR_OK;
}

extern "C" const char* okr_greedy_last_error(const okr_greedy* g) { return g ? g->err.c_str() : "null handle"; }

extern "C" int okr_greedy_plan(okr_greedy* g, int32_t n, const int32_t* parent, const uint8_t* phase, int32_t S,
                               size_t* workspace_bytes) {
  if (!g) return OKR_E_ARG;
  g->planned = false;
  if (!parent || !phase || !workspace_bytes || n < 1 || S < 1) OKRG_FAIL(g, OKR_E_ARG, "null argument, n < 1 or S < 1");
  g->n = n;
  g->S = S;
  g->parent.assign(parent, parent + n);
  g->phase.assign(phase, phase + n);
  if (g->parent[0] != -1) OKRG_FAIL(g, OKR_E_NOT_TREE, "parent[0] must be -1");
  for (int i = 1; i < n; ++i)
    if (g->parent[i] < 0 || g->parent[i] >= n || g->parent[i] == i)
      OKRG_FAIL(g, OKR_E_NOT_TREE, "parent[%d] = %d out of range", i, g->parent[i]);
  std::vector<int> coff(n + 1, 0), cch(std::max(n - 1, 1), 0);  // children by the caller's id
  for (int i = 1; i < n; ++i) coff[g->parent[i] + 1]++;
  for (int i = 0; i < n; ++i) coff[i + 1] += coff[i];
  {
    std::vector<int> fill(coff.begin(), coff.begin() + n);
    for (int i = 1; i < n; ++i) cch[fill[g->parent[i]]++] = i;
  }
  // labels: positions in a depth-first order, children in increasing id
  std::vector<int>& pre = g->pre;
  pre.clear();
  pre.reserve(n);
  {
    std::vector<int> st{0};
    while (!st.empty() && (int)pre.size() <= n) {
      const int v = st.back();
      st.pop_back();
      pre.push_back(v);
      for (int e = coff[v + 1] - 1; e >= coff[v]; --e) st.push_back(cch[e]);
    }
  }
  if ((int)pre.size() != n) OKRG_FAIL(g, OKR_E_NOT_TREE, "parent[] is not a tree rooted at node 0");
  g->pos.assign(n, 0);
  for (int q = 0; q < n; ++q) g->pos[pre[q]] = q;
  std::vector<int> par(n, -1), end(n, 0), depth(n, 0);  // by label
  for (int q = 1; q < n; ++q) par[q] = g->pos[g->parent[pre[q]]];
  for (int q = 0; q < n; ++q) end[q] = q + 1;
  for (int q = n - 1; q >= 1; --q) end[par[q]] = std::max(end[par[q]], end[q]);
  int dmax = 0;
  for (int q = 1; q < n; ++q) {
    depth[q] = depth[par[q]] + 1;
    dmax = std::max(dmax, depth[q]);
  }
  g->nlev = dmax + 1;
  std::vector<int> lvl_off(g->nlev + 1, 0), lvl_nodes(n), ch_off(n + 1, 0), ch(std::max(n - 1, 1), 0);
  for (int q = 0; q < n; ++q) lvl_off[depth[q] + 1]++;
  for (int d = 0; d < g->nlev; ++d) lvl_off[d + 1] += lvl_off[d];
  for (int q = 1; q < n; ++q) ch_off[par[q] + 1]++;
  for (int q = 0; q < n; ++q) ch_off[q + 1] += ch_off[q];
  {
    std::vector<int> fl(lvl_off.begin(), lvl_off.begin() + g->nlev), fc(ch_off.begin(), ch_off.begin() + n);
    for (int q = 0; q < n; ++q) lvl_nodes[fl[depth[q]]++] = q;
    for (int q = 1; q < n; ++q) ch[fc[par[q]]++] = q;
  }
  for (int i = 0; i < n; ++i) {
    if (g->phase[i] == 0 || g->phase[i] > 7) OKRG_FAIL(g, OKR_E_PHASE, "node %d has phase mask %d", i, g->phase[i]);
    if (i > 0 && (g->phase[i] & ~g->phase[g->parent[i]]))
      OKRG_FAIL(g, OKR_E_PHASE, "phases of node %d are not a subset of its parent's", i);
  }
  g->lphase.resize(n);
  for (int q = 0; q < n; ++q) g->lphase[q] = g->phase[pre[q]];
  // packed topology
  g->topo_host.clear();
  auto put = [&](const std::vector<int>& v) {
    const size_t at = g->topo_host.size();
    g->topo_host.insert(g->topo_host.end(), v.begin(), v.end());
    return at;
  };
  g->t_parent = put(par);
  g->t_end = put(end);
  g->t_lvl_off = put(lvl_off);
  g->t_lvl_nodes = put(lvl_nodes);
  g->t_ch_off = put(ch_off);
  g->t_ch = put(ch);
  g->t_pre = put(pre);
  g->t_pos = put(g->pos);
  g->flow = flow_tables(n, end.data(), g->lphase.data(), g->topo_host);
  g->t_phase = g->topo_host.size();
  g->topo_host.resize(g->t_phase + (n + 3) / 4, 0);
  std::memcpy(g->topo_host.data() + g->t_phase, g->lphase.data(), n);
  if (g->topo_host.size() & 1) g->topo_host.push_back(0);  // (8-byte entries follow)
  g->t_status = g->topo_host.size();
  g->topo_host.resize(g->t_status + 4 + 2 * (size_t)S, 0);
  {
    int K = 1;
    while ((1 << K) <= n) ++K;
    std::vector<unsigned long long> sp((size_t)K * n, ~0ull);
    for (int q = 1; q < n; ++q) sp[q] = (unsigned long long)par[q] << 32 | (0xffffffffu - (unsigned)q);
    for (int k = 1; k < K; ++k)
      for (int q = 0; q < n; ++q) {
        const unsigned long long a = sp[(size_t)(k - 1) * n + q];
        const int j = q + (1 << (k - 1));
        sp[(size_t)k * n + q] = j < n ? std::min(a, sp[(size_t)(k - 1) * n + j]) : a;
      }
    g->t_lca = g->topo_host.size();
    g->topo_host.resize(g->t_lca + 2 * sp.size());
    std::memcpy(g->topo_host.data() + g->t_lca, sp.data(), sizeof(unsigned long long) * sp.size());
  }
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) & ~size_t(255);
    return at;
  };
  const size_t c3 = (size_t)S * n * 3;
  g->o_topo = take(sizeof(int) * g->topo_host.size());
  g->o_z = take(sizeof(double2) * 9 * n);
  g->o_Zr = take(sizeof(double2) * 9 * n);
  g->o_Vhat = take(sizeof(double2) * c3);
  g->o_A = take(sizeof(double2) * c3);
  g->o_absV = take(sizeof(double) * c3);
  g->o_I = take(sizeof(double2) * c3);
  g->o_V = take(sizeof(double2) * c3);
  g->o_Ib = take(sizeof(double2) * c3);
  g->o_sup = take(sizeof(int) * (3 * (size_t)n + 1));  // (an assignment's member lists follow)
  g->o_sm = take(sizeof(double) * 2 * n);
  g->o_em = take(sizeof(double) * 2 * n);
  g->o_steps = take(sizeof(GStep) * n);
  g->o_iters = take(sizeof(int) * S);
  const size_t runs = ((size_t)n + 63) / 64;
  for (int k = 0; k < 2; ++k) {
    g->o_gs[k] = take(sizeof(GState));
    g->o_cl[k] = take(sizeof(GClus) * n);
    g->o_rank[k] = take(sizeof(int2) * n);
    g->o_mice[k] = take(sizeof(double) * (size_t)S * n);
    g->o_arr[k] = take(sizeof(double) * n);
    g->o_bmax[k] = take(sizeof(double) * runs);
    g->o_bsum[k] = take(sizeof(double) * runs);
  }
  g->o_ext = take(sizeof(double) * 2 * c3);
  g->o_edge = take(sizeof(GEdge) * n);
  g->o_part = take(sizeof(GPart) * n);
  g->o_blk = take(sizeof(GBlk) * n);
  g->o_rad = take(sizeof(int) * 5 * (size_t)n);
  g->o_radk = take(n);
  g->o_radx = take(sizeof(unsigned long long) * 4);
  g->total = off;
  *workspace_bytes = off;
  g->planned = true;
  return OKR_OK;
}

namespace {
struct GPtrs {
  int *topo, *parent, *end, *lvl_off, *lvl_nodes, *ch_off, *ch, *pre, *pos, *sup, *status, *iters, *csr;
  LcaTab T;
  GreedyState G;
  uint8_t* phase;
  double2 *z, *Zr, *Vhat, *A, *I, *V, *Ib;
  double *absV, *err;
  GStep* steps;
};

GPtrs gptrs(const okr_greedy* g, void* ws) {
  char* b = (char*)ws;
  GPtrs p;
  p.topo = (int*)(b + g->o_topo);
  p.parent = p.topo + g->t_parent;
  p.end = p.topo + g->t_end;
  p.lvl_off = p.topo + g->t_lvl_off;
  p.lvl_nodes = p.topo + g->t_lvl_nodes;
  p.ch_off = p.topo + g->t_ch_off;
  p.ch = p.topo + g->t_ch;
  p.pre = p.topo + g->t_pre;
  p.pos = p.topo + g->t_pos;
  p.T.st = (const unsigned long long*)(p.topo + g->t_lca);
  p.T.n = g->n;
  p.phase = (uint8_t*)(p.topo + g->t_phase);
  p.status = p.topo + g->t_status;
  p.err = (double*)(p.status + 4);
  p.z = (double2*)(b + g->o_z);
  p.Zr = (double2*)(b + g->o_Zr);
  p.Vhat = (double2*)(b + g->o_Vhat);
  p.A = (double2*)(b + g->o_A);
  p.absV = (double*)(b + g->o_absV);
  p.I = (double2*)(b + g->o_I);
  p.V = (double2*)(b + g->o_V);
  p.Ib = (double2*)(b + g->o_Ib);
  p.sup = (int*)(b + g->o_sup);
  p.csr = p.sup + g->n;
  p.steps = (GStep*)(b + g->o_steps);
  p.iters = (int*)(b + g->o_iters);
  GreedyState& G = p.G;
  for (int k = 0; k < 2; ++k) {
    G.gs[k] = (GState*)(b + g->o_gs[k]);
    G.cl[k] = (GClus*)(b + g->o_cl[k]);
    G.rank[k] = (int2*)(b + g->o_rank[k]);
    G.mice[k] = (double*)(b + g->o_mice[k]);
    G.arr[k] = (double*)(b + g->o_arr[k]);
    G.bmax[k] = (double*)(b + g->o_bmax[k]);
    G.bsum[k] = (double*)(b + g->o_bsum[k]);
  }
  G.ext = (double*)(b + g->o_ext);
  G.edge = (GEdge*)(b + g->o_edge);
  G.part = (GPart*)(b + g->o_part);
  G.sm = (double*)(b + g->o_sm);
  G.em = (double*)(b + g->o_em);
  G.blk = (GBlk*)(b + g->o_blk);
  G.sup = p.sup;
  G.V = p.V;
  G.I = p.I;
  return p;
}

// Common set-up of a run or an evaluation: topology upload, branch
// impedances, impedances from the root, scenario library (load flow unless
// V^ is given).  lca: the lowest-common-ancestor table too.  eval: the load flow
// goes on to evaluate that assignment (form 1 of the load flow only).
int setup(okr_greedy* g, const GPtrs& p, const okr_yblocks* Y, const okr_loads* L, const okr_greedy_params* prm,
          bool lca, const FlowEval* eval = nullptr) {
  const hipStream_t st = g->stream;
  const int n = g->n, S = g->S;
  OKRG_HIP(g, hipMemcpyAsync(p.topo, g->topo_host.data(), sizeof(int) * (lca ? g->topo_host.size() : g->t_lca),
                             hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_branch_z, dim3((n + 63) / 64 + (n + 3) / 4), dim3(64), 0, st, n, (n + 63) / 64,
                     (const uint8_t*)p.phase, (const int*)p.ch_off, (const int*)p.ch,
                     (const int*)p.pre, (const double2*)Y->Y_diag, (const double2*)Y->Y_off, p.z, p.status, State{});
  const bool scan = !(prm->flags & OKR_FLAG_VHAT_GIVEN) && g->flow.form;
  if (!scan)  // (otherwise beside the load flow)
    hipLaunchKernelGGL(k_zroot, dim3(1), dim3(1024), 0, st, n, (const int*)p.parent, (const int*)p.lvl_off,
                       (const int*)p.lvl_nodes, g->nlev, (const double2*)p.z, p.Zr);
  const size_t c3 = (size_t)S * n * 3;
  const double2* V0 = (const double2*)L->V0;
  if (prm->flags & OKR_FLAG_VHAT_GIVEN) {
    hipLaunchKernelGGL(k_from_vhat, dim3((unsigned)((c3 + 255) / 256)), dim3(256), 0, st, n, S,
                       (const uint8_t*)p.phase, (const double2*)L->S_load, (const double2*)L->Vhat, 0.0, 1e300, p.A,
                       p.absV, p.status, (const int*)p.pre, (double2*)nullptr);
  } else if (scan) {
    OKRG_HIP(g, flow_prepare(g->flow));
    const FlowArgs a{(const int*)p.topo, p.phase, p.z, (const double2*)L->S_load, {V0[0], V0[1], V0[2]},
                     prm->pf_tol > 0 ? prm->pf_tol : 1e-13, 0.0, 1e300, prm->pf_maxit > 0 ? prm->pf_maxit : 100,
                     p.Vhat, p.Ib, p.A, p.absV, p.iters, p.status, p.pre, nullptr, p.parent, p.lvl_off,
                     p.lvl_nodes, g->nlev, p.Zr};
    if (eval) flow_eval_launch(g->flow, a, *eval, S, st);
    else flow_launch(g->flow, a, S, st);
  } else {
    hipLaunchKernelGGL(k_powerflow, dim3(S), dim3(256), 0, st, n, (const int*)p.parent, (const uint8_t*)p.phase,
                       (const int*)p.lvl_off, (const int*)p.lvl_nodes, g->nlev, (const int*)p.ch_off,
                       (const int*)p.ch, (const double2*)p.z, (const double2*)L->S_load, V0[0], V0[1], V0[2],
                       prm->pf_tol > 0 ? prm->pf_tol : 1e-13, prm->pf_maxit > 0 ? prm->pf_maxit : 100, 0.0, 1e300,
                       p.Vhat, p.Ib, p.A, p.absV, p.iters, p.status, (const int*)p.pre, (double2*)nullptr);
  }
  OKRG_HIP(g, hipGetLastError());
  return OKR_OK;
}

// Voltages V of the aggregated currents I.
int fixed_solve(okr_greedy* g, const GPtrs& p, const double2* V0) {
  const hipStream_t st = g->stream;
  if (g->flow.form) {
    OKRG_HIP(g, flow_prepare(g->flow));
    flow_fixed_launch(g->flow, p.topo, p.phase, p.z, V0, p.I, p.Ib, p.V, g->S, st);
  } else {
    hipLaunchKernelGGL(k_greedy_sweep, dim3(g->S), dim3(kGreedyThreads), 0, st, g->n, (const int*)p.parent,
                       (const uint8_t*)p.phase, (const int*)p.lvl_off, (const int*)p.lvl_nodes, g->nlev,
                       (const int*)p.ch_off, (const int*)p.ch, (const double2*)p.z, V0[0], V0[1], V0[2],
                       (const double2*)p.I, p.Ib, p.V);
  }
  OKRG_HIP(g, hipGetLastError());
  return OKR_OK;
}

int check_status(okr_greedy* g, int hs) {
  if (hs & 1) OKRG_FAIL(g, OKR_E_SINGULAR, "a present-phase branch block is singular");
  if (hs & 2) OKRG_FAIL(g, OKR_E_PHASE, "nonzero admittance entries on absent phases");
  if (hs & (4 | 8)) OKRG_FAIL(g, OKR_E_UNSUPPORTED, "admittance blocks asymmetric or with shunts");
  if (hs & 16) OKRG_FAIL(g, OKR_E_PF_DIVERGED, "load flow did not converge");
  return OKR_OK;
}

int check_call(okr_greedy* g, const okr_yblocks* Y, const okr_loads* L, const okr_greedy_params* prm, void* ws) {
  if (!g->planned) OKRG_FAIL(g, OKR_E_ARG, "okr_greedy_plan has not succeeded");
  if (!Y || !L || !prm || !Y->Y_diag || !Y->Y_off || !L->S_load || !L->V0) OKRG_FAIL(g, OKR_E_ARG, "null argument");
  if (L->S != g->S) OKRG_FAIL(g, OKR_E_ARG, "loads->S = %d, planned for %d", L->S, g->S);
  if ((prm->flags & OKR_FLAG_VHAT_GIVEN) && !L->Vhat) OKRG_FAIL(g, OKR_E_ARG, "OKR_FLAG_VHAT_GIVEN without Vhat");
  if (!ws) OKRG_FAIL(g, OKR_E_WORKSPACE, "no workspace");
  return OKR_OK;
}
// An assignment: super-nodes are their own super-node, every cluster is
// connected (one member whose parent lies outside it), the slack is a
// super-node, and a member's phases lie within its super-node's.
int check_assignment(okr_greedy* g, const int32_t* super) {
  const int n = g->n;
  std::vector<int> top(n, -1);
  for (int x = 0; x < n; ++x) {
    const int s = super[x];
    if (s < 0 || s >= n || super[s] != s) OKRG_FAIL(g, OKR_E_ARG, "super[%d] = %d is not a super-node", x, s);
    if (g->phase[x] & ~g->phase[s]) OKRG_FAIL(g, OKR_E_ARG, "node %d has phases outside its super-node's", x);
  }
  if (super[0] != 0) OKRG_FAIL(g, OKR_E_ARG, "the slack must stay its own super-node");
  for (int x = 0; x < n; ++x) {  // each cluster has one node whose parent lies outside it
    const int s = super[x];
    if (x == 0 || super[g->parent[x]] != s) {
      if (top[s] >= 0) OKRG_FAIL(g, OKR_E_ARG, "the cluster of super-node %d is not connected", s);
      top[s] = x;
    }
  }
  return OKR_OK;
}

// The assignment by label (n entries), then the members of every cluster in the
// caller's node order (CSR over labels: n + 1 offsets, n members).
void assignment(const okr_greedy* g, const int32_t* super, std::vector<int>& out) {
  const int n = g->n;
  out.assign(3 * (size_t)n + 1, 0);
  int *lsup = out.data(), *off = lsup + n, *mem = off + n + 1;
  for (int x = 0; x < n; ++x) {
    lsup[g->pos[x]] = g->pos[super[x]];
    off[g->pos[super[x]] + 1]++;
  }
  for (int y = 0; y < n; ++y) off[y + 1] += off[y];
  std::vector<int> fill(off, off + n);
  for (int x = 0; x < n; ++x) mem[fill[g->pos[super[x]]]++] = g->pos[x];
}

// Waits for the stream and reads the status word and the errors per scenario.
int read_errors(okr_greedy* g, const GPtrs& p, double* err) {
  std::vector<double> r(2 + (size_t)g->S);  // (4 status ints, then the errors)
  OKRG_HIP(g, hipMemcpyAsync(r.data(), p.status, sizeof(double) * r.size(), hipMemcpyDeviceToHost, g->stream));
  OKRG_HIP(g, hipStreamSynchronize(g->stream));
  int status;
  std::memcpy(&status, r.data(), sizeof status);
  std::memcpy(err, r.data() + 2, sizeof(double) * g->S);
  return check_status(g, status);
}
}  // namespace

extern "C" int okr_greedy_run(okr_greedy* g, const okr_yblocks* Y, const okr_loads* L, const okr_greedy_params* prm,
                              void* ws, okr_greedy_result* out) {
  if (!g) return OKR_E_ARG;
  int rc = check_call(g, Y, L, prm, ws);
  if (rc) return rc;
  if (!out || !out->super || !out->steps || !out->err_per_snapshot) OKRG_FAIL(g, OKR_E_ARG, "null result buffer");
  const int n = g->n, S = g->S;
  if (S > kGreedyMaxS) OKRG_FAIL(g, OKR_E_UNSUPPORTED, "the search takes at most %d scenarios", kGreedyMaxS);
  // every candidate sums every cluster while there are few (1000 nodes, 2
  // scenarios: 9.5 us a scoring against 10.7); beyond that, or when asked, only
  // the clusters a move can change.  A level counts as three errors, so that
  // deep feeders near the limit go by the changed clusters too: us per move of
  // the first 320, every cluster against the changed ones, 6000 nodes x 1
  // scenario with 949 levels 80 and 39, 3000 x 2 with 820 levels 50 and 39,
  // 1500 x 4 with 1196 levels 45 and 49
  const bool incremental = (prm->flags & OKR_GREEDY_INCREMENTAL) || (size_t)S * n > kGreedyFullSN ||
                           (size_t)S * n + 3 * (size_t)g->nlev > kGreedyFullSNL;
  if (incremental && n > kGreedyMaxN)
    OKRG_FAIL(g, OKR_E_UNSUPPORTED, "the search takes at most %d nodes", kGreedyMaxN);
  const hipStream_t st = g->stream;
  const GPtrs p = gptrs(g, ws);
  hipEvent_t ev[3];
  for (auto& e : ev) OKRG_HIP(g, hipEventCreate(&e));
  struct EvGuard {
    hipEvent_t* e;
    ~EvGuard() {
      for (int i = 0; i < 3; ++i) (void)hipEventDestroy(e[i]);
    }
  } guard{ev};
  OKRG_HIP(g, hipEventRecord(ev[0], st));
  rc = setup(g, p, Y, L, prm, true);
  if (rc) return rc;
  const double2* V0 = (const double2*)L->V0;
  const size_t c3 = (size_t)S * n * 3;
  hipLaunchKernelGGL(k_greedy_init, dim3((unsigned)((std::max(c3, (size_t)n) + 255) / 256)), dim3(256), 0, st, n, S,
                     (const double2*)p.A, p.I, p.sup, p.G.gs[0]);
  rc = fixed_solve(g, p, V0);
  if (rc) return rc;
  hipLaunchKernelGGL(k_greedy_prep, dim3((unsigned)(n / kGreedyThreads + 1)), dim3(kGreedyThreads), 0, st, n, S,
                     (const int*)p.parent, (const int*)p.end, (const uint8_t*)p.phase, (const double*)p.absV, p.G);
  OKRG_HIP(g, hipGetLastError());
  OKRG_HIP(g, hipEventRecord(ev[1], st));
  const double e_bar = prm->e_bar, tie = prm->tie_tol > 0 ? prm->tie_tol : 1e-11;
  const double amb = prm->amb_tol > 0 ? prm->amb_tol : 1e-13;
  // at most one move per enqueued iteration: the cap is the number enqueued
  const int cap = prm->max_iter > 0 ? std::min(prm->max_iter, n - 1) : n - 1;
  GState hs{};
  int enq = 0;
  constexpr int kBatch = 32;  // moves enqueued between checks of the done flag
  const bool timing = (prm->flags & OKR_FLAG_TIMING) != 0;
  std::vector<hipEvent_t> tev(timing ? 2 * kBatch : 0);
  for (auto& e : tev) OKRG_HIP(g, hipEventCreate(&e));
  struct TevGuard {
    std::vector<hipEvent_t>* v;
    ~TevGuard() {
      for (hipEvent_t e : *v) (void)hipEventDestroy(e);
    }
  } tguard{&tev};
  double score_ms = 0.0;
  int launches = 0;
  // one iteration's two launches (and the timing events around the scoring)
  auto enqueue_iteration = [&](int t) -> hipError_t {
    if (timing) {
      const hipError_t e = hipEventRecord(tev[2 * t], st);
      if (e != hipSuccess) return e;
    }
    const int cur = t & 1;  // batches start with copy 0
    const int edges = incremental ? kGreedyEdges : 1;
    if (incremental)
      hipLaunchKernelGGL(k_greedy_score<false>, dim3((unsigned)((n - 2) / kGreedyEdges + 1)), dim3(kGreedyEdges * 64),
                         0, st, n, S, cur, p.T, (const int*)p.end, (const int*)p.pre, (const double2*)p.Zr, e_bar, amb, p.G);
    else
      hipLaunchKernelGGL(k_greedy_score<true>, dim3((unsigned)(n - 1)), dim3(kGreedyThreads), 0, st, n, S, cur, p.T,
                         (const int*)p.end, (const int*)p.pre, (const double2*)p.Zr, e_bar, amb, p.G);
    if (timing) {
      const hipError_t e = hipEventRecord(tev[2 * t + 1], st);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_greedy_apply, dim3((unsigned)((n - 1) / kGreedyPickThreads + 1)), dim3(kGreedyPickThreads), 0, st, n,
                       S, cur, edges, p.T, (const int*)p.end, (const int*)p.pre, (const double2*)p.Zr, tie, amb, p.steps,
                       p.G);
    return hipGetLastError();
  };
  // Without timing, a full batch of iterations is captured once into a graph
  // and replayed (the launches' arguments do not change between
  // iterations; the state lives in the workspace).  No memset is captured.
  hipGraphExec_t bexec = nullptr;
  struct GraphGuard {
    hipGraphExec_t* e;
    ~GraphGuard() {
      if (*e) (void)hipGraphExecDestroy(*e);
    }
  } gguard{&bexec};
  if (!timing && st != nullptr && cap >= kBatch) {
    hipGraph_t graph = nullptr;
    OKRG_HIP(g, hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    hipError_t ce = hipSuccess;
    for (int t = 0; t < kBatch && ce == hipSuccess; ++t) ce = enqueue_iteration(t);
    const hipError_t ee = hipStreamEndCapture(st, &graph);
    if (ce != hipSuccess || ee != hipSuccess)
      OKRG_FAIL(g, OKR_E_HIP, "graph capture failed: %s", hipGetErrorString(ce != hipSuccess ? ce : ee));
    const hipError_t ie = hipGraphInstantiate(&bexec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ie != hipSuccess) OKRG_FAIL(g, OKR_E_HIP, "graph instantiate failed: %s", hipGetErrorString(ie));
  }
  while (enq < cap) {
    const int b = std::min(kBatch, cap - enq);
    if (bexec && b == kBatch) {
      OKRG_HIP(g, hipGraphLaunch(bexec, st));
    } else {
      for (int t = 0; t < b; ++t) OKRG_HIP(g, enqueue_iteration(t));
    }
    OKRG_HIP(g, hipGetLastError());
    const int before = hs.iter;
    OKRG_HIP(g, hipMemcpyAsync(&hs, p.G.gs[b & 1], sizeof(GState), hipMemcpyDeviceToHost, st));
    OKRG_HIP(g, hipStreamSynchronize(st));
    // score launches that did work: one per move, plus the one that found none
    const int ran = std::min(b, hs.iter - before + (hs.done ? 1 : 0));
    launches += ran;
    if (timing)
      for (int t = 0; t < ran; ++t) {
        float ms = 0.f;
        OKRG_HIP(g, hipEventElapsedTime(&ms, tev[2 * t], tev[2 * t + 1]));
        score_ms += ms;
      }
    enq += b;
    if (hs.done) break;
  }
  OKRG_HIP(g, hipEventRecord(ev[2], st));
  hipLaunchKernelGGL(k_greedy_err, dim3(S), dim3(kGreedyThreads), 0, st, n, (const uint8_t*)p.phase,
                     (const int*)p.sup, (const double2*)p.V, (const double*)p.absV, p.err);
  OKRG_HIP(g, hipGetLastError());
  std::vector<int> iters(S, 0);
  if (!(prm->flags & OKR_FLAG_VHAT_GIVEN))
    OKRG_HIP(g, hipMemcpyAsync(iters.data(), p.iters, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  std::vector<int> lsup(n);
  OKRG_HIP(g, hipMemcpyAsync(lsup.data(), p.sup, sizeof(int) * n, hipMemcpyDeviceToHost, st));
  rc = read_errors(g, p, out->err_per_snapshot);
  if (rc) return rc;
  for (int x = 0; x < n; ++x) out->super[x] = g->pre[lsup[g->pos[x]]];
  if (hs.iter > 0) {
    OKRG_HIP(g, hipMemcpyAsync(out->steps, p.steps, sizeof(GStep) * hs.iter, hipMemcpyDeviceToHost, st));
    OKRG_HIP(g, hipStreamSynchronize(st));
  }
  out->n_steps = hs.iter;
  out->n_kept = n - hs.iter;
  out->n_score_launches = launches;
  out->incremental = incremental ? 1 : 0;
  out->t_score_ms = score_ms;
  {
    int64_t sc = 0;
    for (int i = 0; i < hs.iter; ++i) sc += out->steps[i].n_cand;
    out->n_scored = sc;
  }
  double mx = 0.0;
  for (int l = 0; l < S; ++l) mx = std::max(mx, out->err_per_snapshot[l]);
  out->max_err = mx;
  float a = 0.f, b = 0.f;
  OKRG_HIP(g, hipEventElapsedTime(&a, ev[0], ev[1]));
  OKRG_HIP(g, hipEventElapsedTime(&b, ev[1], ev[2]));
  out->t_pf_ms = a;
  out->t_search_ms = b;
  int im = 0;
  for (int v : iters) im = std::max(im, v);
  out->pf_iterations = im;
  return OKR_OK;
}

extern "C" int okr_greedy_evaluate(okr_greedy* g, const okr_yblocks* Y, const okr_loads* L, const int32_t* super,
                                   const okr_greedy_params* prm, void* ws, double* err, double* max_err) {
  if (!g) return OKR_E_ARG;
  int rc = check_call(g, Y, L, prm, ws);
  if (rc) return rc;
  if (!super || !err) OKRG_FAIL(g, OKR_E_ARG, "null assignment or output");
  const int n = g->n, S = g->S;
  rc = check_assignment(g, super);
  if (rc) return rc;
  const GPtrs p = gptrs(g, ws);
  const hipStream_t st = g->stream;
  const double2* V0 = (const double2*)L->V0;
  std::vector<int> csr;
  assignment(g, super, csr);
  OKRG_HIP(g, hipMemcpyAsync(p.sup, csr.data(), sizeof(int) * csr.size(), hipMemcpyHostToDevice, st));
  const int *moff = p.csr, *mem = p.csr + n + 1;
  if (g->flow.form == 1 && !(prm->flags & OKR_FLAG_VHAT_GIVEN)) {
    // a scenario's load flow, aggregated currents, fixed-current solve and error
    // in one block (1000 nodes, 168 scenarios: 82 us; as four launches 116)
    const FlowEval e{moff, mem, p.sup, p.err};
    rc = setup(g, p, Y, L, prm, false, &e);
    if (rc) return rc;
  } else {
    rc = setup(g, p, Y, L, prm, false);
    if (rc) return rc;
    const size_t c3 = (size_t)S * n * 3;
    hipLaunchKernelGGL(k_greedy_aggregate, dim3((unsigned)((c3 + 255) / 256)), dim3(256), 0, st, n, S, moff, mem,
                       (const double2*)p.A, p.I);
    rc = fixed_solve(g, p, V0);
    if (rc) return rc;
    hipLaunchKernelGGL(k_greedy_err, dim3(S), dim3(kGreedyThreads), 0, st, n, (const uint8_t*)p.phase,
                       (const int*)p.sup, (const double2*)p.V, (const double*)p.absV, p.err);
    OKRG_HIP(g, hipGetLastError());
  }
  rc = read_errors(g, p, err);
  if (rc) return rc;
  if (max_err) {
    double mx = 0.0;
    for (int l = 0; l < S; ++l) mx = std::max(mx, err[l]);
    *max_err = mx;
  }
  return OKR_OK;
}

extern "C" int okr_greedy_radialize(okr_greedy* g, const okr_yblocks* Y, const okr_loads* L, const int32_t* super,
                                    const okr_greedy_params* prm, void* ws, uint8_t* kept_radial,
                                    int32_t* kept_parent, int32_t* n_critical, double* dv_radial,
                                    double* dv_meshed) {
  if (!g) return OKR_E_ARG;
  int rc = check_call(g, Y, L, prm, ws);
  if (rc) return rc;
  if (!super || !kept_radial || !kept_parent || !n_critical) OKRG_FAIL(g, OKR_E_ARG, "null assignment or output");
  rc = check_assignment(g, super);
  if (rc) return rc;
  const int n = g->n, S = g->S;
  const GPtrs p = gptrs(g, ws);
  const hipStream_t st = g->stream;
  rc = setup(g, p, Y, L, prm, true);
  if (rc) return rc;
  const double2* V0 = (const double2*)L->V0;
  std::vector<int> csr;
  assignment(g, super, csr);
  const int* moff = p.csr;
  OKRG_HIP(g, hipMemcpyAsync(p.sup, csr.data(), sizeof(int) * csr.size(), hipMemcpyHostToDevice, st));
  const size_t c3 = (size_t)S * n * 3;
  hipLaunchKernelGGL(k_greedy_aggregate, dim3((unsigned)((c3 + 255) / 256)), dim3(256), 0, st, n, S,
                     (const int*)moff, (const int*)(moff + n + 1), (const double2*)p.A, p.I);
  rc = fixed_solve(g, p, V0);
  if (rc) return rc;
  char* b = (char*)ws;
  int* rad = (int*)(b + g->o_rad);
  int *down = rad, *up = rad + n, *cnt = rad + 2 * n, *kp_rad = rad + 3 * n, *kp_mesh = rad + 4 * n;
  uint8_t* krad = (uint8_t*)(b + g->o_radk);
  unsigned long long* x = (unsigned long long*)(b + g->o_radx);  // [0] critical count, [1] dv radial, [2] dv meshed
  OKRG_HIP(g, hipMemsetAsync(x, 0, sizeof(unsigned long long) * 4, st));
  hipLaunchKernelGGL(k_radialize, dim3(1), dim3(kGreedyPickThreads), 0, st, n, (const int*)p.parent,
                     (const int*)p.ch_off, (const int*)p.ch, (const int*)p.lvl_off, (const int*)p.lvl_nodes, g->nlev,
                     (const int*)p.sup, down, up, cnt, krad, kp_rad, kp_mesh, (int*)x);
  // the check costs n x n per scenario: the first four scenarios suffice
  // (a missed critical node shows in any scenario that loads its branches)
  const int Sc = std::min(S, 4);
  const unsigned nb = (unsigned)(((size_t)n * Sc + kGreedyThreads - 1) / kGreedyThreads);
  hipLaunchKernelGGL(k_radial_check, dim3(nb), dim3(kGreedyThreads), 0, st, n, Sc, (const uint8_t*)p.phase, (const int*)p.pos,
                     p.T,
                     (const double2*)p.Zr, (const int*)p.sup, (const uint8_t*)krad, (const int*)kp_rad, 1,
                     (const double2*)p.I, (const double2*)p.V, V0[0], V0[1], V0[2], x + 1);
  hipLaunchKernelGGL(k_radial_check, dim3(nb), dim3(kGreedyThreads), 0, st, n, Sc, (const uint8_t*)p.phase, (const int*)p.pos,
                     p.T,
                     (const double2*)p.Zr, (const int*)p.sup, (const uint8_t*)krad, (const int*)kp_mesh, 0,
                     (const double2*)p.I, (const double2*)p.V, V0[0], V0[1], V0[2], x + 2);
  OKRG_HIP(g, hipGetLastError());
  int status[4] = {0, 0, 0, 0};
  unsigned long long hx[4] = {0, 0, 0, 0};
  OKRG_HIP(g, hipMemcpyAsync(status, p.status, sizeof(status), hipMemcpyDeviceToHost, st));
  OKRG_HIP(g, hipMemcpyAsync(hx, x, sizeof(hx), hipMemcpyDeviceToHost, st));
  std::vector<uint8_t> hk(n);
  std::vector<int> hp(n);
  OKRG_HIP(g, hipMemcpyAsync(hk.data(), krad, n, hipMemcpyDeviceToHost, st));
  OKRG_HIP(g, hipMemcpyAsync(hp.data(), kp_rad, sizeof(int) * n, hipMemcpyDeviceToHost, st));
  OKRG_HIP(g, hipStreamSynchronize(st));
  rc = check_status(g, status[0]);
  if (rc) return rc;
  for (int q = 0; q < n; ++q) {  // labels to the caller's ids
    kept_radial[g->pre[q]] = hk[q];
    kept_parent[g->pre[q]] = hp[q] < 0 ? -1 : g->pre[hp[q]];
  }
  int nc;
  std::memcpy(&nc, &hx[0], sizeof(int));
  *n_critical = nc;
  double d1, d2;
  std::memcpy(&d1, &hx[1], sizeof(double));
  std::memcpy(&d2, &hx[2], sizeof(double));
  if (dv_radial) *dv_radial = d1;
  if (dv_meshed) *dv_meshed = d2;
  return OKR_OK;
}
