// Device helpers shared by the FP64 scoring and refine kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "okr_internal.h"

namespace okr {

// ---------------------------------------------------------------- complex --
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
  const double d = cabs2(b);
  const double2 t = cmul(a, cconj(b));
  return make_double2(t.x / d, t.y / d);
}
// Note: the bare v_sqrt_f64 instruction is accurate to only about 2^-27
// relative, far outside the 1e-13 decision window; magnitudes in the scoring
// use sqrt_nr() below, elsewhere the libm sqrt.

// ---------------------------------------------------------------- scoring --
// sqrt for arguments in the normal range (here |V|^2 of a bus voltage): the
// hardware reciprocal-square-root estimate (relative error about 2^-24)
// refined by one Newton-Raphson step in Goldschmidt form (g -> sqrt(x),
// h -> 1/(2 sqrt(x)); error about 2^-48) and one residual correction
// g + (x - g^2) h, which leaves it within an ulp (the rounding test checks it
// against libm).  No range scaling: callers pass x in [2^-500, 2^500].
__device__ __forceinline__ double sqrt_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  double g = x * r, h = 0.5 * r;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  const double d = fma(-g, g, x);
  return fma(d, h, g);
}
// |a|^2 in one fixed evaluation order (every magnitude of the scoring goes
// through it, so all scoring forms round alike).
__device__ __forceinline__ double mag2(double2 a) { return fma(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ double vmag(double2 a) { return sqrt_nr(mag2(a)); }

// Walk one chain for one mask: super-node slots top to bottom; a reduced slot
// adds the voltage rise of moving its aggregated current to its current super
// (P from LDS); a kept slot becomes the super of the slots below it.  With ERR,
// every slot cluster's error against its super's magnitude is folded into el, and
// the squared magnitudes of kept slots into (qmin, qmax) for the band (the slack
// is formed once per mask: sqrt is monotone, so min(|V| - vmin) =
// sqrt(min |V|^2) - vmin exactly).  Slot r of the chain has mask bit
// C_BIT0 + r, pairs from C_PAIR0 + r(r+1)/2 and its phases in the C_PHW words.
template <bool ERR>
__device__ __forceinline__ void walk_chain(const int* __restrict__ cr, const double2* Ps, const TargetRec* Ss,
                                           const double2* Hs, int c, uint32_t m, double2 (&B)[3], double& el,
                                           double& qmin, double& qmax) {
  double sm[3] = {0.0, 0.0, 0.0};
  if (ERR) {
    const int hph = cr[C_PHASE];
    const bool inner = cr[C_OUTER] >= 0;  // (else the head is unaffected by the mask)
#pragma unroll
    for (int p = 0; p < 3; ++p)
      if (hph >> p & 1) sm[p] = vmag(inner ? cadd(Hs[c * 3 + p], B[p]) : Hs[c * 3 + p]);
  }
  const int ns = cr[C_NSLOT], s0 = cr[C_SLOT0], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
  const int phw0 = cr[C_PHW0], phw1 = cr[C_PHW1], phw2 = cr[C_PHW2];
  int sidx = 0;
  for (int r = 0; r < ns; ++r) {
    const int w = r < 8 ? phw0 : (r < 16 ? phw1 : phw2);
    const int ph = (w >> (3 * (r & 7))) & 7;
    const TargetRec* tr = Ss + (s0 + r) * 3;
    const bool red = (m >> (bit0 + r)) & 1u;
    const double rf = red ? 1.0 : 0.0;
    const double2* pr = Ps + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (!(ph >> p & 1)) continue;
      const double2 pv = pr[p];
      B[p].x = fma(rf, pv.x, B[p].x);
      B[p].y = fma(rf, pv.y, B[p].y);
      if (ERR) {
        const TargetRec t = tr[p];
        const double vx = t.W.x + B[p].x, vy = t.W.y + B[p].y;
        const double q = fma(vx, vx, vy * vy);
        if (!red) sm[p] = sqrt_nr(q);
        qmin = fmin(qmin, red ? INFINITY : q);
        qmax = fmax(qmax, red ? -INFINITY : q);
        el = fmax(el, fmax(sm[p] - t.lo, t.hi - sm[p]));
      }
    }
    sidx = red ? sidx : r + 1;
  }
}

// The mask's bits at pm's positions, gathered (run by run).
__device__ __forceinline__ uint32_t gather_bits(uint32_t m, uint32_t pm) {
  uint32_t u = 0;
  int j = 0;
  while (pm) {
    const int b = __builtin_ctz(pm);
    const int run = __builtin_ctz(~(pm >> b));
    const uint32_t ones = (1u << run) - 1u;
    u |= ((m >> b) & ones) << j;
    j += run;
    pm &= ~(ones << b);
  }
  return u;
}

// Band slack of a mask from the extreme squared magnitudes of its kept
// node-phases: min(|V| - vmin, vmax - |V|) over them (+inf if there are none).
__device__ __forceinline__ double band_slack(double qmin, double qmax, double vmin, double vmax) {
  const double a = qmin < INFINITY ? sqrt_nr(qmin) - vmin : INFINITY;
  const double b = qmax > 0.0 ? vmax - sqrt_nr(qmax) : INFINITY;
  return fmin(a, b);
}

__device__ __forceinline__ bool feasible(const MaskScore& r, double e_bar) { return r.e <= e_bar && r.slack >= 0.0; }
__device__ __forceinline__ bool near_boundary(const MaskScore& r, double e_bar, double amb) {
  const bool rin = r.e <= e_bar - amb && r.slack >= amb;
  const bool rout = r.e > e_bar + amb || r.slack < -amb;
  return !rin && !rout;
}

// Terms of chain c for one mask and one snapshot folded into el, kept squared
// magnitudes into (qmin, qmax): the nesting path walked to the chain's head
// (voltage rises only), the chain's own slots, then the zone entries anchored
// below it (the first zcap of them from the LDS stage Zs, the rest from global
// memory).  They depend on the mask bits in C_PMASK only.
__device__ __forceinline__ void score_chain(const int* __restrict__ chains, const int* __restrict__ nest, int c,
                                            const double2* Ps, const TargetRec* Ss, const double2* Hs,
                                            const TargetRec* Zs, int zcap, const TargetRec* __restrict__ zrec_l,
                                            uint32_t m, double& el, double& qmin, double& qmax) {
  const int* cr = chains + c * kChainInts;
  double2 B[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) B[p] = make_double2(0.0, 0.0);
  const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
  for (int q = 0; q + 1 < nl; ++q)
    walk_chain<false>(chains + nest[no + q] * kChainInts, Ps, Ss, Hs, nest[no + q], m, B, el, qmin, qmax);
  walk_chain<true>(cr, Ps, Ss, Hs, c, m, B, el, qmin, qmax);
#pragma unroll
  for (int p = 0; p < 3; ++p)
    for (int q = cr[C_ZOFF0 + p], qe = q + cr[C_ZCNT0 + p]; q < qe; ++q) {
      TargetRec t;
      if (q < zcap) t = Zs[q];
      else t = zrec_l[q];
      const double vx = t.W.x + B[p].x, vy = t.W.y + B[p].y;
      const double q2 = fma(vx, vx, vy * vy);
      const double mag = sqrt_nr(q2);
      el = fmax(el, fmax(mag - t.lo, t.hi - mag));
      qmin = fmin(qmin, q2);
      qmax = fmax(qmax, q2);
    }
}

// Orders a wave's own LDS accesses (no other wave takes part).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sum of an int over the first 32 lanes, or the whole wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, ROWS == 0xf);
}
__device__ __forceinline__ int scan32(int v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  return dpp_add<0x142, 0xa>(v);
}
__device__ __forceinline__ int scan64(int v) { return dpp_add<0x143, 0xc>(scan32(v)); }

// ------------------------------------------------------------- SMICE prep --
// Node of Omega_g with flattened index q (ranges: start, end, cumulative).
__device__ __forceinline__ int omega_node(const int* rg, int nr, int q) {
  int r = 0;
  while (r + 1 < nr && rg[3 * (r + 1) + 2] <= q) ++r;
  return rg[3 * r] + (q - rg[3 * r + 2]);
}

// Zone entry of the lowest present phase of node i, or -1 if i is not a
// zone target of this segment.
__device__ __forceinline__ int sm_first_entry(const Topo& T, const State& St, int i, int nz) {
  const unsigned ph = T.phase[i];
  for (int p = 0; p < 3; ++p)
    if (ph >> p & 1u) {
      const int e = St.zent_of[i * 3 + p];
      return (e >= 0 && e < nz) ? e : -1;
    }
  return -1;
}

// The chains' distinct heads in chain order, by wave 0: hnode, hin (1: the head
// lies below another chain) and their number; returns the head number of the
// lane's chain.  (LDS outputs; a barrier is up to the caller.)
__device__ __forceinline__ int distinct_heads(const SegHdr& H, const int* tab, int* hnode, int* hin, int* nh) {
  const int lane = threadIdx.x & 63, nch = H.nchains;
  int head = -1, outer = -1, first = lane;
  if (lane < nch) {
    head = tab[H.o_chain + lane * kChainInts + C_HEAD];
    outer = tab[H.o_chain + lane * kChainInts + C_OUTER];
  }
  for (int q = nch - 1; q >= 0; --q)
    if (q < lane && __builtin_amdgcn_readlane(head, q) == head) first = q;
  const uint32_t firsts = (uint32_t)__ballot(lane < nch && first == lane);
  const int x = __popc(firsts & ((1u << (first & 31)) - 1u));  // the head's number
  if (lane < nch && first == lane) {
    hnode[x] = head;
    hin[x] = outer >= 0 ? 1 : 0;
  }
  if (lane == 0) *nh = __popc(firsts);
  return x;
}

// Fixed error of the cluster of every head outside Omega_g in snapshot l (one
// block): the largest error over its members (every node whose super-node it is,
// itself included) and their phases, against its unchanging voltage.
__device__ __forceinline__ void smice_hconst(const SegHdr& H, const int* tab, const Topo& T, const State& St,
                                             const double2* Vcur, const double* absV, double* hK, int S, int l) {
  __shared__ int c_hnode[kMaxK], c_hin[kMaxK], c_nh;
  __shared__ unsigned long long c_max[kMaxK];
  if (!H.valid) return;
  if (threadIdx.x < 64) distinct_heads(H, tab, c_hnode, c_hin, &c_nh);
  if (threadIdx.x < kMaxK) c_max[threadIdx.x] = 0ull;
  __syncthreads();
  const int n = T.n, nh = c_nh;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int sp = St.sup[i];
    int x = -1;
    for (int y = 0; y < nh; ++y)
      if (c_hnode[y] == sp && !c_hin[y]) x = y;
    if (x < 0) continue;
    const unsigned ph = T.phase[i];
    double e = 0.0;
    for (int p = 0; p < 3; ++p)
      if (ph >> p & 1u)
        e = fmax(e, fabs(vmag(Vcur[((size_t)l * n + sp) * 3 + p]) - absV[((size_t)l * n + i) * 3 + p]));
    atomicMax(&c_max[x], (unsigned long long)__double_as_longlong(e));
  }
  __syncthreads();
  if ((int)threadIdx.x < nh) hK[threadIdx.x * S + l] = __longlong_as_double((long long)c_max[threadIdx.x]);
}

// A segment's SMICE tables (one block of up to 1024 threads): distinct heads in
// chain order, zone targets grouped by anchor chain in Omega_g order.  With the
// heads' fixed errors, further blocks of the arg-min's launch: they read nothing
// of each other's (as launches of their own, one thread looping over the heads, a
// serial sum over 256 threads' counts and atomics into memory, 11 and 4.6 us per
// chunk at 1000 nodes).
__device__ __forceinline__ void smice_prep(const SegHdr& H, const int* tab, const Topo& T, const State& St, int* stab) {
  __shared__ int s_hnode[kMaxK], s_hin[kMaxK], s_nh, s_cnt[kMaxK], s_run[kMaxK], s_w[16][kMaxK];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
  if (!H.valid) {
    if (tid == 0) {
      stab[SM_NH] = 0;
      stab[SM_NZN] = 0;
    }
    return;
  }
  const int nch = H.nchains, nom = H.nomega;
  if (wv == 0) {
    const int x = distinct_heads(H, tab, s_hnode, s_hin, &s_nh);
    if (lane < nch) {
      stab[SM_CHX + lane] = x;
      s_cnt[lane] = 0;
    }
  }
  __syncthreads();
  const int nh = s_nh;
  if (tid == 0) stab[SM_NH] = nh;
  if (tid < nh) {
    stab[SM_HNODE + tid] = s_hnode[tid];
    stab[SM_HIN + tid] = s_hin[tid];
  }
  const int* rg = tab + H.o_range;
  auto anchor = [&](int q, int& i) {  // anchor chain of Omega_g node q, -1: no target
    i = omega_node(rg, H.nrange, q);
    const int e = sm_first_entry(T, St, i, H.nz);
    return e >= 0 ? tab[H.o_zent + 3 * e + 2] : -1;
  };
  int node = 0, at = tid < nom ? anchor(tid, node) : -1;
  for (int q = tid; q < nom; q += blockDim.x) {
    int i = node;
    const int c = q == tid ? at : anchor(q, i);
    if (c >= 0) atomicAdd(&s_cnt[c], 1);
  }
  __syncthreads();
  if (wv == 0) {
    const int v = lane < nch ? s_cnt[lane] : 0, x = scan32(v);
    if (lane < nch) stab[SM_ZOFF + lane] = s_run[lane] = x - v;
    if (lane == nch - 1) stab[SM_ZOFF + nch] = stab[SM_NZN] = x;
  }
  __syncthreads();
  for (int q = tid; q - tid < nom; q += blockDim.x) {  // (rounds of the whole block, in order)
    int c = -1;
    if (q < nom) c = q == tid ? at : anchor(q, node);
    int rank = 0;
    for (int y = 0; y < nch; ++y) {
      const unsigned long long b = __ballot(c == y);
      if (c == y) rank = __popcll(b & ((1ull << lane) - 1ull));
      if (lane == 0) s_w[wv][y] = __popcll(b);
    }
    __syncthreads();
    if (c >= 0) {
      int to = s_run[c] + rank;
      for (int w = 0; w < wv; ++w) to += s_w[w][c];
      int* zr = stab + SM_ZREC + to * kZrecInts;
      zr[0] = node;
      const unsigned ph = T.phase[node];
      for (int p = 0; p < 3; ++p) {
        const int ep = St.zent_of[node * 3 + p];
        zr[1 + p] = ((ph >> p & 1u) && ep >= 0 && ep < H.nz) ? ep : -1;
      }
      int hx = -1;
      for (int x = 0; x < nh; ++x)
        if (s_hnode[x] == node) hx = x;
      zr[4] = hx;
    }
    __syncthreads();
    if (tid < nch)
      for (int w = 0; w < nw; ++w) s_run[tid] += s_w[w][tid];
    __syncthreads();
  }
}

// ---------------------------------------------------------- state update --
// The structural part of applying a mask to segment H (one block, called by
// every thread): kept flags and super-nodes over Omega_g, and the node -> slot
// and zone-entry maps cleared for the next segment.  Run by the kernel that
// settles the decision, so that the next chunk's table build can start while
// the voltages and currents of this one are still being moved.
// Before the decision (load): a slot is a kept node, its nearest kept proper
// ancestor is another slot or stays kept, and a node's super-node is a slot or
// stays.  After it (store): a reduced slot's super-node is found over the slots
// in LDS, and each node takes its old super-node's.  Climbing the tree in
// memory after the decision took 2.3 us of the 10.1 us arg-min at 1000 nodes.
struct StateUpdate {
  int up[kMaxK], upnode[kMaxK], node[kMaxK], bit[kMaxK];  // (LDS)
  // i, s, js: this thread's first node of Omega_g, its super-node and that
  // one's slot.  Ends with the map reads done (before the caller's barrier).
  __device__ __forceinline__ void load(const SegHdr& H, const int* tab, const Topo& T, const State& St, int& i, int& s,
                                       int& js) {
    const int* slots = tab + H.o_slot;
    i = s = js = -1;
    if ((int)threadIdx.x < H.nomega) {
      i = omega_node(tab + H.o_range, H.nrange, threadIdx.x);
      s = St.sup[i];
      js = St.slot_of[s];
    }
    if ((int)threadIdx.x < H.nslots) {
      const int* sr = slots + threadIdx.x * kSlotInts;
      node[threadIdx.x] = sr[SL_NODE];
      bit[threadIdx.x] = sr[SL_BIT];
      const int a = St.sup[T.parent[sr[SL_NODE]]];  // (the slack is no slot)
      upnode[threadIdx.x] = a;
      up[threadIdx.x] = St.slot_of[a];
    }
  }
  // Slot j's super-node under mask m (after a barrier behind load).
  __device__ __forceinline__ int super_of(int j, uint32_t m) const {
    int v = node[j];
    while (j >= 0 && ((m >> bit[j]) & 1u)) {
      v = upnode[j];
      j = up[j];
    }
    return v;
  }
  __device__ __forceinline__ void store(const SegHdr& H, const int* tab, const State& St, uint32_t m, int i, int s,
                                        int js) const {
    if (i >= 0 && js >= 0) {
      const int v = super_of(js, m);
      if (v != s) St.sup[i] = v;
    }
    for (int q = threadIdx.x + blockDim.x; q < H.nomega; q += blockDim.x) {
      const int x = omega_node(tab + H.o_range, H.nrange, q), y = St.sup[x], j = St.slot_of[y];
      if (j >= 0) St.sup[x] = super_of(j, m);
    }
    __syncthreads();  // the slot map is read
    if ((int)threadIdx.x < H.nslots) {
      if ((m >> bit[threadIdx.x]) & 1u) St.kept[node[threadIdx.x]] = 0;
      St.slot_of[node[threadIdx.x]] = -1;
    }
    for (int q = threadIdx.x; q < H.nz; q += blockDim.x) {
      const int* ze = tab + H.o_zent + q * 3;
      St.zent_of[ze[0] * 3 + ze[1]] = -1;
    }
  }
};

// ------------------------------------------------------------ block reduce --
// The larger of two non-negative values, NaN if either is (the bit patterns
// order like the values, with every NaN above infinity).
__device__ __forceinline__ double nan_max(double a, double b) {
  return (unsigned long long)__double_as_longlong(a) > (unsigned long long)__double_as_longlong(b) ? a : b;
}

template <typename T>
__device__ __forceinline__ T shfl_xor_of(T v, int o) {
  return __shfl_xor(v, o, 64);
}

template <typename T, typename Op>
__device__ T block_reduce(T v, Op op, T* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  for (int o = 32; o > 0; o >>= 1) v = op(v, shfl_xor_of(v, o));
  __syncthreads();
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  T r = sh[0];
  for (int w = 1; w < nw; ++w) r = op(r, sh[w]);
  __syncthreads();
  return r;
}

}  // namespace okr
