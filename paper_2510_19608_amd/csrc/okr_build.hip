// Device-side construction of one segment's tables from the cumulative kept
// state (no host round trip between segments), and the numeric state update of
// the segments decided before it.
//
//   build_struct    (1 block)  chains, slots, pairs, nesting, Omega ranges,
//                              zone entries grouped by (chain, phase)
//
// The numeric tables that follow from them (per snapshot) are built by
// k_seg_terms (okr_score.hip).
//
// The tables have the layout the scoring kernel reads (okr_internal.h).
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "okr_internal.h"

namespace okr {

constexpr int kOmegaLds = 4096;  // Omega_g nodes whose zone classification is kept in shared memory
// structural part of a segment's tables (chains, nesting, slots, pairs, ranges)
constexpr int kTabLds = kMaxK * kChainInts + kMaxK * kMaxK + kMaxK * kSlotInts + kMaxPairs * kPairInts + 3 * kMaxK;

// Child of kept node h on the tree path down to its descendant v.
__device__ __forceinline__ int child_toward(const Topo& T, int h, int v) {
  for (int q = T.ch_off[h]; q < T.ch_off[h + 1]; ++q) {
    const int x = T.ch[q];
    if (x <= v && v < x + T.size[x]) return x;
  }
  return -1;
}

__device__ __forceinline__ void build_struct(Topo T, State St, const int* __restrict__ segs, int z, size_t lstride,
                                                      int S, SegHdr* __restrict__ hdrs, int* __restrict__ tab,
                                                      int tab_cap, int* __restrict__ status,
                                                      unsigned long long* __restrict__ pat,
                                                      unsigned long long* __restrict__ ecmax,
                                                      int2* __restrict__ pat32) {
  __shared__ int s_top[kMaxK], s_slotnode[kMaxK], s_slotbit[kMaxK], s_slotchain[kMaxK];
  __shared__ int s_cslot0[kMaxK + 1], s_head[kMaxK], s_outer[kMaxK], s_jslot[kMaxK];
  __shared__ int s_spos[kMaxK], s_ssize[kMaxK], s_sph[kMaxK];           // segment node j
  __shared__ int s_tpos[kMaxK], s_tsize[kMaxK], s_thead[kMaxK], s_thph[kMaxK];  // its chain top
  __shared__ int s_cpos[kMaxK], s_csize[kMaxK], s_chph[kMaxK];          // chain c: top pos/size, head phase
  __shared__ int s_rs[kMaxK], s_rcum[kMaxK + 1];                       // Omega_g ranges: start, cumulative size
  __shared__ int s_seg[kMaxK], s_thpos[kMaxK], s_first[kMaxK];          // segment node j, its top's head position,
                                                                        // first segment node with its top
  __shared__ int s_chpos[kMaxK], s_rkeep[kMaxK], s_depth[kMaxK];        // chain c: head position, new range, nesting
  __shared__ int s_pmask[kMaxK];                                        // chain c: mask bits of its nesting path
  __shared__ int s_okey[kMaxK];  // chain c: (preorder position << 5) | j of the deepest segment node above its head
  // exclusive prefix sums over the chains (entry nch: the totals) of: nesting
  // depth, pairs, new Omega_g range, its nodes, chain patterns
  __shared__ int s_xs[5][kMaxK + 1];
  __shared__ int s_keycnt[kMaxK * 3], s_keyoff[kMaxK * 3], s_keycur[kMaxK * 3];
  __shared__ SegHdr s_h;
  __shared__ int s_err, s_nch;
  __shared__ int s_zi[kOmegaLds], s_zk[kOmegaLds];  // zone pass: node and key of Omega index q
  __shared__ int s_tab[kTabLds];                     // structural tables before they are written out
  const int g = segs[z];
  tab = lane_ptr_z(tab, lstride, z);
  const int* parent = T.parent;
  const int* segment = T.segment;
  const int tid = threadIdx.x;
  const int o0 = T.seg_off[g];
  const int k = T.seg_off[g + 1] - o0;
  if (tid == 0) {
    // an earlier segment failed: leave every later one invalid (its scratch
    // maps may be stale)
    s_err = ((*status & kStatusBuild) || k < 1 || k > kMaxK) ? 1 : 0;
    s_nch = 0;
  }
  if (tid < kMaxK) {
    s_okey[tid] = -1;
    s_rkeep[tid] = 1;
  }
  __syncthreads();
  // chain top of every segment node: the highest node above it reachable
  // through segment or reduced nodes (runs of reduced nodes are crossed in
  // one step: their nearest kept ancestor is known)
  if (!s_err && tid < k) {
    const int e = T.seg_nodes[o0 + tid];
    int c = T.seg_top[e], guard = 0;  // (runs of this segment's nodes climbed at plan time)
    for (;;) {
      const int p = parent[c];
      if (p < 0 || ++guard > T.n) break;
      if (segment[p] == g) { c = T.seg_top[p]; continue; }
      if (St.kept[p]) break;
      const int h = St.sup[p];
      const int x = (h >= 0 && h != p) ? child_toward(T, h, p) : -1;
      if (x < 0) { atomicOr(&s_err, 1); break; }
      c = x;
    }
    s_top[tid] = c;
    s_spos[tid] = e;
    s_ssize[tid] = T.size[e];
    s_sph[tid] = T.phase[e];
    const int hd = parent[c];
    s_tpos[tid] = c;
    s_tsize[tid] = T.size[c];
    s_thead[tid] = hd;
    s_thph[tid] = hd >= 0 ? T.phase[hd] : 0;
    s_thpos[tid] = hd;
    s_seg[tid] = e;
  }
  __syncthreads();
  // chains: one per distinct chain top, ordered by the tops' preorder
  // positions (distinct nodes, so the order is strict); slots chain by chain,
  // top to bottom (segment nodes are in preorder).  One thread per segment
  // node, shared-memory data only from here on.
  if (!s_err && tid < k) {
    const int top = s_top[tid];
    int j0 = tid;  // first segment node with this chain top
    for (int q = tid - 1; q >= 0; --q)
      if (s_top[q] == top) j0 = q;
    s_first[tid] = j0;
  }
  __syncthreads();
  if (!s_err && tid < k) {
    const int j = tid, j0 = s_first[j], tp = s_tpos[j];
    int c = 0, before = 0, within = 0, nch = 0;
    for (int q = 0; q < k; ++q) {
      const bool lower = s_tpos[q] < tp;  // q's chain comes before j's
      const bool opens = s_first[q] == q;
      nch += opens;
      c += opens && lower;
      before += lower;
      within += (s_first[q] == j0) && q < j;
    }
    const int s = before + within;
    s_jslot[j] = s;
    s_slotnode[s] = s_seg[j];
    s_slotbit[s] = j;
    s_slotchain[s] = c;
    if (j0 == j) {
      s_cpos[c] = tp;
      s_csize[c] = s_tsize[j];
      s_chph[c] = s_thph[j];
      s_head[c] = s_thead[j];
      s_chpos[c] = s_thpos[j];
      s_cslot0[c] = before;
    }
    if (j == 0) {
      s_nch = nch;
      s_cslot0[nch] = k;
    }
  }
  __syncthreads();
  // per chain: the outer chain (whose bottom slot is the deepest segment node
  // above the head), the path and consecutive-bit invariants, and whether its
  // top's subtree starts a new Omega_g range (laminar intervals in preorder:
  // a top inside an earlier top's subtree adds nothing)
  const int nch = s_nch;
  // over (chain, segment node) pairs: the deepest segment node whose subtree
  // holds the chain's head (positions are distinct, so the largest key is
  // that node); over (chain, earlier chain) pairs: whether the chain's top
  // lies in an earlier chain top's subtree (then it starts no new range)
  if (!s_err) {
    for (int x = tid; x < nch * k; x += blockDim.x) {
      const int c = x / k, j = x - c * k, ph = s_chpos[c];
      if (ph >= 0 && s_spos[j] <= ph && ph < s_spos[j] + s_ssize[j]) atomicMax(&s_okey[c], (s_spos[j] << 5) | j);
    }
    for (int x = tid; x < nch * nch; x += blockDim.x) {
      const int c = x / nch, q = x - c * nch;
      if (q < c && s_cpos[q] <= s_cpos[c] && s_cpos[c] < s_cpos[q] + s_csize[q]) s_rkeep[c] = 0;
    }
  }
  __syncthreads();
  if (!s_err && tid < nch) {
    const int c = tid;
    const int best = s_okey[c] >= 0 ? (s_okey[c] & 31) : -1;
    int oc = -1;
    if (best >= 0) {
      const int s = s_jslot[best];
      oc = s_slotchain[s];
      if (s != s_cslot0[oc + 1] - 1 || oc >= c) atomicOr(&s_err, 1);
    }
    s_outer[c] = oc;
    // every chain is a path: each slot lies below the previous one (the first
    // below the chain top); its nodes have at most one child, so its slots
    // are consecutive segment nodes in preorder: consecutive mask bits
    int pu = s_cpos[c], su = s_csize[c];
    const int s0 = s_cslot0[c], s1 = s_cslot0[c + 1];
    for (int s = s0; s < s1; ++s) {
      const int j = s_slotbit[s], pv = s_spos[j];
      if (!(pu <= pv && pv < pu + su) || (s > s0 && pv == pu) || j != s_slotbit[s0] + (s - s0))
        atomicOr(&s_err, 1);
      pu = pv;
      su = s_ssize[j];
    }
  }
  __syncthreads();
  if (tid < nch) {
    // nesting depth (outer chains have smaller indices) and the mask bits of
    // the chains on the nesting path, the chain itself included
    int d = 0, pm = 0;
    if (!s_err)
      for (int x = tid; x >= 0; x = s_outer[x]) {
        ++d;
        pm |= ((1 << (s_cslot0[x + 1] - s_cslot0[x])) - 1) << s_slotbit[s_cslot0[x]];
      }
    s_depth[tid] = d;
    s_pmask[tid] = pm;
  }
  __syncthreads();
  // the chains' table offsets: prefix sums in one wave (lane = chain)
  if (tid < 64) {
    int v[5] = {0, 0, 0, 0, 0};
    if (tid < nch) {
      const int n = s_cslot0[tid + 1] - s_cslot0[tid];
      v[0] = s_depth[tid];
      v[1] = n * (n + 1) / 2;
      v[2] = s_rkeep[tid];
      v[3] = s_rkeep[tid] ? s_csize[tid] : 0;
      v[4] = 1 << __popc(s_pmask[tid]);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      int x = v[i];
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (tid >= o) x += y;
      }
      if (tid <= nch) s_xs[i][tid] = x - v[i];
    }
  }
  __syncthreads();
  // table layout
  const int nest_tot = s_xs[0][nch], npairs = s_xs[1][nch], nr = s_xs[2][nch], nom = s_xs[3][nch],
            npat = s_xs[4][nch];
  const int o_nest = nch * kChainInts, o_slot = o_nest + nest_tot, o_pair = o_slot + k * kSlotInts;
  const int o_range = o_pair + npairs * kPairInts, o_zent = o_range + 3 * nr;
  if (tid == 0) {
    SegHdr H;
    for (int q = 0; q < (int)(sizeof(SegHdr) / sizeof(int)); ++q) ((int*)&H)[q] = 0;
    H.g = g;
    H.k = k;
    H.S = S;
    H.o_chain = 0;
    H.o_nest = o_nest;
    H.o_slot = o_slot;
    H.o_pair = o_pair;
    H.o_range = o_range;
    H.o_zent = o_zent;
    H.nrange = nr;
    H.nomega = nom;
    H.nchains = nch;
    H.nslots = k;
    H.npairs = npairs;
    H.npat = npat;
    // the structural part must fit the segment's table (and the shared image,
    // which holds the largest possible one)
    if (o_zent > tab_cap || o_zent > kTabLds) s_err = 1;
    // the chain patterns number at most 2^(k+1) (a nesting forest whose
    // chains hold k bits in all): the pattern table's capacity
    if (npat > (2 << k)) s_err = 1;
    H.valid = s_err ? 0 : 1;
    s_h = H;
  }
  if (tid < kMaxK * 3) {
    s_keycnt[tid] = 0;
    s_keycur[tid] = 0;
  }
  __syncthreads();
  if (s_err) {
    if (tid == 0) {
      SegHdr H = s_h;
      H.valid = 0;
      hdrs[g] = H;
      atomicOr(status, kStatusBuild);
    }
    return;
  }
  // records: one thread per chain, one per slot
  if (tid < nch) {
    const int c = tid, s0 = s_cslot0[c], n = s_cslot0[c + 1] - s0;
    const int nest_off = s_xs[0][c], pair0 = s_xs[1][c], ridx = s_xs[2][c], rcum = s_xs[3][c], pbase = s_xs[4][c];
    const int d = s_depth[c];
    int q = d - 1;
    for (int x = c; x >= 0; x = s_outer[x]) s_tab[o_nest + nest_off + q--] = x;
    if (s_rkeep[c]) {
      s_tab[o_range + 3 * ridx] = s_cpos[c];
      s_tab[o_range + 3 * ridx + 1] = s_cpos[c] + s_csize[c];
      s_tab[o_range + 3 * ridx + 2] = rcum;
    }
    int phw[3] = {0, 0, 0};
    for (int r = 0; r < n; ++r) phw[r >> 3] |= s_sph[s_slotbit[s0 + r]] << (3 * (r & 7));
    int* cr = s_tab + c * kChainInts;
    cr[C_HEAD] = s_head[c];
    cr[C_NSLOT] = n;
    cr[C_SLOT0] = s0;
    cr[C_NEST_OFF] = nest_off;
    cr[C_NEST_LEN] = d;
    cr[C_OUTER] = s_outer[c];
    cr[C_PHASE] = s_chph[c];
    cr[C_BIT0] = s_slotbit[s0];
    cr[C_PAIR0] = pair0;
    cr[C_PHW0] = phw[0];
    cr[C_PHW1] = phw[1];
    cr[C_PHW2] = phw[2];
    cr[C_PMASK] = s_pmask[c];
    cr[C_PBASE] = pbase;
    for (int p = 0; p < 3; ++p) {
      cr[C_ZOFF0 + p] = 0;  // zone ranges filled after the zone pass
      cr[C_ZCNT0 + p] = 0;
    }
  }
  if (tid < k) {
    // slot s = r-th slot of chain c: pairs (super, reduced) with the super
    // node the head or one of the r slots above it
    const int s = tid, c = s_slotchain[s], s0 = s_cslot0[c], r = s - s0;
    const int pb = s_xs[1][c] + r * (r + 1) / 2;
    int* sr = s_tab + o_slot + s * kSlotInts;
    sr[SL_NODE] = s_slotnode[s];
    sr[SL_BIT] = s_slotbit[s];
    sr[SL_PHASE] = s_sph[s_slotbit[s]];
    sr[SL_PAIRBASE] = pb;
    sr[SL_CHAIN] = c;
    for (int sx = 0; sx <= r; ++sx) {
      int* pr = s_tab + o_pair + (pb + sx) * kPairInts;
      pr[PR_RNODE] = s_slotnode[s];
      pr[PR_SUPER] = (sx == 0) ? s_head[c] : s_slotnode[s0 + sx - 1];
      pr[PR_RSLOT] = s;
    }
    St.slot_of[s_slotnode[s]] = s;
  }
  __syncthreads();
  // the pattern accumulators the scoring folds into (error, smallest and
  // largest kept squared magnitude of each pattern; the largest constant
  // error): cleared here, where their number is first known, which saves the
  // scoring a launch of its own (4.3 us per chunk)
  pat = lane_ptr_z(pat, lstride, z);
  for (int q = tid; q < npat; q += blockDim.x) {
    pat[3 * q] = 0ull;
    pat[3 * q + 1] = (unsigned long long)__double_as_longlong(INFINITY);
    pat[3 * q + 2] = 0ull;
  }
  if (pat32) {  // the FP32 screen's (error, ordered bits of the slack)
    pat32 = lane_ptr_z(pat32, lstride, z);
    for (int q = tid; q < npat; q += blockDim.x) pat32[q] = make_int2(0, __float_as_int(INFINITY));
  }
  if (tid == 0) *lane_ptr_z(ecmax, lstride, z) = 0ull;
  // the structural tables, built in shared memory, written out by all threads
  for (int q = tid; q < o_zent; q += blockDim.x) tab[q] = s_tab[q];
  // Omega_g ranges for the zone pass (shared copy)
  if (tid < nch && s_rkeep[tid]) {
    s_rs[s_xs[2][tid]] = s_cpos[tid];
    s_rcum[s_xs[2][tid]] = s_xs[3][tid];
  }
  if (tid == 0) s_rcum[nr] = nom;
  __syncthreads();
  SegHdr H = s_h;
  // zone targets: kept nodes of Omega_g outside the segment; anchor = chain
  // whose bottom slot is the first segment node above the target.  The
  // counting pass keeps what it found for the first kOmegaLds nodes in
  // shared memory, so the placing pass re-reads nothing for them; ranges,
  // slot chains and chain bottoms come from shared memory throughout.
  auto classify = [&](int q, int& node, int& key) {  // key = chain * 8 | phase bits, -1: not a target
    int r = 0;
    while (r + 1 < nr && s_rcum[r + 1] <= q) ++r;
    const int i = s_rs[r] + (q - s_rcum[r]);
    node = i;
    key = -1;
    if (segment[i] == g || !St.kept[i]) return;
    const int pi = i;
    int best = -1;
    for (int j = 0; j < k; ++j)
      if (s_spos[j] < pi && pi < s_spos[j] + s_ssize[j] && (best < 0 || s_spos[j] > s_spos[best])) best = j;
    const int s = (best >= 0) ? s_jslot[best] : -1;
    if (s < 0) { atomicOr(&s_err, 1); return; }
    const int c = s_slotchain[s];
    if (s != s_cslot0[c + 1] - 1) { atomicOr(&s_err, 1); return; }  // must be the chain's bottom
    key = c * 8 + (int)T.phase[i];
  };
  for (int q = threadIdx.x; q < nom; q += blockDim.x) {
    int i, key;
    classify(q, i, key);
    if (q < kOmegaLds) {
      s_zi[q] = i;
      s_zk[q] = key;
    }
    if (key < 0) continue;
    for (int p = 0; p < 3; ++p)
      if (key >> p & 1) atomicAdd(&s_keycnt[(key >> 3) * 3 + p], 1);
  }
  __syncthreads();
  // zone entries grouped by key (chain, phase): offsets by an exclusive sum
  if (!s_err && tid < nch * 3) {
    int acc = 0;
    for (int q = 0; q < tid; ++q) acc += s_keycnt[q];
    const int cnt = s_keycnt[tid];
    s_keyoff[tid] = acc;
    int* cr = tab + H.o_chain + (tid / 3) * kChainInts;
    cr[C_ZOFF0 + tid % 3] = acc;
    cr[C_ZCNT0 + tid % 3] = cnt;
    if (tid == nch * 3 - 1) {
      s_h.nz = acc + cnt;
      s_h.total_ints = H.o_zent + 3 * (acc + cnt);
      if (s_h.total_ints > tab_cap) s_err = 1;
    }
  }
  // Pattern items of the table kernel: where one block's threads cannot take a
  // pattern each, an item of a chain of 6 bits or more enumerates its bottom
  // slots, up to 3 (the walk above them is done once for 8 patterns), fewer
  // with zone entries below the chain (at most 8 entry terms per item).
  if (tid < 64) {
    int items = 0, d = 0;
    if (tid < nch) {
      const int bits = __popc(s_pmask[tid]), n = s_cslot0[tid + 1] - s_cslot0[tid];
      const int z = s_keycnt[tid * 3] + s_keycnt[tid * 3 + 1] + s_keycnt[tid * 3 + 2];
      if (npat > 256 && bits >= 6) d = min(n, z <= 1 ? 3 : (z <= 2 ? 2 : (z <= 4 ? 1 : 0)));
      items = 1 << (bits - d);
    }
    int x = items;
    for (int o = 1; o < 32; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (tid >= o) x += y;
    }
    if (tid < nch) {
      int* cr = tab + H.o_chain + tid * kChainInts;
      cr[C_D] = d;
      cr[C_IBASE] = x - items;
      if (tid == nch - 1) s_h.nitem = x;
    }
  }
  __syncthreads();
  if (!s_err)
    for (int q = threadIdx.x; q < nom; q += blockDim.x) {
      int i, key;
      if (q < kOmegaLds) {
        i = s_zi[q];
        key = s_zk[q];
      } else {
        classify(q, i, key);
      }
      if (key < 0) continue;
      const int c = key >> 3;
      for (int p = 0; p < 3; ++p) {
        if (!(key >> p & 1)) continue;
        const int idx = s_keyoff[c * 3 + p] + atomicAdd(&s_keycur[c * 3 + p], 1);
        int* ze = tab + H.o_zent + 3 * idx;
        ze[0] = i;
        ze[1] = p;
        ze[2] = c;
        St.zent_of[i * 3 + p] = idx;
      }
    }
  __syncthreads();
  if (threadIdx.x == 0) {
    H = s_h;
    if (s_err) {
      H.valid = 0;
      atomicOr(status, kStatusBuild);
    }
    hdrs[g] = H;
  }
}

// The numeric part of applying a segment's decided mask (Algorithm 1 state
// update), one wave per snapshot: aggregated currents move to the new
// super-nodes, kept slots and zone targets take their candidate voltages (same
// arithmetic as the scoring).  Bs: the wave's chains' exit values.
__device__ __forceinline__ void apply_values(const SegHdr& H, const int* tab, int n, int l, bool on, uint32_t m,
                                             const double2* P, const TargetRec* srec, const TargetRec* zrec,
                                             double2* Vcur, double2* A, double2* Bs) {
  const int lane = threadIdx.x & 63;
  if (on && lane < 3) {  // phases are independent: one thread each
    const int p = lane;
    const cint* chains = as_cint(tab + H.o_chain);
    const cint* slots = as_cint(tab + H.o_slot);
    const double2* Pl = P + (size_t)l * H.npairs * 3;
    const TargetRec* srec_l = srec + (size_t)l * H.nslots * 3;
    for (int c = 0; c < H.nchains; ++c) {
      const cint* cr = chains + c * kChainInts;
      const int outer = cr[C_OUTER];
      double2 S = outer >= 0 ? Bs[outer * 3 + p] : make_double2(0.0, 0.0);
      int sidx = 0;
      // the current super-node's aggregated current, kept in a register
      // while reduced slots add theirs (the same additions, in order)
      size_t a = ((size_t)l * n + cr[C_HEAD]) * 3 + p;
      double2 acc = A[a];
      const int ns = cr[C_NSLOT], s0 = cr[C_SLOT0];
      for (int r = 0; r < ns; ++r) {
        const cint* sr = slots + (s0 + r) * kSlotInts;
        const int node = sr[SL_NODE];
        if ((m >> sr[SL_BIT]) & 1u) {
          const double2 pv = Pl[(sr[SL_PAIRBASE] + sidx) * 3 + p];
          S = make_double2(S.x + pv.x, S.y + pv.y);
          const size_t b = ((size_t)l * n + node) * 3 + p;
          const double2 ab = A[b];
          acc = make_double2(acc.x + ab.x, acc.y + ab.y);
          A[b] = make_double2(0.0, 0.0);
        } else {
          if (sr[SL_PHASE] >> p & 1) {
            const double2 w = srec_l[(s0 + r) * 3 + p].W;
            Vcur[((size_t)l * n + node) * 3 + p] = make_double2(w.x + S.x, w.y + S.y);
          }
          sidx = r + 1;
          A[a] = acc;
          a = ((size_t)l * n + node) * 3 + p;
          acc = A[a];
        }
      }
      A[a] = acc;
      Bs[c * 3 + p] = S;
    }
  }
  __syncthreads();
  if (!on) return;
  for (int q = lane; q < H.nz; q += 64) {
    const int* ze = tab + H.o_zent + q * 3;
    const int node = ze[0], p = ze[1], c = ze[2];
    const double2 w = zrec[(size_t)l * H.nz + q].W, b = Bs[c * 3 + p];
    Vcur[((size_t)l * n + node) * 3 + p] = make_double2(w.x + b.x, w.y + b.y);
  }
}

// One step between two chunks' scorings: blocks [0, nz) build the structural
// tables of the next chunk's segments, the others move the voltages and
// currents of the previous chunk's decided segments (4 snapshots per block).
// The two share nothing: the kept set and super-nodes are final when the
// previous decision is, the build reads and writes no voltage or current, and
// the chunks' tables alternate between two buffers.  As launches of their own
// the build (13.7 us) and the update (11.6) ran one after the other.
__global__ __launch_bounds__(256) void k_step(Topo T, State St, const int* __restrict__ segs, int nz, size_t lstride,
                                              int S, SegHdr* __restrict__ hdrs, int* __restrict__ tab, int tab_cap,
                                              int* __restrict__ status, unsigned long long* __restrict__ pat,
                                              unsigned long long* __restrict__ ecmax, int2* __restrict__ pat32,
                                              const int* __restrict__ psegs, const int* __restrict__ ptab,
                                              const DevDecision* __restrict__ decs, const double2* __restrict__ P,
                                              const TargetRec* __restrict__ srec, const TargetRec* __restrict__ zrec,
                                              double2* __restrict__ Vcur, double2* __restrict__ A) {
  if ((int)blockIdx.x < nz) {
    build_struct(T, St, segs, blockIdx.x, lstride, S, hdrs, tab, tab_cap, status, pat, ecmax, pat32);
    return;
  }
  __shared__ double2 s_B[4][kMaxK * 3];
  const int per = (S + 3) / 4, x = (int)blockIdx.x - nz, z = x / per;
  const int l = (x - z * per) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = *as_cint(psegs + z);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid) return;
  apply_values(H, lane_ptr_z(ptab, lstride, z), T.n, l, l < S, *as_cint((const int*)&decs[g].mask),
               lane_ptr_z(P, lstride, z), lane_ptr_z(srec, lstride, z), lane_ptr_z(zrec, lstride, z), Vcur, A,
               s_B[threadIdx.x >> 6]);
}

}  // namespace okr
