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

#include "okr_device.h"
#include "okr_internal.h"
#include "okr_kron.h"

namespace okr {

constexpr uint8_t kNoKey = 255;
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

// Structural tables of segment segs[z] (one block).  Wave 0 finds the chains on
// its own: a lane per segment node, then per chain, comparisons over readlane
// and ballots, no barrier; then all threads write records and classify the zone,
// the zone ranges are summed, and the tables go out (four barriers in all, 15
// when every step was one of the block's: 12 us of its 14 in k_step, bound by
// the latency of serial LDS loops over 16 slots).
__device__ __forceinline__ void build_struct(Topo T, State St, const int* __restrict__ segs, int z, size_t lstride,
                                             int S, SegHdr* __restrict__ hdrs, int* __restrict__ tab, int tab_cap,
                                             int* __restrict__ status, unsigned long long* __restrict__ pat,
                                             unsigned long long* __restrict__ ecmax, int2* __restrict__ pat32) {
  __shared__ int s_slotnode[kMaxK], s_slotbit[kMaxK], s_slotchain[kMaxK], s_cslot0[kMaxK + 1], s_jslot[kMaxK];
  __shared__ int s_spos[kMaxK], s_ssize[kMaxK], s_sph[kMaxK];           // segment node j
  __shared__ int s_cpos[kMaxK], s_csize[kMaxK], s_chph[kMaxK], s_head[kMaxK];  // chain c: top pos/size, head phase
  __shared__ int s_rs[kMaxK], s_rcum[kMaxK + 1];                       // Omega_g ranges: start, cumulative size
  __shared__ int s_outer[kMaxK], s_rkeep[kMaxK], s_depth[kMaxK], s_pmask[kMaxK];
  // exclusive prefix sums over the chains (entry nch: the totals) of: nesting
  // depth, pairs, new Omega_g range, its nodes, chain patterns
  __shared__ int s_xs[5][kMaxK + 1];
  __shared__ int s_keycnt[kMaxK * 3], s_keyoff[kMaxK * 3], s_keycur[kMaxK * 3];
  __shared__ SegHdr s_h;
  __shared__ int s_err, s_nch;
  __shared__ int s_zi[kOmegaLds];      // zone pass: node of Omega index q
  __shared__ uint8_t s_zk[kOmegaLds];  // its key (chain * 8 | phases: below 192), kNoKey: no target
  __shared__ int s_tab[kTabLds];                     // structural tables before they are written out
  const int g = segs[z];
  tab = lane_ptr_z(tab, lstride, z);
  pat = lane_ptr_z(pat, lstride, z);
  const int tid = threadIdx.x;
  const int o0 = T.seg_off[g];
  const int k = T.seg_off[g + 1] - o0;
  if (tid >= 64) {
    if (tid < 64 + kMaxK * 3) s_keycnt[tid - 64] = s_keycur[tid - 64] = 0;
  } else {
    // an earlier segment failed: leave every later one invalid (its scratch
    // maps may be stale)
    bool err = (*status & kStatusBuild) || k < 1 || k > kMaxK;
    const int lane = tid;
    const bool on = !err && lane < k;
    // chain top of every segment node: the highest node above it reachable
    // through segment or reduced nodes (runs of reduced nodes are crossed in
    // one step: their nearest kept ancestor is known)
    int e = 0, top = 0, hd = -1, esize = 0, eph = 0, tsize = 0, hph = 0;
    if (on) {
      e = T.seg_nodes[o0 + lane];
      esize = T.size[e];
      eph = T.phase[e];
      top = T.seg_top[e];  // (runs of this segment's nodes climbed at plan time)
      for (int guard = 0;;) {
        const int p = T.parent[top];
        if (p < 0 || ++guard > T.n) break;
        const int sg = T.segment[p], kp = St.kept[p], h = St.sup[p];
        if (sg == g) { top = T.seg_top[p]; continue; }
        if (kp) break;
        const int x = (h >= 0 && h != p) ? child_toward(T, h, p) : -1;
        if (x < 0) { err = true; break; }
        top = x;
      }
      tsize = T.size[top];
      hd = T.parent[top];
      hph = hd >= 0 ? T.phase[hd] : 0;
    }
    err = __ballot(err) != 0ull;
    // chains: one per distinct chain top, ordered by the tops' preorder
    // positions (distinct nodes, so the order is strict); slots chain by chain,
    // top to bottom (segment nodes are in preorder)
    uint32_t same = 0, lower = 0;
    for (int q = 0; q < k && !err; ++q) {
      const int tq = __builtin_amdgcn_readlane(top, q);
      same |= (uint32_t)(tq == top) << q;
      lower |= (uint32_t)(tq < top) << q;
    }
    const uint32_t below = (1u << (lane & 31)) - 1u;
    const bool first = on && !err && (same & below) == 0u;  // the chain's first node
    const uint32_t opens = (uint32_t)__ballot(first);
    const int nch = __popc(opens), mychain = __popc(lower & opens);
    const int before = __popc(lower), slot = before + __popc(same & below);
    if (on && !err) {
      // every chain is a path: each slot lies below the previous one (the first
      // below the chain top); its nodes have at most one child, so its slots
      // are consecutive segment nodes in preorder: consecutive mask bits
      s_jslot[lane] = slot;
      s_slotnode[slot] = e;
      s_slotbit[slot] = lane;
      s_slotchain[slot] = mychain;
      s_spos[lane] = e;
      s_ssize[lane] = esize;
      s_sph[lane] = eph;
      if (first) {
        s_cpos[mychain] = top;
        s_csize[mychain] = tsize;
        s_chph[mychain] = hph;
        s_head[mychain] = hd;
        s_cslot0[mychain] = before;
      }
      if (lane == 0) s_cslot0[nch] = k;
    }
    {
      const int prev = (same & below) ? 31 - __clz(same & below) : lane;
      const int pu = __shfl(e, prev, 64), su = __shfl(esize, prev, 64);
      bool bad = false;
      if (on && !err) {
        if (first) bad = !(top <= e && e < top + tsize);
        else bad = !(pu < e && e < pu + su) || prev != lane - 1;
      }
      err = err || __ballot(bad) != 0ull;
    }
    wave_fence();
    // a lane per chain: the outer chain (whose bottom slot is the deepest
    // segment node above the head), and whether its top's subtree starts a new
    // Omega_g range (laminar intervals in preorder: a top inside an earlier
    // top's subtree adds nothing)
    const bool ch = !err && lane < nch;
    const int cpos = ch ? s_cpos[lane] : 0, csize = ch ? s_csize[lane] : 0, head = ch ? s_head[lane] : -1;
    const int s0 = ch ? s_cslot0[lane] : 0, s1 = ch ? s_cslot0[lane + 1] : 0, bit0 = ch ? s_slotbit[s0] : 0;
    int best = -1, rkeep = 1;
    for (int q = 0; q < k && !err; ++q) {  // (positions ascend: the last one found is the deepest)
      const int pq = __builtin_amdgcn_readlane(e, q), sq = __builtin_amdgcn_readlane(esize, q);
      if (head >= 0 && pq <= head && head < pq + sq) best = q;
    }
    for (int q = 0; q < nch && !err; ++q) {
      const int pq = __builtin_amdgcn_readlane(cpos, q), sq = __builtin_amdgcn_readlane(csize, q);
      if (q < lane && pq <= cpos && cpos < pq + sq) rkeep = 0;
    }
    int outer = -1;
    {
      const int bs = __shfl(slot, max(best, 0), 64), bc = __shfl(mychain, max(best, 0), 64);
      const int bend = __shfl(s1, bc, 64);
      if (ch && best >= 0) outer = bc;
      const bool bad = ch && best >= 0 && (bs != bend - 1 || bc >= lane);
      err = err || __ballot(bad) != 0ull;
    }
    // nesting depth (outer chains have smaller indices) and the mask bits of
    // the chains on the nesting path, the chain itself included
    const int cbits = ch ? ((1 << (s1 - s0)) - 1) << bit0 : 0;
    int depth = 0, pm = 0;
    for (int x = ch ? lane : -1; !err && __ballot(x >= 0);) {
      const int xb = __shfl(cbits, max(x, 0), 64), xo = __shfl(outer, max(x, 0), 64);
      if (x >= 0) {
        ++depth;
        pm |= xb;
        x = xo;
      }
    }
    // the chains' table offsets
    const int nc = s1 - s0;
    const int v0 = ch ? depth : 0, v1 = nc * (nc + 1) / 2, v2 = ch ? rkeep : 0, v3 = ch && rkeep ? csize : 0,
              v4 = ch ? 1 << __popc(pm) : 0;
    const int x0 = scan32(v0) - v0, x1 = scan32(v1) - v1, x2 = scan32(v2) - v2, x3 = scan32(v3) - v3,
              x4 = scan32(v4) - v4;
    if (lane <= nch && lane <= kMaxK) {
      s_xs[0][lane] = x0;
      s_xs[1][lane] = x1;
      s_xs[2][lane] = x2;
      s_xs[3][lane] = x3;
      s_xs[4][lane] = x4;
    }
    if (ch) {
      s_outer[lane] = outer;
      s_rkeep[lane] = rkeep;
      s_depth[lane] = depth;
      s_pmask[lane] = pm;
      if (rkeep) {
        s_rs[x2] = cpos;
        s_rcum[x2] = x3;
      }
    }
    // table layout
    const int nest_tot = __builtin_amdgcn_readlane(x0, nch), npairs = __builtin_amdgcn_readlane(x1, nch);
    const int nr = __builtin_amdgcn_readlane(x2, nch), nom = __builtin_amdgcn_readlane(x3, nch);
    const int npat = __builtin_amdgcn_readlane(x4, nch);
    if (lane == 0) {
      SegHdr H;
      for (int q = 0; q < (int)(sizeof(SegHdr) / sizeof(int)); ++q) ((int*)&H)[q] = 0;
      H.g = g;
      H.k = k;
      H.S = S;
      H.o_chain = 0;
      H.o_nest = nch * kChainInts;
      H.o_slot = H.o_nest + nest_tot;
      H.o_pair = H.o_slot + k * kSlotInts;
      H.o_range = H.o_pair + npairs * kPairInts;
      H.o_zent = H.o_range + 3 * nr;
      H.nrange = nr;
      H.nomega = nom;
      H.nchains = nch;
      H.nslots = k;
      H.npairs = npairs;
      H.npat = npat;
      // the structural part must fit the segment's table (and the shared image,
      // which holds the largest possible one)
      if (H.o_zent > tab_cap || H.o_zent > kTabLds) err = true;
      // the chain patterns number at most 2^(k+1) (a nesting forest whose
      // chains hold k bits in all): the pattern table's capacity
      if (!err && npat > (2 << k)) err = true;
      H.valid = err ? 0 : 1;
      s_h = H;
      s_nch = nch;
      s_rcum[min(nr, kMaxK)] = nom;
      s_err = err ? 1 : 0;
    }
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
  const int nch = s_nch, nr = s_h.nrange, nom = s_h.nomega, npat = s_h.npat;
  const int o_nest = s_h.o_nest, o_slot = s_h.o_slot, o_pair = s_h.o_pair, o_range = s_h.o_range, o_zent = s_h.o_zent;
  // zone targets: kept nodes of Omega_g outside the segment; anchor = chain
  // whose bottom slot is the first segment node above the target.  The
  // counting pass keeps what it found for the first kOmegaLds nodes in
  // shared memory, so the placing pass re-reads nothing for them; ranges,
  // slot chains and chain bottoms come from shared memory throughout.
  auto omega = [&](int q) {
    int r = 0;
    while (r + 1 < nr && s_rcum[r + 1] <= q) ++r;
    return s_rs[r] + (q - s_rcum[r]);
  };
  auto classify = [&](int i, int sg, int kp, int ph) {  // key = chain * 8 | phase bits, -1: not a target
    if (sg == g || !kp) return -1;
    int best = -1;
#pragma unroll 4
    for (int j = 0; j < k; ++j)  // (positions ascend: the last one found is the deepest)
      if ((unsigned)(i - s_spos[j] - 1) < (unsigned)(s_ssize[j] - 1)) best = j;
    if (best < 0) { atomicOr(&s_err, 1); return -1; }
    const int s = s_jslot[best], c = s_slotchain[s];
    if (s != s_cslot0[c + 1] - 1) { atomicOr(&s_err, 1); return -1; }  // must be the chain's bottom
    return c * 8 + ph;
  };
  // this thread's first Omega_g node: its loads run under the records
  int zi = 0, zseg = 0, zkept = 0, zph = 0;
  if (tid < nom) {
    zi = omega(tid);
    zseg = T.segment[zi];
    zkept = St.kept[zi];
    zph = T.phase[zi];
  }
  // the pattern accumulators the scoring folds into (error, smallest and
  // largest kept squared magnitude of each pattern; the largest constant
  // error): cleared here, where their number is first known, which saves the
  // scoring a launch of its own (4.3 us per chunk)
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
  // records: a thread per chain (wave 1), per slot (wave 2), per pair (all)
  if (tid >= 64 && tid < 64 + nch) {
    const int c = tid - 64, s0 = s_cslot0[c], n = s_cslot0[c + 1] - s0, bit0 = s_slotbit[s0];
    const int nest_off = s_xs[0][c], ridx = s_xs[2][c];
    const int d = s_depth[c];
    int q = d - 1;
    for (int x = c; x >= 0; x = s_outer[x]) s_tab[o_nest + nest_off + q--] = x;
    if (s_rkeep[c]) {
      s_tab[o_range + 3 * ridx] = s_cpos[c];
      s_tab[o_range + 3 * ridx + 1] = s_cpos[c] + s_csize[c];
      s_tab[o_range + 3 * ridx + 2] = s_xs[3][c];
    }
    int phw[3] = {0, 0, 0};
#pragma unroll
    for (int w = 0; w < 3; ++w)
      for (int r = 8 * w; r < min(n, 8 * w + 8); ++r) phw[w] |= s_sph[bit0 + r] << (3 * (r & 7));
    int* cr = s_tab + c * kChainInts;
    cr[C_HEAD] = s_head[c];
    cr[C_NSLOT] = n;
    cr[C_SLOT0] = s0;
    cr[C_NEST_OFF] = nest_off;
    cr[C_NEST_LEN] = d;
    cr[C_OUTER] = s_outer[c];
    cr[C_PHASE] = s_chph[c];
    cr[C_BIT0] = bit0;
    cr[C_PAIR0] = s_xs[1][c];
    cr[C_PHW0] = phw[0];
    cr[C_PHW1] = phw[1];
    cr[C_PHW2] = phw[2];
    cr[C_PMASK] = s_pmask[c];
    cr[C_PBASE] = s_xs[4][c];
  }
  if (tid >= 128 && tid < 128 + k) {
    const int s = tid - 128, c = s_slotchain[s], r = s - s_cslot0[c];
    int* sr = s_tab + o_slot + s * kSlotInts;
    sr[SL_NODE] = s_slotnode[s];
    sr[SL_BIT] = s_slotbit[s];
    sr[SL_PHASE] = s_sph[s_slotbit[s]];
    sr[SL_PAIRBASE] = s_xs[1][c] + r * (r + 1) / 2;
    sr[SL_CHAIN] = c;
    St.slot_of[s_slotnode[s]] = s;
  }
  // slot s = r-th slot of chain c: pairs (super, reduced) with the super
  // node the head or one of the r slots above it
  for (int x = tid; x < k * 32; x += blockDim.x) {
    const int s = x >> 5, sx = x & 31, c = s_slotchain[s], s0 = s_cslot0[c], r = s - s0;
    if (sx > r) continue;
    int* pr = s_tab + o_pair + (s_xs[1][c] + r * (r + 1) / 2 + sx) * kPairInts;
    pr[PR_RNODE] = s_slotnode[s];
    pr[PR_SUPER] = (sx == 0) ? s_head[c] : s_slotnode[s0 + sx - 1];
    pr[PR_RSLOT] = s;
  }
  for (int q = tid; q < nom; q += blockDim.x) {
    if (q != tid) {
      zi = omega(q);
      zseg = T.segment[zi];
      zkept = St.kept[zi];
      zph = T.phase[zi];
    }
    const int key = classify(zi, zseg, zkept, zph);
    if (q < kOmegaLds) {
      s_zi[q] = zi;
      s_zk[q] = key < 0 ? kNoKey : (uint8_t)key;
    }
    if (key < 0) continue;
    for (int p = 0; p < 3; ++p)
      if (key >> p & 1) atomicAdd(&s_keycnt[(key >> 3) * 3 + p], 1);
  }
  __syncthreads();
  // zone entries grouped by key (chain, phase): offsets by an exclusive sum,
  // two keys per lane of wave 1
  if (tid >= 64 && tid < 128) {
    const int k0 = 2 * (tid - 64), nk = nch * 3;
    const int a = k0 < nk ? s_keycnt[k0] : 0, b = k0 + 1 < nk ? s_keycnt[k0 + 1] : 0;
    const int end = scan64(a + b);
    for (int h = 0; h < 2; ++h) {
      const int q = k0 + h;
      if (q >= nk) break;
      const int off = end - a - b + (h ? a : 0);
      s_keyoff[q] = off;
      int* cr = s_tab + (q / 3) * kChainInts;
      cr[C_ZOFF0 + q % 3] = off;
      cr[C_ZCNT0 + q % 3] = h ? b : a;
    }
    if (tid == 127) {
      s_h.nz = end;
      s_h.total_ints = o_zent + 3 * end;
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
      const int zc = s_keycnt[tid * 3] + s_keycnt[tid * 3 + 1] + s_keycnt[tid * 3 + 2];
      if (npat > 256 && bits >= 6) d = min(n, zc <= 1 ? 3 : (zc <= 2 ? 2 : (zc <= 4 ? 1 : 0)));
      items = 1 << (bits - d);
    }
    const int x = scan32(items);
    if (tid < nch) {
      int* cr = s_tab + tid * kChainInts;
      cr[C_D] = d;
      cr[C_IBASE] = x - items;
      if (tid == nch - 1) s_h.nitem = x;
    }
  }
  __syncthreads();
  // the structural tables, built in shared memory, written out by all threads
  for (int q = tid; q < o_zent; q += blockDim.x) tab[q] = s_tab[q];
  if (!s_err)
    for (int q = threadIdx.x; q < nom; q += blockDim.x) {
      int i, key;
      if (q < kOmegaLds) {
        i = s_zi[q];
        key = s_zk[q] == kNoKey ? -1 : s_zk[q];
      } else {
        i = omega(q);
        key = classify(i, T.segment[i], St.kept[i], T.phase[i]);
      }
      if (key < 0) continue;
      const int c = key >> 3;
      for (int p = 0; p < 3; ++p) {
        if (!(key >> p & 1)) continue;
        const int idx = s_keyoff[c * 3 + p] + atomicAdd(&s_keycur[c * 3 + p], 1);
        int* ze = tab + o_zent + 3 * idx;
        ze[0] = i;
        ze[1] = p;
        ze[2] = c;
        St.zent_of[i * 3 + p] = idx;
      }
    }
  if (tid == 0) {
    SegHdr H = s_h;
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
// arithmetic as the scoring).  Everything the walk reads is loaded at once, a
// lane per (slot, phase); the walk itself, a lane per phase, runs in LDS.
struct ApplyLds {
  double2 B[kMaxK * 3];   // chains' exit values
  double2 H[kMaxK * 3];   // heads' aggregated currents (at the first chain of a head)
  double2 A[kMaxK * 3];   // slots' aggregated currents
  double2 X[kMaxK * 3];   // reduced slots: the added change; kept ones: W, then the new voltage
};

__device__ __forceinline__ void apply_values(const SegHdr& H, const int* tab, int n, int l, bool on, uint32_t m,
                                             const double2* P, const TargetRec* srec, const TargetRec* zrec,
                                             double2* Vcur, double2* A, ApplyLds& L) {
  const int lane = threadIdx.x & 63;
  if (!on) return;
  const int nch = H.nchains, ns = H.nslots;
  // lane = chain
  int head = -1, outer = -1, cs0 = 0, cn = 0, hc = lane;
  if (lane < nch) {
    const int* cr = tab + H.o_chain + lane * kChainInts;
    head = cr[C_HEAD];
    outer = cr[C_OUTER];
    cs0 = cr[C_SLOT0];
    cn = cr[C_NSLOT];
  }
  // lane = slot: whether it is reduced
  int bit = 31, chain = 0;
  if (lane < ns) {
    const int* sr = tab + H.o_slot + lane * kSlotInts;
    bit = sr[SL_BIT];
    chain = sr[SL_CHAIN];
  }
  const uint32_t red = (uint32_t)__ballot(lane < ns && ((m >> bit) & 1u));
  const double2* Pl = P + (size_t)l * H.npairs * 3;
  const TargetRec* srec_l = srec + (size_t)l * ns * 3;
  double2* Al = A + (size_t)l * n * 3;
  double2* Vl = Vcur + (size_t)l * n * 3;
  int node[2], ph[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int x = lane + 64 * u, s = x / 3, p = x - 3 * s;
    node[u] = -1;
    const int c = __shfl(chain, s, 64), s0 = __shfl(cs0, c, 64);
    if (s >= ns) continue;
    const int* sr = tab + H.o_slot + s * kSlotInts;
    node[u] = sr[SL_NODE];
    ph[u] = sr[SL_PHASE] >> p & 1;
    L.A[x] = Al[(size_t)node[u] * 3 + p];
    if (red >> s & 1u) {
      // the super-node: the last kept slot above it in the chain, or the head
      const uint32_t kept = ~(red >> s0) & ((1u << (s - s0)) - 1u);
      const int sidx = kept ? 32 - __clz(kept) : 0;
      L.X[x] = Pl[(sr[SL_PAIRBASE] + sidx) * 3 + p];
    } else {
      L.X[x] = srec_l[x].W;
    }
  }
  for (int q = 0; q < nch; ++q)  // the first chain with the same head
    if (q < hc && __builtin_amdgcn_readlane(head, q) == head) hc = q;
  int hnode[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int x = lane + 64 * u, c = x / 3, p = x - 3 * c;
    const int hn = __shfl(head, c, 64), first = __shfl(hc, c, 64);
    hnode[u] = c < nch && first == c ? hn : -1;
    if (hnode[u] >= 0) L.H[x] = Al[(size_t)hn * 3 + p];
  }
  wave_fence();
  {
    const int p = lane < 3 ? lane : 0;  // phases are independent: one lane each (the others write nothing)
    for (int c = 0; c < nch; ++c) {
      const int o = __builtin_amdgcn_readlane(outer, c), s0 = __builtin_amdgcn_readlane(cs0, c);
      const int s1 = s0 + __builtin_amdgcn_readlane(cn, c), h = __builtin_amdgcn_readlane(hc, c);
      double2 S = o >= 0 ? L.B[o * 3 + p] : make_double2(0.0, 0.0);
      double2* a = &L.H[h * 3 + p];
      // the current super-node's aggregated current, kept in a register while
      // reduced slots add theirs (the same additions, in order)
      double2 acc = *a;
      for (int s = s0; s < s1; ++s) {
        const double2 x = L.X[s * 3 + p], b = L.A[s * 3 + p];
        if (red >> s & 1u) {
          S = make_double2(S.x + x.x, S.y + x.y);
          acc = make_double2(acc.x + b.x, acc.y + b.y);
          if (lane < 3) L.A[s * 3 + p] = make_double2(0.0, 0.0);
        } else {
          if (lane < 3) {
            L.X[s * 3 + p] = make_double2(x.x + S.x, x.y + S.y);
            *a = acc;
          }
          a = &L.A[s * 3 + p];
          acc = b;
        }
      }
      if (lane < 3) {
        *a = acc;
        L.B[c * 3 + p] = S;
      }
      wave_fence();
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int x = lane + 64 * u, s = x / 3, p = x - 3 * s;
    if (node[u] >= 0) {
      Al[(size_t)node[u] * 3 + p] = L.A[x];
      if (!(red >> s & 1u) && ph[u]) Vl[(size_t)node[u] * 3 + p] = L.X[x];
    }
    if (hnode[u] >= 0) Al[(size_t)hnode[u] * 3 + p] = L.H[x];
  }
  for (int q = lane; q < H.nz; q += 64) {
    const int* ze = tab + H.o_zent + q * 3;
    const int zn = ze[0], p = ze[1], c = ze[2];
    const double2 w = zrec[(size_t)l * H.nz + q].W, b = L.B[c * 3 + p];
    Vl[(size_t)zn * 3 + p] = make_double2(w.x + b.x, w.y + b.y);
  }
}

// One step between two chunks' scorings: blocks [0, nz) build the structural
// tables of the next chunk's segments, the others move the voltages and
// currents of the previous chunk's decided segments (4 snapshots per block).
// After the last chunk, the first ny blocks form the admittances of the kept
// branches instead, which need only the structure (a wave of nodes each: long
// FP64 chains).
// The two share nothing: the kept set and super-nodes are final when the
// previous decision is, the build reads and writes no voltage or current, and
// the chunks' tables alternate between two buffers.  As launches of their own
// the build (13.7 us) and the update (11.6) ran one after the other; together
// 14.0 us at 1000 nodes and 16.1 at 6000, 9.7 and 10.9 with the chains found by
// one wave and the update's loads issued together.
__global__ __launch_bounds__(256) void k_step(Topo T, State St, const int* __restrict__ segs, int nz, size_t lstride,
                                              int S, SegHdr* __restrict__ hdrs, int* __restrict__ tab, int tab_cap,
                                              int* __restrict__ status, unsigned long long* __restrict__ pat,
                                              unsigned long long* __restrict__ ecmax, int2* __restrict__ pat32,
                                              const int* __restrict__ psegs, const int* __restrict__ ptab,
                                              const DevDecision* __restrict__ decs, const double2* __restrict__ P,
                                              const TargetRec* __restrict__ srec, const TargetRec* __restrict__ zrec,
                                              double2* __restrict__ Vcur, double2* __restrict__ A, int ny,
                                              const double2* __restrict__ z, double2* __restrict__ yeq,
                                              double2* __restrict__ Yk_off, int* __restrict__ kp_out) {
  if ((int)blockIdx.x < ny) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && x < T.n) kron_yeq(x, T, St, z, yeq, Yk_off, kp_out, status);
    return;
  }
  if ((int)blockIdx.x < nz) {
    build_struct(T, St, segs, blockIdx.x, lstride, S, hdrs, tab, tab_cap, status, pat, ecmax, pat32);
    return;
  }
  __shared__ ApplyLds s_apply[4];
  const int per = (S + 3) / 4, x = (int)blockIdx.x - nz - ny, pz = x / per;
  const int l = (x - pz * per) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = *as_cint(psegs + pz);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid) return;
  apply_values(H, lane_ptr_z(ptab, lstride, pz), T.n, l, l < S, *as_cint((const int*)&decs[g].mask),
               lane_ptr_z(P, lstride, pz), lane_ptr_z(srec, lstride, pz), lane_ptr_z(zrec, lstride, pz), Vcur, A,
               s_apply[threadIdx.x >> 6]);
}

}  // namespace okr
