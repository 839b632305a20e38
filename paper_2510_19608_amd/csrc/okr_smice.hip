// SMICE as the search's second key (Algorithm 1's selection, MICE of Section
// II.C): among the feasible masks of the chosen level, the one whose clusters'
// largest member errors, summed over clusters and snapshots, are smallest.
//
// Only clusters that a mask can touch are summed (the others add the same
// constant to every mask): every kept slot's cluster (the slot and the
// reduced slots below it down to the next kept one), every zone target's
// cluster, and every chain head's cluster (the head's own members, whose
// error is fixed when the head lies outside Omega_g, plus the reduced slots
// at the top of each chain below it).  A cluster's error on a phase is
// max(|V_super| - lo, hi - |V_super|) over its member groups (lo, hi: the
// groups' extreme |V^|), so each group enters once per phase, as in the
// per-mask scoring.
//
//   (k_argmin)                lists mask 0 and the candidate masks; its second
//                             block, smice_prep: distinct heads, zone targets
//                             grouped by their anchor chain in Omega_g order;
//                             a block per snapshot, smice_hconst: fixed error of
//                             each outside head's cluster
//   k_smice_score  (grid)     SMICE of every listed mask
//   k_smice_argmin (1 block)  the smallest SMICE, tie rule, margin, flags
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_internal.h"

namespace okr {

// Voltage shift at the bottom of one chain for mask m (the currents its
// reduced slots move to their super-nodes), added to B.
__device__ __forceinline__ void sm_shift_chain(const cint* cr, const double2* Pl, uint32_t m, double2 (&B)[3]) {
  const int ns = cr[C_NSLOT], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
  const int phw0 = cr[C_PHW0], phw1 = cr[C_PHW1], phw2 = cr[C_PHW2];
  int sidx = 0;
  for (int r = 0; r < ns; ++r) {
    if ((m >> (bit0 + r)) & 1u) {
      const int w = r < 8 ? phw0 : (r < 16 ? phw1 : phw2);
      const int ph = (w >> (3 * (r & 7))) & 7;
      const double2* pr = Pl + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3;
      const double2 d[3] = {pr[0], pr[1], pr[2]};
#pragma unroll
      for (int p = 0; p < 3; ++p)
        if (ph >> p & 1) B[p] = cadd(B[p], d[p]);  // the slot's present phases only
    } else {
      sidx = r + 1;
    }
  }
}

// Error of one member group (extreme |V^| lo, hi) against a super-node
// magnitude.
__device__ __forceinline__ double sm_group(double mag, double lo, double hi) { return fmax(mag - lo, hi - mag); }

// SMICE over the clusters a mask can touch, summed over the snapshots, for
// every listed mask (mask 0 first, then the feasible masks of the chosen
// level).  A wave per mask, its lanes the snapshots, their sums folded in a
// fixed order; per-lane head maxima in LDS.  The walk of one (mask, snapshot) is
// a serial chain of table reads, bound by their latency: with one mask in a wave
// its branches are scalar and the tables' indices scalar loads, and the next
// record is read while one is worked on.  26 us a launch at 1000 nodes, 24
// snapshots (30 with two masks in a wave, each record read when it is needed;
// 320-420 with one lane per mask).
constexpr int kSmiceThreads = 128;
__global__ __launch_bounds__(kSmiceThreads) void k_smice_score(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ tab,
    const double2* __restrict__ P, const TargetRec* __restrict__ srec, const double2* __restrict__ headV,
    const TargetRec* __restrict__ zrec, const int* __restrict__ stab, const double* __restrict__ hK,
    const uint32_t* __restrict__ slist, const int* __restrict__ scount, double* __restrict__ smv) {
  __shared__ double s_acc[kMaxK][kSmiceThreads];
  const int g = segs[blockIdx.z];
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid) return;
  slist = lane_ptr(slist, lstride);
  scount = lane_ptr(scount, lstride);
  constexpr int kMasks = kSmiceThreads / 64;  // masks per block and round
  const int count = *as_cint(scount);
  tab = lane_ptr(tab, lstride);
  P = lane_ptr(P, lstride);
  srec = lane_ptr(srec, lstride);
  headV = lane_ptr(headV, lstride);
  zrec = lane_ptr(zrec, lstride);
  stab = lane_ptr(stab, lstride);
  hK = lane_ptr(hK, lstride);
  smv = lane_ptr(smv, lstride);
  const int tid = threadIdx.x, sl = tid & 63;
  const cint* sm = as_cint(stab);
  const int S = H.S, nh = sm[SM_NH];
  const cint* chains = as_cint(tab + H.o_chain);
  const cint* nest = as_cint(tab + H.o_nest);
  const cint* zr0 = sm + SM_ZREC;
  for (int i = blockIdx.x * kMasks + __builtin_amdgcn_readfirstlane(tid >> 6); i < count; i += gridDim.x * kMasks) {
  const uint32_t m = (uint32_t)as_cint((const int*)slist)[i];
  double total = 0.0;
  for (int l = sl; l < S; l += 64) {
    const double2* Pl = P + (size_t)l * H.npairs * 3;
    const TargetRec* Tl = srec + (size_t)l * H.nslots * 3;
    const double2* Hl = headV + (size_t)l * H.nchains * 3;
    const TargetRec* Zl = zrec + (size_t)l * H.nz;
    for (int x = 0; x < nh; ++x) s_acc[x][tid] = sm[SM_HIN + x] ? 0.0 : hK[x * S + l];
    double tot = 0.0;
    for (int c = 0; c < H.nchains; ++c) {
      const cint* cr = chains + c * kChainInts;
      double2 B[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) B[p] = make_double2(0.0, 0.0);
      const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
      for (int q = 0; q + 1 < nl; ++q) sm_shift_chain(chains + nest[no + q] * kChainInts, Pl, m, B);
      // the head's magnitude (moved by the outer chains when it lies below one)
      const int hph = cr[C_PHASE];
      const bool inner = cr[C_OUTER] >= 0;
      double smag[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double2 v = inner ? cadd(Hl[c * 3 + p], B[p]) : Hl[c * 3 + p];
        smag[p] = (hph >> p & 1) ? vmag(v) : 0.0;
      }
      const int hx = sm[SM_CHX + c];
      const int ns = cr[C_NSLOT], s0 = cr[C_SLOT0], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
      const int phw0 = cr[C_PHW0], phw1 = cr[C_PHW1], phw2 = cr[C_PHW2];
      int sidx = 0;
      bool open = false;
      double cl = 0.0, hd = 0.0;
      TargetRec nt[3];
      double2 np[3];
      // record of slot r and, if it is reduced, the rise of moving it to slot sidx
      auto fetch = [&](int r) {
        const TargetRec* tr = Tl + (s0 + r) * 3;
        const double2* pr = Pl + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3;
#pragma unroll
        for (int p = 0; p < 3; ++p) nt[p] = tr[p];
        if ((m >> (bit0 + r)) & 1u) {
#pragma unroll
          for (int p = 0; p < 3; ++p) np[p] = pr[p];
        }
      };
      if (ns > 0) fetch(0);
      for (int r = 0; r < ns; ++r) {
        const int w = r < 8 ? phw0 : (r < 16 ? phw1 : phw2);
        const int ph = (w >> (3 * (r & 7))) & 7;
        const TargetRec t[3] = {nt[0], nt[1], nt[2]};
        const double2 pr[3] = {np[0], np[1], np[2]};
        const bool red = (m >> (bit0 + r)) & 1u, top = sidx == 0;
        if (!red) sidx = r + 1;
        if (r + 1 < ns) fetch(r + 1);
        double er = 0.0;
        if (red) {  // its group joins the current super-node's cluster
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            if (!(ph >> p & 1)) continue;
            B[p] = cadd(B[p], pr[p]);
            er = fmax(er, sm_group(smag[p], t[p].lo, t[p].hi));
          }
          if (top) hd = fmax(hd, er);
          else cl = fmax(cl, er);
        } else {  // kept: closes the cluster above, opens its own
          if (open) tot += cl;
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            if (!(ph >> p & 1)) continue;
            smag[p] = vmag(cadd(t[p].W, B[p]));
            er = fmax(er, sm_group(smag[p], t[p].lo, t[p].hi));
          }
          cl = er;
          open = true;
        }
      }
      s_acc[hx][tid] = fmax(s_acc[hx][tid], hd);
      if (open) tot += cl;
      // zone targets anchored at this chain: their voltage moves with the
      // chain's bottom shift; a target that heads chains below keeps the
      // maximum for the head's cluster
      for (int z = sm[SM_ZOFF + c], ze = sm[SM_ZOFF + c + 1]; z < ze; ++z) {
        const cint* zr = zr0 + z * kZrecInts;
        TargetRec t[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) t[p] = Zl[max(zr[1 + p], 0)];
        double ez = 0.0;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          if (zr[1 + p] >= 0) ez = fmax(ez, sm_group(vmag(cadd(t[p].W, B[p])), t[p].lo, t[p].hi));
        if (zr[4] >= 0) s_acc[zr[4]][tid] = fmax(s_acc[zr[4]][tid], ez);
        else tot += ez;
      }
    }
    for (int x = 0; x < nh; ++x) tot += s_acc[x][tid];
    total += tot;
  }
  for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
  if (sl == 0) smv[i] = total;
  }
}

struct SmicePick {
  double runner;  // smallest measure above the tie threshold
  unsigned pick;  // lowest tied mask
  int amb;
};
__device__ __forceinline__ SmicePick shfl_xor_of(const SmicePick& v, int o) {
  return SmicePick{__shfl_xor(v.runner, o, 64), (unsigned)__shfl_xor((int)v.pick, o, 64), __shfl_xor(v.amb, o, 64)};
}

// The decision under SMICE: the smallest SMICE among the candidates, the
// lowest mask within tol of it, the margin to the next one outside, and the
// ambiguity flags (a candidate within tol/100 of the tie-window edge, or a
// mask at the chosen level or above near the e_bar / band boundary).
// Decision by the measure: the lowest mask within tol of the smallest one.  One
// block per segment, a chain of dependent steps: the minimum, then pick,
// runner-up and flag in one reduction, the tiles' records read with the measures
// (8.6 us per chunk at 1000 nodes, 9.8 with three reductions and the records
// after them).
__global__ __launch_bounds__(1024) void k_smice_argmin(const SegHdr* __restrict__ hdrs, const int* __restrict__ segs,
                                                       size_t lstride, const MaskScore* __restrict__ fin,
                                                       const TileRec* __restrict__ tiles,
                                                       const uint32_t* __restrict__ slist,
                                                       const int* __restrict__ scount,
                                                       const double* __restrict__ smv, double tol,
                                                       DevDecision* __restrict__ decs, const int* __restrict__ tab,
                                                       Topo T, State St) {
  __shared__ double shd[16];
  __shared__ SmicePick shp[16];
  const int g = segs[blockIdx.z];
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid) return;
  DevDecision d = decs[g];
  tab = lane_ptr(tab, lstride);
  __shared__ StateUpdate su;
  int ui, us, uj;
  su.load(H, tab, T, St, ui, us, uj);
  __syncthreads();
  if (!d.found) {
    su.store(H, tab, St, d.mask, ui, us, uj);
    return;
  }
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  slist = lane_ptr(slist, lstride);
  scount = lane_ptr(scount, lstride);
  smv = lane_ptr(smv, lstride);
  const int ntiles = (int)((1u << H.k) >> tile_bits(H.k));
  // (the list's first entry is mask 0, a candidate at level 0 only)
  const int count = *scount, first = d.popcount == 0 ? 0 : 1;
  int amb = 0;
  for (int t = threadIdx.x; t < ntiles; t += blockDim.x)
    if (tiles[t].near >= d.popcount) amb = 1;
  double smin = INFINITY;
  for (int i = first + threadIdx.x; i < count; i += blockDim.x) smin = fmin(smin, smv[i]);
  smin = block_reduce(smin, [](double a, double b) { return fmin(a, b); }, shd);
  const double thr = smin + tol, atol = tol / 100.0;
  unsigned pick = 0xffffffffu;
  int at = -1;  // list position of this thread's pick
  double runner = INFINITY;
  for (int i = first + threadIdx.x; i < count; i += blockDim.x) {
    const double v = smv[i];
    if (fabs(v - thr) <= atol) amb = 1;
    if (v > thr) {
      runner = fmin(runner, v);
    } else if (slist[i] < pick) {
      pick = slist[i];
      at = i;
    }
  }
  const unsigned mine = pick;
  {
    const SmicePick v = block_reduce(SmicePick{runner, pick, amb},
                                     [](const SmicePick& a, const SmicePick& b) {
                                       return SmicePick{fmin(a.runner, b.runner), (unsigned)min(a.pick, b.pick),
                                                        a.amb | b.amb};
                                     },
                                     shp);
    runner = v.runner;
    pick = v.pick;
    amb = v.amb;
  }
  if (at >= 0 && mine == pick) {  // one thread: the list holds a mask once
    d.mask = pick;
    d.e_loc = fin[pick].e;
    d.ambiguous = amb;
    d.key_gap = runner - smin;
    d.smice_rise = smv[at] - smv[0];
    decs[g] = d;
  }
  su.store(H, tab, St, pick != 0xffffffffu ? pick : d.mask, ui, us, uj);
}

}  // namespace okr
