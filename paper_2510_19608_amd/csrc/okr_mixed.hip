// Mixed-precision search of one segment: FP32 screening of every mask in
// difference form, then FP64 rescoring of a shortlist that provably contains
// every mask the FP64 decision depends on, so that the decision equals the
// FP64 path's whenever |e32 - e64| <= delta and |slack32 - slack64| <= delta.
//
//   k_seg_terms      FP64 tables and FP64 chain patterns    [okr_score.hip]
//   k_pat32          FP32 chain patterns
//   k_combine32      every mask, FP32; tile records of sure / possible /
//                    uncertain feasibility (band delta + amb around e_bar and
//                    the voltage band)
//   k_mixed_decide   list A: uncertain masks at or above the best sure level,
//                    their FP64 scores from the FP64 patterns; best level P*;
//                    list B: possibly feasible masks at P* whose FP32 error is
//                    within tie + 2 delta + amb of the smallest FP64-confirmed
//                    one, their FP64 scores; FP64 arg-min over list B,
//                    ambiguity from A and B
//
// A listed mask's FP64 score is one pattern entry per chain, so the selections,
// the scores of both lists and the decision are one launch (ten before: three
// selections and the lists' chain walks, 100 us per chunk on the 6000-node
// feeder).  One block per segment, bound by latency: 17 us per chunk there, 21
// with the tile records read again for each of four passes and every maximum
// reduced by itself.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_internal.h"

namespace okr {

struct Levels {
  int lo, hi;
};
struct Verdict {
  double dev, runner;
  unsigned pick;
  int amb;
};

__device__ __forceinline__ Levels shfl_xor_of(const Levels& v, int o) {
  return Levels{__shfl_xor(v.lo, o, 64), __shfl_xor(v.hi, o, 64)};
}
__device__ __forceinline__ Verdict shfl_xor_of(const Verdict& v, int o) {
  return Verdict{__shfl_xor(v.dev, o, 64), __shfl_xor(v.runner, o, 64), (unsigned)__shfl_xor((int)v.pick, o, 64),
                 __shfl_xor(v.amb, o, 64)};
}

__device__ __forceinline__ bool skip_segment(const SegHdr& H, const int* status) {
  return !H.valid || (*status & (16 | 32));
}

__global__ __launch_bounds__(1024) void k_mixed_decide(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ tab,
    const unsigned long long* __restrict__ pat, const unsigned long long* __restrict__ ecmax,
    const MaskScore32* __restrict__ fin, const TileRec32* __restrict__ tiles, SelParams sp,
    const int* __restrict__ status, MixedState* __restrict__ ms, uint32_t* listA, MaskScore* scoreA, uint32_t* listB,
    MaskScore* scoreB, DevDecision* __restrict__ decs, int* __restrict__ redo) {
  __shared__ double shd[16];
  __shared__ int shi[16];
  __shared__ Levels shv[16];
  __shared__ Verdict shr[16];
  __shared__ int s_pm[kMaxK], s_pb[kMaxK];
  __shared__ int cand[1024], ncand, nlist;
  const int g = segs[blockIdx.z];
  const SegHdr H = load_hdr_g(hdrs, g);
  tab = lane_ptr(tab, lstride);
  pat = lane_ptr(pat, lstride);
  ecmax = lane_ptr(ecmax, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  listA = lane_ptr(listA, lstride);
  scoreA = lane_ptr(scoreA, lstride);
  listB = lane_ptr(listB, lstride);
  scoreB = lane_ptr(scoreB, lstride);
  const int tid = threadIdx.x, bd = blockDim.x;
  auto nothing = [&](int ambiguous) {
    DevDecision d;
    d.mask = 0; d.popcount = 0; d.e_loc = 0.0; d.e_min = 0.0; d.ambiguous = ambiguous; d.found = 0;
    d.key_gap = INFINITY;
    d.smice_rise = 0.0;
    decs[g] = d;
    redo[g] = 0;
  };
  if (skip_segment(H, status)) {
    if (tid == 0) {
      ms[g].lo_level = ms[g].hi_level = ms[g].best = -1;
      ms[g].nA = ms[g].nB = 0;
      ms[g].max_dev = 0.0;
      nothing(0);
    }
    return;
  }
  const int nch = H.nchains;
  if (tid < nch) {
    s_pm[tid] = tab[H.o_chain + tid * kChainInts + C_PMASK];
    s_pb[tid] = tab[H.o_chain + tid * kChainInts + C_PBASE];
  }
  const double ec = __longlong_as_double((long long)*ecmax);
  __syncthreads();
  auto score64 = [&](uint32_t m) {  // FP64: one entry per chain
    double e = ec, qn = INFINITY, qx = 0.0;
    for (int c = 0; c < nch; ++c) {
      const size_t i = 3 * (size_t)(s_pb[c] + (int)gather_bits(m, (uint32_t)s_pm[c]));
      e = fmax(e, __longlong_as_double((long long)pat[i]));
      qn = fmin(qn, __longlong_as_double((long long)pat[i + 1]));
      qx = fmax(qx, __longlong_as_double((long long)pat[i + 2]));
    }
    MaskScore r;
    r.e = e;
    r.slack = band_slack(qn, qx, sp.vmin, sp.vmax);
    return r;
  };
  const int lb = tile_bits(H.k);
  const int ntiles = (int)((1u << H.k) >> lb);
  const double dd = sp.delta + sp.amb;
  auto is_sure = [&](const MaskScore32& r) { return (double)r.e <= sp.e_bar - dd && (double)r.slack >= dd; };
  auto is_poss = [&](const MaskScore32& r) { return (double)r.e <= sp.e_bar + dd && (double)r.slack >= -dd; };
  // the first kTileRegs tile records of each thread (all of them for segments of
  // up to 20 nodes) are read once, together, and kept in registers
  constexpr int kTileRegs = 16;
  TileRec32 rt[kTileRegs];
#pragma unroll
  for (int u = 0; u < kTileRegs; ++u) {
    if (u * bd >= ntiles) break;
    if (tid + u * bd < ntiles) rt[u] = tiles[tid + u * bd];
  }
  auto each_tile = [&](auto f) {
#pragma unroll
    for (int u = 0; u < kTileRegs; ++u) {
      if (u * bd >= ntiles) break;
      if (tid + u * bd < ntiles) f(rt[u], tid + u * bd);
    }
    for (int t = tid + kTileRegs * bd; t < ntiles; t += bd) f(tiles[t], t);
  };
  // visit(mask, its FP32 score) of every mask of the tiles that `want`: of all of
  // them at once, or (more than the list holds) a tile per thread at a time.
  // ncand is 0 at the start and again at the end.
  auto visit_all = [&](auto visit) {
    for (int q = tid, nc = ncand; q < nc * 64; q += bd)
      if (((q & 63) >> lb) == 0) {
        const uint32_t m = (uint32_t)cand[q >> 6] << lb | (uint32_t)(q & 63);
        visit(m, fin[m]);
      }
  };
  auto scan = [&](auto want, auto visit) {
    each_tile([&](const TileRec32& t, int at) {
      if (want(t)) {
        const int i = atomicAdd(&ncand, 1);
        if (i < 1024) cand[i] = at;
      }
    });
    __syncthreads();
    const bool all = ncand <= 1024;
    if (all) visit_all(visit);
    __syncthreads();
    if (tid == 0) ncand = 0;
    __syncthreads();
    for (int base = 0; !all && base < ntiles; base += bd) {
      if (base + tid < ntiles && want(tiles[base + tid])) cand[atomicAdd(&ncand, 1)] = base + tid;
      __syncthreads();
      visit_all(visit);
      __syncthreads();
      if (tid == 0) ncand = 0;
      __syncthreads();
    }
  };
  // list A: masks whose FP32 verdict is uncertain, at or above the best level
  // holding a surely feasible mask
  int lo = -1, hi = -1;
  each_tile([&](const TileRec32& t, int) {
    lo = max(lo, t.sure);
    hi = max(hi, t.poss);
  });
  if (tid == 0) ncand = nlist = 0;
  {
    const Levels v = block_reduce(
        Levels{lo, hi}, [](const Levels& a, const Levels& b) { return Levels{max(a.lo, b.lo), max(a.hi, b.hi)}; }, shv);
    lo = v.lo;
    hi = v.hi;
  }
  scan([&](const TileRec32& t) { return t.unc >= lo && t.unc >= 0; },
       [&](uint32_t m, const MaskScore32& r) {
         if (is_poss(r) && !is_sure(r) && __popc(m) >= lo) listA[atomicAdd(&nlist, 1)] = m;
       });
  const int nA = nlist;
  __syncthreads();
  // best level, and an upper bound on the smallest FP64 error there
  int best = lo;
  for (int q = tid; q < nA; q += bd) {
    const MaskScore r = score64(listA[q]);
    scoreA[q] = r;
    if (feasible(r, sp.e_bar)) best = max(best, __popc(listA[q]));
  }
  best = block_reduce(best, [](int a, int b) { return max(a, b); }, shi);
  if (tid == 0) {
    ms[g].lo_level = lo;
    ms[g].hi_level = hi;
    ms[g].nA = nA;
    ms[g].best = best;
    nlist = 0;
  }
  if (best < 0) {
    if (tid == 0) {
      ms[g].nB = 0;
      ms[g].max_dev = 0.0;
      nothing(1);
    }
    return;
  }
  double eup = INFINITY;
  scan([&](const TileRec32& t) { return t.sure >= best; },
       [&](uint32_t m, const MaskScore32& r) {
         if (__popc(m) == best && is_sure(r)) eup = fmin(eup, (double)r.e + sp.delta);
       });
  for (int q = tid; q < nA; q += bd)
    if (__popc(listA[q]) == best && feasible(scoreA[q], sp.e_bar)) eup = fmin(eup, scoreA[q].e);
  eup = block_reduce(eup, [](double a, double b) { return fmin(a, b); }, shd);
  const double bound = eup + sp.tie + sp.delta + sp.amb;
  // list B
  scan([&](const TileRec32& t) { return t.poss >= best; },
       [&](uint32_t m, const MaskScore32& r) {
         if (is_poss(r) && __popc(m) == best && (double)r.e <= bound) listB[atomicAdd(&nlist, 1)] = m;
       });
  const int nB = nlist;
  // FP64 arg-min over list B; ambiguity from the FP64 scores of A and B; the
  // largest FP32 deviation seen on refined masks is kept for reporting
  double emin = INFINITY, dev = 0.0;
  for (int q = tid; q < nB; q += bd) {
    const MaskScore r = score64(listB[q]);
    scoreB[q] = r;
    if (feasible(r, sp.e_bar)) emin = fmin(emin, r.e);
    if (r.e <= 2.0 * sp.e_bar) dev = fmax(dev, fabs((double)fin[listB[q]].e - r.e));
  }
  emin = block_reduce(emin, [](double a, double b) { return fmin(a, b); }, shd);
  const double thr = emin + sp.tie;
  unsigned pick = 0xffffffffu;
  int amb = 0;
  double runner = INFINITY;  // among the FP64-rescored masks of list B
  for (int q = tid; q < nB; q += bd) {
    const MaskScore r = scoreB[q];
    if (!feasible(r, sp.e_bar)) continue;
    if (fabs(r.e - thr) <= sp.amb) amb = 1;
    if (r.e <= thr) pick = min(pick, listB[q]);
    else runner = fmin(runner, r.e);
  }
  for (int q = tid; q < nA; q += bd) {
    const MaskScore r = scoreA[q];
    if (__popc(listA[q]) >= best && near_boundary(r, sp.e_bar, sp.amb)) amb = 1;
    if (r.e <= 2.0 * sp.e_bar) dev = fmax(dev, fabs((double)fin[listA[q]].e - r.e));
  }
  {
    const Verdict v = block_reduce(Verdict{dev, runner, pick, amb},
                                   [](const Verdict& a, const Verdict& b) {
                                     return Verdict{fmax(a.dev, b.dev), fmin(a.runner, b.runner),
                                                    (unsigned)min(a.pick, b.pick),
                                                    a.amb | b.amb};
                                   },
                                   shr);
    pick = v.pick;
    amb = v.amb;
    dev = v.dev;
    runner = v.runner;
  }
  if (tid == 0) {
    DevDecision d;
    const bool found = pick != 0xffffffffu;
    d.mask = found ? pick : 0u;
    d.popcount = best;
    d.e_loc = found ? score64(pick).e : 0.0;
    d.e_min = emin;
    d.ambiguous = amb;
    d.found = found;
    d.key_gap = runner - emin;
    d.smice_rise = 0.0;
    decs[g] = d;
    ms[g].nB = nB;
    ms[g].e_up = eup;
    ms[g].max_dev = dev;
    // the shortlists are complete only while |e32 - e64| <= delta: past the
    // bound the segment is decided again from every mask's FP64 score (and
    // that decision replaces this one)
    redo[g] = dev > sp.delta ? 1 : 0;
  }
}

}  // namespace okr
