// Candidate scoring kernels: a segment's numeric tables and chain patterns, every
// mask's score from them (FP64, and the FP32 difference-form screen of the
// mixed-precision search), and FP64 scores of a mask list.  Built with NaNs excluded (no input or intermediate here is
// NaN), which lets max/min compile to single instructions.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_internal.h"

namespace okr {

// ---------------------------------------------------------------- scoring --
// ------------------------------------------------- chain-term kernels --
// Exact FP64 terms of chains for given mask bits, folded into per-item
// accumulators by 64-bit atomics on the IEEE bit patterns.  Items are either
// (listed mask, chain) pairs -- the scores of a short mask list -- or chain
// patterns: for chain c and assignment u of its C_PMASK bits (bit j of u at
// the j-th lowest set bit), the chain's terms.  Every folded value is a
// non-negative double (errors max(|V| - lo, hi - |V|) with lo <= hi, squared
// magnitudes), and for those the bit patterns order like the values; max and
// min are exact, so any grouping of the folds gives the same scores.  qmax
// starts at +0 instead of -inf: band_slack treats both alike (no kept
// node-phase).

// ---- a segment's numeric tables and its chain patterns, per snapshot ----
//
// A block serves NS snapshots (blockIdx.x; 256 threads and tables of its own
// each) of one unit (a segment of the chunk, or a part of its pattern items).
// With BUILD it forms the snapshots' tables in LDS from the search state -- P =
// Z(super -> reduced) A_reduced with Z(s -> r) = Zroot(r) - Zroot(s), the
// records' voltages, every cluster's smallest and largest |V^| over its
// members, the constant error of clusters outside Omega_g -- and writes them
// out (part 0) for the kernels that read them later (state update, SMICE, short
// lists, the FP32 screen); without, it stages the tables an earlier launch
// wrote.  With PAT it then folds every pattern's terms into the segment's
// pattern table, in LDS over its NS snapshots first where the table fits there:
// the atomics to memory are performed beyond the XCDs' caches and bound the
// launch (31 of 78 us on the 8400-node feeder with one snapshot per block).
//
// Building where the patterns are evaluated saves two launches and the
// tables' round trip through memory.  An item walks its chain's upper slots
// once and enumerates the bottom C_D of them by nested loops whose branch is
// the same for the whole wave: about 2.75 slot evaluations per pattern of a
// chain of 11 bits instead of 11.  (Chains with zone entries enumerate fewer
// slots: a thread would go through the entries once per pattern of its item.)
//
// A chain with more zone entries below it than it has patterns (and at least
// kZoneWave of them) leaves the few threads of its patterns with hundreds of
// entries in turn while the block waits (launches of 150 to 650 us on the
// 8400-node feeder, whose chains carry up to 1,115 entries).  Its entries are
// evaluated by whole waves instead: one wave per pattern walks the chain for
// its exit value and takes an entry per lane.
//
// Per launch (chunks of up to 8 segments): 11.1 us at 1000 nodes and 24
// snapshots, 21.5 at 6000 and 96, 58.4 at 8400 and 288 (with k_fac_combine 18,
// 31 and 74), where the tables took 13, 20 and 26 us in two launches and scoring
// mask by mask 79, 577 and 4412.
struct ChainState {
  double2 S[3];   // voltage shift
  double sm[3];   // magnitude of the current super
  int sidx;       // its slot + 1 (0: the head)
  double e, qn, qx;
};

// One slot for the present phases `ph`: reduced (the moved current's rise pr,
// the slot's cluster against the current super) or kept (it becomes the super
// of the slots below).  No branch on the phase: the three phases' loads and
// square roots overlap (a branch each made a slot wait for them in turn), and
// an absent phase contributes nothing -- its magnitude is taken of 1 and its
// terms are discarded; its shift is never read again, since phases only
// shrink down a chain.  SKIP branches instead: segments with thousands of
// patterns keep every lane of a wave on one chain and are bound by the
// arithmetic (79 against 88 ms on a 300-node feeder of 20-node chains).
template <bool SKIP>
__device__ __forceinline__ void slot_reduced(ChainState& s, int ph, const double2* pr, const TargetRec* tr) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (SKIP && !(ph >> p & 1)) continue;
    const double2 pv = pr[p];
    s.S[p].x += pv.x;
    s.S[p].y += pv.y;
    const double d = fmax(s.sm[p] - tr[p].lo, tr[p].hi - s.sm[p]);
    s.e = fmax(s.e, (ph >> p & 1) ? d : 0.0);
  }
}
template <bool SKIP>
__device__ __forceinline__ void slot_kept(ChainState& s, int ph, int r, const TargetRec* tr) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (SKIP && !(ph >> p & 1)) continue;
    const bool on = ph >> p & 1;
    const TargetRec t = tr[p];
    const double vx = t.W.x + s.S[p].x, vy = t.W.y + s.S[p].y;
    const double q = on ? fma(vx, vx, vy * vy) : 1.0;
    s.sm[p] = sqrt_nr(q);
    s.qn = fmin(s.qn, on ? q : INFINITY);
    s.qx = fmax(s.qx, on ? q : 0.0);
    const double d = fmax(s.sm[p] - t.lo, t.hi - s.sm[p]);
    s.e = fmax(s.e, on ? d : 0.0);
  }
  s.sidx = r + 1;
}
// The same with lanes that differ in the slot's bit: both sides by selects.
template <bool SKIP>
__device__ __forceinline__ void slot_either(ChainState& s, int ph, int r, bool red, const double2* pr,
                                            const TargetRec* tr) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (SKIP && !(ph >> p & 1)) continue;
    const bool on = ph >> p & 1;
    const TargetRec t = tr[p];
    const double2 pv = pr[p];
    s.S[p].x += red ? pv.x : 0.0;
    s.S[p].y += red ? pv.y : 0.0;
    const double vx = t.W.x + s.S[p].x, vy = t.W.y + s.S[p].y;
    const double q = on ? fma(vx, vx, vy * vy) : 1.0;
    const double m = sqrt_nr(q);
    s.sm[p] = red ? s.sm[p] : m;
    s.qn = fmin(s.qn, on && !red ? q : INFINITY);
    s.qx = fmax(s.qx, on && !red ? q : 0.0);
    const double d = fmax(s.sm[p] - t.lo, t.hi - s.sm[p]);
    s.e = fmax(s.e, on ? d : 0.0);
  }
  s.sidx = red ? s.sidx : r + 1;
}
// One zone entry of the chain, shifted by its exit value b.
__device__ __forceinline__ void zone_term(ChainState& s, const TargetRec& t, double2 b) {
  const double vx = t.W.x + b.x, vy = t.W.y + b.y;
  const double q = fma(vx, vx, vy * vy);
  const double mag = sqrt_nr(q);
  s.e = fmax(s.e, fmax(mag - t.lo, t.hi - mag));
  s.qn = fmin(s.qn, q);
  s.qx = fmax(s.qx, q);
}
// Voltage shift of one slot alone.
__device__ __forceinline__ void slot_shift(double2 (&S)[3], int& sidx, int r, bool red, const double2* pr) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const double2 pv = pr[p];
    S[p].x += red ? pv.x : 0.0;
    S[p].y += red ? pv.y : 0.0;
  }
  sidx = red ? sidx : r + 1;
}

// Voltage shift through a whole chain (its rows of the pair table at P).  A
// slot's row is zero on phases absent from the chain's paths; a row's value on
// a phase absent from its slot only reaches phases that no lower slot has.
__device__ __forceinline__ void chain_shift(const int* cr, const double2* P, uint32_t m, double2 (&S)[3]) {
  const int ns = cr[C_NSLOT], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
  int sidx = 0;
  for (int r = 0; r < ns; ++r)
    slot_shift(S, sidx, r, (m >> (bit0 + r)) & 1u, P + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3);
}

constexpr int kTermsBlock = 256;  // threads of a chain-term block
constexpr int kZoneWave = 32;     // zone entries from which a chain's patterns may take them by waves

// Whether the zone entries of a chain are taken by a wave per pattern: where
// it has 8 times as many entries as patterns (a wave takes about 2000 cycles
// per pattern -- the walk, the entries, a 6-step fold -- and a block has 4; a
// thread going through the entries of its pattern about 70 per entry).
__device__ __forceinline__ bool zone_by_wave(const int* cr) {
  const int z = cr[C_ZCNT0] + cr[C_ZCNT1] + cr[C_ZCNT2];
  return z >= kZoneWave && (8 << __popc((uint32_t)cr[C_PMASK])) <= z;
}

// The mask whose bits at pm's positions are u's low bits, the rest 0.
__device__ __forceinline__ uint32_t deposit_bits(uint32_t u, uint32_t pm) {
  uint32_t mask = 0;
  for (; pm; u >>= 1) {
    const uint32_t low = pm & (0u - pm);
    if (u & 1u) mask |= low;
    pm ^= low;
  }
  return mask;
}

template <bool BUILD, bool PAT, int NS, bool DEEP>
__global__ __launch_bounds__(kTermsBlock * NS) void k_seg_terms(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ units,
    const int* __restrict__ tab, Topo T, State St, const double2* __restrict__ Zroot,
    const double2* __restrict__ Vcur, const double2* __restrict__ A, const double* __restrict__ absV,
    double2* __restrict__ P, TargetRec* __restrict__ srec, double2* __restrict__ headV,
    TargetRec* __restrict__ zrec, double* __restrict__ econst, TermsCaps caps,
    unsigned long long* __restrict__ pat, unsigned long long* __restrict__ ecmax, const int* __restrict__ gates,
    int* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char ct_lds[];
  __shared__ double s_ecs[NS];
  __shared__ int s_zw[kMaxK + 1];  // patterns of the chains before c whose zone entries go by waves
  const int u = *as_cint(units + blockIdx.y);
  const int uz = u & 255, part = (u >> 8) & 255, parts = u >> 16;
  const int g = *as_cint(segs + uz);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid || (gates && gates[g] == 0)) return;
  const int sub = NS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kTermsBlock) : 0;
  const int tid = threadIdx.x - sub * kTermsBlock;  // within the snapshot's threads
  // (parts come from the plan's bound on the patterns; a part without items
  // may still have zone patterns, which are fewer than the segment's entries)
  if (PAT && part > 0 && part * kTermsBlock >= (DEEP ? H.nitem : H.npat) && part * (kTermsBlock / 64) >= H.nz) return;
  // the plan's bounds hold the tables (zone entries beyond their LDS take
  // memory; with BUILD and PAT together they all fit)
  if (H.npairs > caps.pairs || H.nslots > caps.slots || H.o_slot > caps.ints ||
      (BUILD && PAT && H.nz > caps.zones)) {
    if (threadIdx.x == 0) atomicOr(status, kStatusBuild);
    return;
  }
  tab = lane_ptr_z(tab, lstride, uz);
  P = lane_ptr_z(P, lstride, uz);
  srec = lane_ptr_z(srec, lstride, uz);
  headV = lane_ptr_z(headV, lstride, uz);
  zrec = lane_ptr_z(zrec, lstride, uz);
  econst = lane_ptr_z(econst, lstride, uz);
  const int l = blockIdx.x * NS + sub, n = T.n;
  const bool on = l < H.S;  // (the last block's surplus threads only pass the barriers)
  const int nint = H.o_slot;  // chain records and nesting paths
  const int zst = min(H.nz, caps.zones);
  const bool fold_lds = NS > 1 && H.npat <= caps.pats;  // patterns folded in LDS over the block's snapshots
  int* si = (int*)ct_lds;
  unsigned long long* sA = (unsigned long long*)(ct_lds + (size_t)(caps.ints + 3) / 4 * 16);
  double2* sP = (double2*)((unsigned char*)(sA + (size_t)(caps.pats + 1) / 2 * 6) + (size_t)sub * terms_snap_lds(caps));
  TargetRec* sS = (TargetRec*)(sP + (size_t)caps.pairs * 3);
  double2* sH = (double2*)(sS + (size_t)caps.slots * 3);
  TargetRec* sZ = (TargetRec*)(sH + (size_t)caps.slots * 3);
  double& s_ec = s_ecs[sub];
  double2* gP = P + (size_t)l * H.npairs * 3;
  TargetRec* gS = srec + (size_t)l * H.nslots * 3;
  double2* gH = headV + (size_t)l * H.nchains * 3;
  TargetRec* gZ = zrec + (size_t)l * H.nz;
  for (int i = threadIdx.x; i < nint; i += kTermsBlock * NS) si[i] = tab[i];
  if (fold_lds)
    for (int x = threadIdx.x; x < H.npat; x += kTermsBlock * NS) {
      sA[3 * x] = 0ull;
      sA[3 * x + 1] = (unsigned long long)__double_as_longlong(INFINITY);
      sA[3 * x + 2] = 0ull;
    }
  const double2* Vl = Vcur + (size_t)l * n * 3;
  if (BUILD) {
    const double2* Al = A + (size_t)l * n * 3;
    const double* av = absV + (size_t)l * n * 3;
    if (tid == 0) s_ec = 0.0;
    // members: every node of Omega_g contributes |V^| to the cluster of its
    // current super-node (a slot, a zone target, or a head outside Omega_g,
    // whose error is mask-independent and folds into the constant error).  The
    // last threads take the first nodes, so that their chain of loads (node,
    // super-node, its slot or entry) runs beside the pairs' of the first ones.
    const int* rg = tab + H.o_range;
    struct Member {
      int to[3];    // -1: nothing; slot record; kMZone | zone entry; kMConst
      double a[3];  // |V^|, or the error against a head outside
    };
    constexpr int kMZone = 1 << 28, kMConst = 1 << 29;
    auto member = [&](int q) {
      Member m;
#pragma unroll
      for (int p = 0; p < 3; ++p) m.to[p] = -1;
      if (q >= H.nomega) return m;
      int r = 0;
      while (r + 1 < H.nrange && rg[3 * (r + 1) + 2] <= q) ++r;
      const int i = rg[3 * r] + (q - rg[3 * r + 2]);
      const int sp = St.sup[i];
      const unsigned ph = T.phase[i];
#pragma unroll
      for (int p = 0; p < 3; ++p) m.a[p] = av[(size_t)i * 3 + p];
      const int sg = T.segment[sp], s = St.slot_of[sp];
      int zi[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) zi[p] = St.zent_of[sp * 3 + p];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        if (!(ph >> p & 1u)) continue;
        if (sg == g) {
          if (s >= 0 && s < H.nslots) m.to[p] = s * 3 + p;
        } else if (zi[p] >= 0) {
          if (zi[p] < H.nz) m.to[p] = kMZone | zi[p];
        } else {
          const double2 v = Vl[(size_t)sp * 3 + p];
          m.to[p] = kMConst;
          m.a[p] = fabs(sqrt(v.x * v.x + v.y * v.y) - m.a[p]);
        }
      }
      return m;
    };
    auto fold = [](TargetRec* r, double v) {
      atomicMin((unsigned long long*)&r->lo, (unsigned long long)__double_as_longlong(v));
      atomicMax((unsigned long long*)&r->hi, (unsigned long long)__double_as_longlong(v));
    };
    auto fold_member = [&](const Member& m) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        if (m.to[p] < 0) continue;
        if (m.to[p] == kMConst) {
          atomicMax((unsigned long long*)&s_ec, (unsigned long long)__double_as_longlong(m.a[p]));
        } else if (m.to[p] & kMZone) {
          const int zi = m.to[p] & ~kMZone;
          if (zi < zst) fold(&sZ[zi], m.a[p]);
          else fold(&gZ[zi], m.a[p]);
        } else {
          fold(&sS[m.to[p]], m.a[p]);
        }
      }
    };
    const int q0 = on ? kTermsBlock - 1 - tid : INT_MAX;
    const Member m0 = member(q0);
    // one index space over pairs, slot-phases, chains and zone entries
    const int nP = H.npairs, nS = H.nslots * 3, nC = H.nchains * 3;
    for (int x = on ? tid : INT_MAX; x < nP + nS + nC + H.nz; x += kTermsBlock) {
      if (x < nP) {
        const int* pr = tab + H.o_pair + x * kPairInts;
        const int rn = pr[PR_RNODE], sn = pr[PR_SUPER];
        const double2 *zr = Zroot + (size_t)rn * 9, *zs = Zroot + (size_t)sn * 9;
        const double2* a = Al + (size_t)rn * 3;
        double2 Z[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) Z[e] = csub(zr[e], zs[e]);
#pragma unroll
        for (int r = 0; r < 3; ++r)
          sP[x * 3 + r] = cadd(cadd(cmul(Z[r * 3], a[0]), cmul(Z[r * 3 + 1], a[1])), cmul(Z[r * 3 + 2], a[2]));
      } else if (x < nP + nS) {
        const int y = x - nP, s = y / 3, p = y - s * 3;
        TargetRec rec;
        rec.W = Vl[(size_t)tab[H.o_slot + s * kSlotInts + SL_NODE] * 3 + p];
        rec.lo = INFINITY;
        rec.hi = 0.0;
        sS[y] = rec;
      } else if (x < nP + nS + nC) {
        const int y = x - nP - nS, c = y / 3, p = y - c * 3;
        sH[y] = Vl[(size_t)tab[H.o_chain + c * kChainInts + C_HEAD] * 3 + p];
      } else {
        const int q = x - nP - nS - nC;
        const int* ze = tab + H.o_zent + q * 3;
        TargetRec rec;
        rec.W = Vl[(size_t)ze[0] * 3 + ze[1]];
        rec.lo = INFINITY;
        rec.hi = 0.0;
        if (q < zst) sZ[q] = rec;
        else gZ[q] = rec;
      }
    }
    __syncthreads();
    fold_member(m0);
    for (int q = on ? q0 + kTermsBlock : INT_MAX; q < H.nomega; q += kTermsBlock) fold_member(member(q));
    __syncthreads();
    if (part == 0 && on) {
      uint4 *dP = (uint4*)gP, *dS = (uint4*)gS, *dH = (uint4*)gH, *dZ = (uint4*)gZ;
      for (int i = tid; i < H.npairs * 3; i += kTermsBlock) dP[i] = ((const uint4*)sP)[i];
      for (int i = tid; i < H.nslots * 6; i += kTermsBlock) dS[i] = ((const uint4*)sS)[i];
      for (int i = tid; i < H.nchains * 3; i += kTermsBlock) dH[i] = ((const uint4*)sH)[i];
      for (int i = tid; i < zst * 2; i += kTermsBlock) dZ[i] = ((const uint4*)sZ)[i];
      if (tid == 0) econst[l] = s_ec;
    }
  } else {
    const int cP = H.npairs * 3, cS = H.nslots * 6, cH = H.nchains * 3, cZ = zst * 2;
    for (int i = on ? tid : INT_MAX; i < cP + cS + cH + cZ; i += kTermsBlock) {
      if (i < cP) ((uint4*)sP)[i] = ((const uint4*)gP)[i];
      else if (i < cP + cS) ((uint4*)sS)[i - cP] = ((const uint4*)gS)[i - cP];
      else if (i < cP + cS + cH) ((uint4*)sH)[i - cP - cS] = ((const uint4*)gH)[i - cP - cS];
      else ((uint4*)sZ)[i - cP - cS - cH] = ((const uint4*)gZ)[i - cP - cS - cH];
    }
    if (tid == 0 && on) s_ec = econst[l];
    __syncthreads();
  }
  if (!PAT) return;
  pat = lane_ptr_z(pat, lstride, uz);
  if (part == 0 && tid == 0 && on)
    atomicMax(lane_ptr_z(ecmax, lstride, uz), (unsigned long long)__double_as_longlong(s_ec));
  const int* chains = si + H.o_chain;
  const int* nest = si + H.o_nest;
  const int nch = H.nchains;
  auto emit = [&](int x, double e, double qn, double qx) {
    const unsigned long long ve = (unsigned long long)__double_as_longlong(e),
                             vn = (unsigned long long)__double_as_longlong(qn),
                             vx = (unsigned long long)__double_as_longlong(qx);
    if (fold_lds) {
      atomicMax(&sA[3 * x], ve);
      atomicMin(&sA[3 * x + 1], vn);
      atomicMax(&sA[3 * x + 2], vx);
    } else {
      atomicMax(&pat[3 * (size_t)x], ve);
      if (qn < INFINITY) atomicMin(&pat[3 * (size_t)x + 1], vn);
      if (qx > 0.0) atomicMax(&pat[3 * (size_t)x + 2], vx);
    }
  };
  if (threadIdx.x < 64) {
    const bool zw = tid < nch && zone_by_wave(chains + tid * kChainInts);
    const int v = zw ? 1 << __popc((uint32_t)chains[tid * kChainInts + C_PMASK]) : 0;
    int x = v;
    for (int o = 1; o < 32; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (tid >= o) x += y;
    }
    if (tid <= nch) s_zw[tid] = x - v;
  }
  constexpr int kBase = DEEP ? (int)C_IBASE : (int)C_PBASE;
  const int nitem = DEEP ? H.nitem : H.npat;
  int c = 0;  // (a thread's items increase, so its chain index only moves forward)
  for (int it = on ? part * kTermsBlock + tid : INT_MAX; it < nitem; it += parts * kTermsBlock) {
    while (c + 1 < nch && chains[(c + 1) * kChainInts + kBase] <= it) ++c;
    const int* cr = chains + c * kChainInts;
    const uint32_t ulow = (uint32_t)(it - cr[kBase]);
    const uint32_t pm = (uint32_t)cr[C_PMASK];
    const int d = DEEP ? cr[C_D] : 0, ub = __popc(pm) - d;  // the item's own bits; the d bits above them are enumerated
    const uint32_t mask = deposit_bits(ulow, pm);
    const bool zw = zone_by_wave(cr);
    ChainState s0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      s0.S[p] = make_double2(0.0, 0.0);
      s0.sm[p] = 0.0;
    }
    s0.sidx = 0;
    s0.e = 0.0;
    s0.qn = INFINITY;
    s0.qx = 0.0;
    const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
    for (int q = 0; q + 1 < nl; ++q)  // the nesting path down to the chain's head: voltage shifts only
      chain_shift(chains + nest[no + q] * kChainInts, sP, mask, s0.S);
    {  // the head's magnitude (1 on absent phases, never read), moved by the outer chains when it lies below one
      const int hph = cr[C_PHASE];
#pragma unroll
      for (int p = 0; p < 3; ++p)
      {
        const double2 h = nl > 1 ? cadd(sH[c * 3 + p], s0.S[p]) : sH[c * 3 + p];
        s0.sm[p] = sqrt_nr((hph >> p & 1) ? mag2(h) : 1.0);
      }
    }
    const int ns = cr[C_NSLOT], slot0 = cr[C_SLOT0], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
    const int phw0 = cr[C_PHW0], phw1 = cr[C_PHW1], phw2 = cr[C_PHW2];
    auto phase_of = [&](int r) { return ((r < 8 ? phw0 : (r < 16 ? phw1 : phw2)) >> (3 * (r & 7))) & 7; };
    auto pair_row = [&](int r, int sidx) { return sP + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3; };
    for (int r = 0; r < ns - d; ++r)  // the item's own slots
      slot_either<DEEP>(s0, phase_of(r), r, (mask >> (bit0 + r)) & 1u, pair_row(r, s0.sidx), sS + (slot0 + r) * 3);
    const int pb = cr[C_PBASE] + (int)ulow;
    auto zones = [&](ChainState& s, int p, double2 b) {  // the entries anchored below, shifted by the chain's exit value
      int q = cr[C_ZOFF0 + p];
      const int qe = zw ? q : q + cr[C_ZCNT0 + p];
#pragma unroll 2
      for (const int ql = min(qe, zst); q < ql; ++q) zone_term(s, sZ[q], b);
      if (!BUILD)  // (entries past the LDS stage, which holds them all when this launch built them)
        for (; q < qe; ++q) zone_term(s, gZ[q], b);
    };
    auto finish = [&](ChainState& s, int x) {
      zones(s, 0, s.S[0]);
      zones(s, 1, s.S[1]);
      zones(s, 2, s.S[2]);
      emit(x, s.e, s.qn, s.qx);
    };
    if (!DEEP) {
      finish(s0, pb);
    } else {
      auto step = [&](ChainState& s, int r, int red) {
        const int ph = phase_of(r);
        const TargetRec* tr = sS + (slot0 + r) * 3;
        if (red) slot_reduced<true>(s, ph, pair_row(r, s.sidx), tr);
        else slot_kept<true>(s, ph, r, tr);
      };
#pragma unroll 1
      for (int b0 = 0; b0 < (d > 2 ? 2 : 1); ++b0) {
        ChainState s1 = s0;
        if (d > 2) step(s1, ns - 3, b0);
#pragma unroll 1
        for (int b1 = 0; b1 < (d > 1 ? 2 : 1); ++b1) {
          ChainState s2 = s1;
          if (d > 1) step(s2, ns - 2, b1);
#pragma unroll 1
          for (int b2 = 0; b2 < (d > 0 ? 2 : 1); ++b2) {
            ChainState s3 = s2;
            if (d > 0) step(s3, ns - 1, b2);
            finish(s3, pb + (((b0 | b1 << 1 | b2 << 2) >> (3 - d)) << ub));
          }
        }
      }
    }
  }
  // zone entries by waves: one (chain, pattern) per wave, one entry per lane
  __syncthreads();
  const int nzw = on ? s_zw[nch] : 0, lane = tid & 63;
  constexpr int kWaves = kTermsBlock / 64;
  c = 0;
  for (int x = part * kWaves + (tid >> 6); x < nzw; x += parts * kWaves) {
    while (s_zw[c + 1] <= x) ++c;  // (chains without a wave pattern have equal entries: skipped)
    const int* cr = chains + c * kChainInts;
    const int ux = x - s_zw[c];
    const uint32_t mm = deposit_bits((uint32_t)ux, (uint32_t)cr[C_PMASK]);
    double2 B[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) B[p] = make_double2(0.0, 0.0);
    for (int q = 0, no = cr[C_NEST_OFF]; q < cr[C_NEST_LEN]; ++q)  // (the path ends with the chain itself)
      chain_shift(chains + nest[no + q] * kChainInts, sP, mm, B);
    ChainState t;
    t.e = 0.0;
    t.qn = INFINITY;
    t.qx = 0.0;
    auto zones = [&](int p, double2 b) {
      int q = cr[C_ZOFF0 + p] + lane;
      const int qe = cr[C_ZOFF0 + p] + cr[C_ZCNT0 + p];
      for (const int ql = min(qe, zst); q < ql; q += 64) zone_term(t, sZ[q], b);
      if (!BUILD)
        for (; q < qe; q += 64) zone_term(t, gZ[q], b);
    };
    zones(0, B[0]);
    zones(1, B[1]);
    zones(2, B[2]);
    double e = t.e, qn = t.qn, qx = t.qx;
    for (int o = 32; o > 0; o >>= 1) {
      e = fmax(e, __shfl_xor(e, o, 64));
      qn = fmin(qn, __shfl_xor(qn, o, 64));
      qx = fmax(qx, __shfl_xor(qx, o, 64));
    }
    if (lane == 0) emit(cr[C_PBASE] + ux, e, qn, qx);
  }
  if (!fold_lds) return;
  __syncthreads();
  for (int x = threadIdx.x; x < H.npat; x += kTermsBlock * NS) {
    if (sA[3 * x] != 0ull) atomicMax(&pat[3 * (size_t)x], sA[3 * x]);
    if (sA[3 * x + 1] != (unsigned long long)__double_as_longlong(INFINITY))
      atomicMin(&pat[3 * (size_t)x + 1], sA[3 * x + 1]);
    if (sA[3 * x + 2] != 0ull) atomicMax(&pat[3 * (size_t)x + 2], sA[3 * x + 2]);
  }
}

#define OKR_SEG_TERMS_INST(B_, P_, N_, D_)                                                                            \
  template __global__ void k_seg_terms<B_, P_, N_, D_>(                                                               \
      const SegHdr*, const int*, size_t, const int*, const int*, Topo, State, const double2*, const double2*,         \
      const double2*, const double*, double2*, TargetRec*, double2*, TargetRec*, double*, TermsCaps,                  \
      unsigned long long*, unsigned long long*, const int*, int*);
OKR_SEG_TERMS_INST(true, true, 1, false)
OKR_SEG_TERMS_INST(true, true, 2, false)
OKR_SEG_TERMS_INST(true, true, 1, true)
OKR_SEG_TERMS_INST(true, false, 1, false)
OKR_SEG_TERMS_INST(false, true, 1, true)
#undef OKR_SEG_TERMS_INST

// ---- terms of a short mask list ----

// Clears the list's accumulators (the pattern table's are cleared by
// the table build).
__global__ void k_terms_init(const int* __restrict__ count, int cap, size_t lstride,
                             unsigned long long* __restrict__ acc) {
  count = lane_ptr(count, lstride);
  acc = lane_ptr(acc, lstride);
  const int n = min(*count, cap);
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
    acc[3 * q] = 0ull;
    acc[3 * q + 1] = (unsigned long long)__double_as_longlong(INFINITY);
    acc[3 * q + 2] = 0ull;
  }
}

// One lane per (listed mask, chain, snapshot).  A block serves one snapshot
// (blockIdx.y) of one segment (blockIdx.z of a chunk): it first stages the
// chain records and nesting paths and the snapshot's pair, slot, head and
// first zcap zone records in LDS (one coalesced round trip), then walks every
// item's chain from there.
__global__ __launch_bounds__(kTermsBlock) void k_chain_terms(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ tab,
    const double2* __restrict__ P, const TargetRec* __restrict__ srec, const double2* __restrict__ headV,
    const TargetRec* __restrict__ zrec, const double* __restrict__ econst, const uint32_t* __restrict__ list,
    const int* __restrict__ count, int cap, int icap, int zcap, unsigned long long* __restrict__ acc) {
  extern __shared__ __align__(16) unsigned char ct_lds[];
  const SegHdr H = load_hdr(hdrs, segs);
  if (!H.valid) return;
  tab = lane_ptr(tab, lstride);
  P = lane_ptr(P, lstride);
  srec = lane_ptr(srec, lstride);
  headV = lane_ptr(headV, lstride);
  zrec = lane_ptr(zrec, lstride);
  econst = lane_ptr(econst, lstride);
  list = lane_ptr(list, lstride);
  count = lane_ptr(count, lstride);
  acc = lane_ptr(acc, lstride);
  const int items = min(*count, cap) * H.nchains;
  const int l = blockIdx.y;
  if ((int)(blockIdx.x * blockDim.x) >= items) return;  // whole block idle
  // stage: chain records and nesting paths (ints [0, o_slot)), then this
  // snapshot's pairs, slot records, heads and first zone records
  const int nint = H.o_slot;
  const int zst = min(H.nz, zcap);
  int* si = (int*)ct_lds;
  double2* sP = (double2*)(ct_lds + (size_t)((icap * 4 + 15) / 16) * 16);
  TargetRec* sS = (TargetRec*)(sP + (size_t)H.npairs * 3);
  double2* sH = (double2*)(sS + (size_t)H.nslots * 3);
  TargetRec* sZ = (TargetRec*)(sH + (size_t)H.nchains * 3);
  const uint4* gP = (const uint4*)(P + (size_t)l * H.npairs * 3);
  const uint4* gS = (const uint4*)(srec + (size_t)l * H.nslots * 3);
  const uint4* gH = (const uint4*)(headV + (size_t)l * H.nchains * 3);
  const uint4* gZ = (const uint4*)(zrec + (size_t)l * H.nz);
  const int cP = H.npairs * 3, cS = H.nslots * 6, cH = H.nchains * 3, cZ = zst * 2;
  for (int i = threadIdx.x; i < nint; i += blockDim.x) si[i] = tab[i];
  for (int i = threadIdx.x; i < cP + cS + cH + cZ; i += blockDim.x) {
    if (i < cP) ((uint4*)sP)[i] = gP[i];
    else if (i < cP + cS) ((uint4*)sS)[i - cP] = gS[i - cP];
    else if (i < cP + cS + cH) ((uint4*)sH)[i - cP - cS] = gH[i - cP - cS];
    else ((uint4*)sZ)[i - cP - cS - cH] = gZ[i - cP - cS - cH];
  }
  __syncthreads();
  const int* chains = si + H.o_chain;
  const int* nest = si + H.o_nest;
  const int nch = H.nchains;
  const double ec = econst[l];
  // a block's items cover consecutive listed masks (each with all its
  // chains): fold them in LDS first, then one global atomic per mask
  __shared__ unsigned long long s_acc[3 * (kTermsBlock + 2)];
  for (int base = blockIdx.x * blockDim.x; base < items; base += gridDim.x * blockDim.x) {
    const int q0 = base / nch, q1 = min(items - 1, base + (int)blockDim.x - 1) / nch;
    for (int i = threadIdx.x; i <= q1 - q0; i += blockDim.x) {
      s_acc[3 * i] = 0ull;
      s_acc[3 * i + 1] = (unsigned long long)__double_as_longlong(INFINITY);
      s_acc[3 * i + 2] = 0ull;
    }
    __syncthreads();
    const int it = base + threadIdx.x;
    if (it < items) {
      const int q = it / nch, c = it - q * nch;
      double el = ec, qn = INFINITY, qx = 0.0;
      score_chain(chains, nest, c, sP, sS, sH, sZ, zst, zrec + (size_t)l * H.nz, list[q], el, qn, qx);
      unsigned long long* a = s_acc + 3 * (q - q0);
      atomicMax(&a[0], (unsigned long long)__double_as_longlong(el));
      if (qn < INFINITY) atomicMin(&a[1], (unsigned long long)__double_as_longlong(qn));
      if (qx > 0.0) atomicMax(&a[2], (unsigned long long)__double_as_longlong(qx));
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= q1 - q0; i += blockDim.x) {
      const int q = q0 + i;
      atomicMax(&acc[3 * q], s_acc[3 * i]);
      if (s_acc[3 * i + 1] != (unsigned long long)__double_as_longlong(INFINITY))
        atomicMin(&acc[3 * q + 1], s_acc[3 * i + 1]);
      if (s_acc[3 * i + 2] != 0ull) atomicMax(&acc[3 * q + 2], s_acc[3 * i + 2]);
    }
    __syncthreads();
  }
}

// Scores of a short mask list from its accumulators.
__global__ void k_list_finish(const int* __restrict__ count, const unsigned long long* __restrict__ acc, int cap,
                              SelParams sp, MaskScore* __restrict__ out, size_t lstride) {
  count = lane_ptr(count, lstride);
  acc = lane_ptr(acc, lstride);
  out = lane_ptr(out, lstride);
  const int n = min(*count, cap);
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
    MaskScore r;
    r.e = __longlong_as_double((long long)acc[3 * q]);
    r.slack = band_slack(__longlong_as_double((long long)acc[3 * q + 1]),
                         __longlong_as_double((long long)acc[3 * q + 2]), sp.vmin, sp.vmax);
    out[q] = r;
  }
}

// Every mask's score from the pattern table: the largest constant error and
// each chain's entry for the mask's bits, then the per-mask scores and 64-mask
// tile records that the arg-min reads.
//
// A wave takes per tiles (2, 4 or 8).  Against a tile's 6 lane bits a chain is
// inside (its entry is the lane's for every tile: folded once per wave),
// outside (the same for the tile's 64 masks: tile t's fold is formed in lane t
// and read from there) or across (an entry per mask); so a mask costs about one
// entry instead of one per chain (11 on the 1000-node workload).  Entries are
// (error, band slack): the slack of an entry's extreme squared magnitudes is
// formed once when it is staged, which is exact, the square root being
// monotone.  Levels come from ballots, and a score is stored only where it is
// read: every mask when all are wanted (dumps, surrogate targets), else mask 0
// and the tile's masks at its best feasible level (on segments of 20 nodes the
// stores of all, 16 MB each, took most of the launch).
constexpr int kPatLds = 2048;      // pattern-table entries staged in LDS (32 KB)

__global__ __launch_bounds__(256) void k_fac_combine(const SegHdr* __restrict__ hdrs, const int* __restrict__ segs,
                                                     size_t lstride, const int* __restrict__ tab,
                                                     const unsigned long long* __restrict__ pat,
                                                     const unsigned long long* __restrict__ ecmax, SelParams sp,
                                                     MaskScore* __restrict__ fin, TileRec* __restrict__ tiles,
                                                     const int* __restrict__ gates, int full_fin, int per) {
  __shared__ int s_pm[kMaxK], s_pb[kMaxK];
  __shared__ double2 s_pat[kPatLds];
  const int g = *as_cint(segs + blockIdx.z);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid || (gates && gates[g] == 0)) return;
  const int lb = tile_bits(H.k);
  const uint32_t ntiles = 1u << (H.k - lb);
  if (blockIdx.x * (4 * per) >= ntiles) return;  // past this segment's masks
  tab = lane_ptr(tab, lstride);
  pat = lane_ptr(pat, lstride);
  ecmax = lane_ptr(ecmax, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  const int tid = threadIdx.x, lane = tid & 63;
  const int nch = H.nchains;
  if (tid < nch) {
    s_pm[tid] = tab[H.o_chain + tid * kChainInts + C_PMASK];
    s_pb[tid] = tab[H.o_chain + tid * kChainInts + C_PBASE];
  }
  auto entry = [&](int i) {  // (error, band slack) of pattern i
    return make_double2(__longlong_as_double((long long)pat[3 * (size_t)i]),
                        band_slack(__longlong_as_double((long long)pat[3 * (size_t)i + 1]),
                                   __longlong_as_double((long long)pat[3 * (size_t)i + 2]), sp.vmin, sp.vmax));
  };
  for (int i = tid; i < min(H.npat, kPatLds); i += 256) s_pat[i] = entry(i);
  const double ec = __longlong_as_double((long long)*ecmax);
  __syncthreads();
  auto look = [&](int i) { return i < kPatLds ? s_pat[i] : entry(i); };
  const uint32_t t0 = (blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6)) * per;
  if (t0 >= ntiles) return;
  const uint32_t lmask = (1u << lb) - 1u;
  double el = ec, sl = INFINITY;    // chains inside the lane bits, this lane's
  double eu = 0.0, su = INFINITY;   // chains outside, of tile t0 + lane
  uint32_t across = 0;              // chains across
  const uint32_t mt = (t0 + (uint32_t)(lane & (per - 1))) << lb;
  for (int c = 0; c < nch; ++c) {
    const uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane(s_pm[c]);
    const int pb = __builtin_amdgcn_readfirstlane(s_pb[c]);
    if ((pm & lmask) == 0) {
      const double2 v = look(pb + (int)gather_bits(mt, pm));
      eu = fmax(eu, v.x);
      su = fmin(su, v.y);
    } else if ((pm & ~lmask) == 0) {
      const double2 v = look(pb + (int)gather_bits((uint32_t)lane & lmask, pm));
      el = fmax(el, v.x);
      sl = fmin(sl, v.y);
    } else {
      across |= 1u << c;
    }
  }
  // lanes by popcount: level[j] of the lane bits
  const int pcl = __popc((uint32_t)lane);
  const bool valid = (uint32_t)lane <= lmask;
  const int nt = (int)min((uint32_t)per, ntiles - t0);
  for (int i = 0; i < nt; ++i) {
    const uint32_t tile = t0 + i, m = tile << lb | ((uint32_t)lane & lmask);
    MaskScore r;
    r.e = fmax(el, __shfl(eu, i, 64));
    r.slack = fmin(sl, __shfl(su, i, 64));
    for (uint32_t x = across; x; x &= x - 1) {
      const int c = __builtin_ctz(x);
      const uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane(s_pm[c]);
      const double2 v = look(__builtin_amdgcn_readfirstlane(s_pb[c]) + (int)gather_bits(m, pm));
      r.e = fmax(r.e, v.x);
      r.slack = fmin(r.slack, v.y);
    }
    const bool feas = valid && feasible(r, sp.e_bar), near = valid && near_boundary(r, sp.e_bar, sp.amb);
    const int pct = __popc(tile);
    TileRec t;
    t.best = t.near = -1;
    t.emin = INFINITY;
    const unsigned long long fb = __ballot(feas), nb = __ballot(near);
    if (nb)
      for (int j = lb; j >= 0; --j)
        if (nb & __ballot(pcl == j)) {
          t.near = pct + j;
          break;
        }
    if (fb) {
      int j = lb;
      unsigned long long at = 0;
      for (; j >= 0; --j)
        if ((at = fb & __ballot(pcl == j)) != 0) break;
      t.best = pct + j;
      double em = (at >> lane & 1ull) ? r.e : INFINITY;
      if (at & (at - 1)) {
        for (int o = 32; o > 0; o >>= 1) em = fmin(em, __shfl_xor(em, o, 64));
      } else {
        em = __shfl(em, __builtin_ctzll(at), 64);
      }
      t.emin = em;
    }
    if (lane == 0) tiles[tile] = t;
    if (valid && (full_fin || m == 0 || pct + pcl == t.best)) fin[m] = r;
  }
}

// d = |W + S| - |W| in difference form (w = |W| given):
// d = (2 Re(conj(W) S) + |S|^2) / (|W + S| + |W|).  The hardware square root
// and reciprocal (each within 1 ulp) suffice: |W| ~ 1 and |d| <~ 0.05, so
// they add well under 1e-8 absolute to d.
__device__ __forceinline__ float diff32(float2 W, float w, float2 S) {
  const float vx = W.x + S.x, vy = W.y + S.y;
  const float m = __builtin_amdgcn_sqrtf(vx * vx + vy * vy);
  const float num = 2.f * (W.x * S.x + W.y * S.y) + (S.x * S.x + S.y * S.y);
  return num * __builtin_amdgcn_rcpf(m + w);
}

// ---- FP32 screen ----
// The chain patterns again, in FP32 difference form: k_pat32 evaluates every
// pattern's terms per snapshot and folds them into (error, band slack) pairs,
// k_combine32 gives every mask its pair and the tiles their levels.  The terms
// are those of walking each chain for each mask in FP32, so the screen's
// scores are too; walking them took 34 of the 45 ms of the 6000-node search.

// Floats as ints that order alike (the slack can be negative).
__device__ __forceinline__ int float_key(float x) {
  const int i = __float_as_int(x);
  return i < 0 ? i ^ 0x7fffffff : i;
}
__device__ __forceinline__ float key_float(int k) { return __int_as_float(k < 0 ? k ^ 0x7fffffff : k); }

__device__ __forceinline__ Rec32 rec32(const TargetRec& r, double vmin, double vmax, bool on) {
  const double w = sqrt(cabs2(r.W));
  Rec32 o;
  o.W = make_float2((float)r.W.x, (float)r.W.y);
  o.w = (float)w;
  o.a = on ? (float)(w - r.lo) : -INFINITY;
  o.b = on ? (float)(r.hi - w) : -INFINITY;
  o.bmin = on ? (float)(w - vmin) : INFINITY;
  o.bmax = on ? (float)(vmax - w) : INFINITY;
  o.pad = 0.f;
  return o;
}

// A block serves one snapshot (blockIdx.x) of one unit (blockIdx.y, as in
// k_seg_terms): the snapshot's FP32 tables are formed in LDS from the FP64
// ones (rounded once), then every pattern is a thread's.  Zone entries past
// the LDS stage are formed from memory.
__global__ __launch_bounds__(kTermsBlock) void k_pat32(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ units,
    const int* __restrict__ tab, const double2* __restrict__ P, const TargetRec* __restrict__ srec,
    const double2* __restrict__ headV, const TargetRec* __restrict__ zrec, double vmin, double vmax, TermsCaps caps,
    int2* __restrict__ pat32, int* __restrict__ status) {
  extern __shared__ __align__(16) unsigned char ct_lds[];
  const int u = *as_cint(units + blockIdx.y);
  const int uz = u & 255, part = (u >> 8) & 255, parts = u >> 16;
  const int g = *as_cint(segs + uz);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid) return;
  const int tid = threadIdx.x, l = blockIdx.x;
  if (part > 0 && part * kTermsBlock >= H.npat) return;
  if (H.npairs > caps.pairs || H.nslots > caps.slots || H.o_range > caps.ints) {  // never in a consistent plan
    if (tid == 0) atomicOr(status, kStatusBuild);
    return;
  }
  tab = lane_ptr_z(tab, lstride, uz);
  const double2* gP = lane_ptr_z(P, lstride, uz) + (size_t)l * H.npairs * 3;
  const TargetRec* gS = lane_ptr_z(srec, lstride, uz) + (size_t)l * H.nslots * 3;
  const double2* gH = lane_ptr_z(headV, lstride, uz) + (size_t)l * H.nchains * 3;
  const TargetRec* gZ = lane_ptr_z(zrec, lstride, uz) + (size_t)l * H.nz;
  pat32 = lane_ptr_z(pat32, lstride, uz);
  const int zst = min(H.nz, caps.zones);
  int* si = (int*)ct_lds;
  Pair32* sP = (Pair32*)(ct_lds + (size_t)(caps.ints + 3) / 4 * 16);
  Rec32* sS = (Rec32*)(sP + (size_t)caps.pairs * 3);
  Head32* sH = (Head32*)(sS + (size_t)caps.slots * 3);
  Rec32* sZ = (Rec32*)(sH + (size_t)caps.slots * 3);
  for (int i = tid; i < H.o_range; i += kTermsBlock) si[i] = tab[i];  // chains, nesting paths, slots, pairs
  __syncthreads();
  const int nP = H.npairs * 3, nS = H.nslots * 3, nC = H.nchains * 3;
  for (int x = tid; x < nP + nS + nC + zst; x += kTermsBlock) {
    if (x < nP) {
      const int q = x / 3, p = x - q * 3;
      const int rs = si[H.o_pair + q * kPairInts + PR_RSLOT];
      const int* sr = si + H.o_slot + rs * kSlotInts;
      const int c = sr[SL_CHAIN], sx = q - sr[SL_PAIRBASE];  // the super: the chain's head, or its slot sx - 1
      const double2 pv = gP[x];
      const TargetRec r = gS[rs * 3 + p];
      const double2 w = sx == 0 ? gH[c * 3 + p] : gS[(si[c * kChainInts + C_SLOT0] + sx - 1) * 3 + p].W;
      const double ws = sqrt(cabs2(w));
      const bool on = sr[SL_PHASE] >> p & 1;
      Pair32 o;
      o.P = make_float2((float)pv.x, (float)pv.y);
      o.a = on ? (float)(ws - r.lo) : -INFINITY;
      o.b = on ? (float)(r.hi - ws) : -INFINITY;
      sP[x] = o;
    } else if (x < nP + nS) {
      const int y = x - nP, s = y / 3, p = y - s * 3;
      sS[y] = rec32(gS[y], vmin, vmax, si[H.o_slot + s * kSlotInts + SL_PHASE] >> p & 1);
    } else if (x < nP + nS + nC) {
      const double2 v = gH[x - nP - nS];
      Head32 o;
      o.W = make_float2((float)v.x, (float)v.y);
      o.w = (float)sqrt(cabs2(v));
      o.pad = 0.f;
      sH[x - nP - nS] = o;
    } else {
      sZ[x - nP - nS - nC] = rec32(gZ[x - nP - nS - nC], vmin, vmax, true);
    }
  }
  __syncthreads();
  const int* chains = si + H.o_chain;
  const int* nest = si + H.o_nest;
  const int nch = H.nchains;
  int c = 0;  // (a thread's items increase, so its chain index only moves forward)
  for (int it = part * kTermsBlock + tid; it < H.npat; it += parts * kTermsBlock) {
    while (c + 1 < nch && chains[(c + 1) * kChainInts + C_PBASE] <= it) ++c;
    const int* cr = chains + c * kChainInts;
    const uint32_t m = deposit_bits((uint32_t)(it - cr[C_PBASE]), (uint32_t)cr[C_PMASK]);
    float2 S[3];
    float dd[3];  // d of the current super on each phase
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      S[p] = make_float2(0.f, 0.f);
      dd[p] = 0.f;
    }
    float e = 0.f, slack = INFINITY;
    const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
    for (int q = 0; q < nl; ++q) {  // the nesting path down to the head, then the chain itself
      const bool own = q + 1 == nl;
      const int* xr = chains + nest[no + q] * kChainInts;
      if (own && nl > 1) {  // the head is moved by the outer chains
        const int hph = cr[C_PHASE];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const Head32 h = sH[c * 3 + p];
          const float d = diff32(h.W, h.w, S[p]);
          dd[p] = (hph >> p & 1) ? d : 0.f;
        }
      }
      const int ns = xr[C_NSLOT], s0 = xr[C_SLOT0], pair0 = xr[C_PAIR0], bit0 = xr[C_BIT0];
      const int phw0 = xr[C_PHW0], phw1 = xr[C_PHW1], phw2 = xr[C_PHW2];
      int sidx = 0;
      for (int r = 0; r < ns; ++r) {
        const int ph = ((r < 8 ? phw0 : (r < 16 ? phw1 : phw2)) >> (3 * (r & 7))) & 7;
        const bool red = (m >> (bit0 + r)) & 1u;
        const Pair32* pr = sP + (pair0 + ((r * (r + 1)) >> 1) + sidx) * 3;
        const Rec32* tr = sS + (s0 + r) * 3;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const bool on = ph >> p & 1;
          const Pair32 q32 = pr[p];
          S[p].x += red && on ? q32.P.x : 0.f;
          S[p].y += red && on ? q32.P.y : 0.f;
          if (own) {
            const Rec32 t = tr[p];
            const float d = diff32(t.W, t.w, S[p]);
            const float ek = fmaxf(t.a + d, t.b - d), er = fmaxf(q32.a + dd[p], q32.b - dd[p]);
            const float sk = fminf(t.bmin + d, t.bmax - d);
            e = fmaxf(e, on ? (red ? er : ek) : 0.f);
            slack = fminf(slack, on && !red ? sk : INFINITY);
            dd[p] = on && !red ? d : dd[p];
          }
        }
        sidx = red ? sidx : r + 1;
      }
    }
    auto zones = [&](int p, float2 b) {
      int q = cr[C_ZOFF0 + p];
      const int qe = q + cr[C_ZCNT0 + p];
      auto term = [&](const Rec32& t) {
        const float d = diff32(t.W, t.w, b);
        e = fmaxf(e, fmaxf(t.a + d, t.b - d));
        slack = fminf(slack, fminf(t.bmin + d, t.bmax - d));
      };
#pragma unroll 4
      for (const int ql = min(qe, zst); q < ql; ++q) term(sZ[q]);
      for (; q < qe; ++q) term(rec32(gZ[q], vmin, vmax, true));
    };
    zones(0, S[0]);
    zones(1, S[1]);
    zones(2, S[2]);
    atomicMax(&pat32[it].x, __float_as_int(e));  // (e >= 0: its bits order like it)
    atomicMin(&pat32[it].y, float_key(slack));
  }
}

// Every mask's FP32 score from the FP32 pattern table (chains inside, outside
// and across a tile's lane bits as in k_fac_combine), and the tiles' levels of
// surely feasible, possibly feasible and uncertain masks.
__global__ __launch_bounds__(256) void k_combine32(const SegHdr* __restrict__ hdrs, const int* __restrict__ segs,
                                                   size_t lstride, const int* __restrict__ tab,
                                                   const int2* __restrict__ pat32,
                                                   const unsigned long long* __restrict__ ecmax, SelParams sp,
                                                   MaskScore32* __restrict__ fin, TileRec32* __restrict__ tiles,
                                                   int per) {
  __shared__ int s_pm[kMaxK], s_pb[kMaxK];
  __shared__ float2 s_pat[kPatLds];
  const SegHdr H = load_hdr(hdrs, segs);
  if (!H.valid) return;
  const int lb = tile_bits(H.k);
  const uint32_t ntiles = 1u << (H.k - lb);
  if (blockIdx.x * (4 * per) >= ntiles) return;  // past this segment's masks
  tab = lane_ptr(tab, lstride);
  pat32 = lane_ptr(pat32, lstride);
  ecmax = lane_ptr(ecmax, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  const int tid = threadIdx.x, lane = tid & 63;
  const int nch = H.nchains;
  if (tid < nch) {
    s_pm[tid] = tab[H.o_chain + tid * kChainInts + C_PMASK];
    s_pb[tid] = tab[H.o_chain + tid * kChainInts + C_PBASE];
  }
  auto entry = [&](int i) {
    const int2 v = pat32[i];
    return make_float2(__int_as_float(v.x), key_float(v.y));
  };
  for (int i = tid; i < min(H.npat, kPatLds); i += 256) s_pat[i] = entry(i);
  const float ec = (float)__longlong_as_double((long long)*ecmax);
  __syncthreads();
  auto look = [&](int i) { return i < kPatLds ? s_pat[i] : entry(i); };
  const uint32_t t0 = (blockIdx.x * 4 + (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6)) * per;
  if (t0 >= ntiles) return;
  const uint32_t lmask = (1u << lb) - 1u;
  float el = ec, sl = INFINITY;    // chains inside the lane bits, this lane's
  float eu = 0.f, su = INFINITY;   // chains outside, of tile t0 + lane
  uint32_t across = 0;             // chains across
  const uint32_t mt = (t0 + (uint32_t)(lane & (per - 1))) << lb;
  for (int c = 0; c < nch; ++c) {
    const uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane(s_pm[c]);
    const int pb = __builtin_amdgcn_readfirstlane(s_pb[c]);
    if ((pm & lmask) == 0) {
      const float2 v = look(pb + (int)gather_bits(mt, pm));
      eu = fmaxf(eu, v.x);
      su = fminf(su, v.y);
    } else if ((pm & ~lmask) == 0) {
      const float2 v = look(pb + (int)gather_bits((uint32_t)lane & lmask, pm));
      el = fmaxf(el, v.x);
      sl = fminf(sl, v.y);
    } else {
      across |= 1u << c;
    }
  }
  const int pcl = __popc((uint32_t)lane);
  const bool valid = (uint32_t)lane <= lmask;
  const double dlt = sp.delta + sp.amb;
  const int nt = (int)min((uint32_t)per, ntiles - t0);
  for (int i = 0; i < nt; ++i) {
    const uint32_t tile = t0 + i, m = tile << lb | ((uint32_t)lane & lmask);
    MaskScore32 r;
    r.e = fmaxf(el, __shfl(eu, i, 64));
    r.slack = fminf(sl, __shfl(su, i, 64));
    for (uint32_t x = across; x; x &= x - 1) {
      const int c = __builtin_ctz(x);
      const uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane(s_pm[c]);
      const float2 v = look(__builtin_amdgcn_readfirstlane(s_pb[c]) + (int)gather_bits(m, pm));
      r.e = fmaxf(r.e, v.x);
      r.slack = fminf(r.slack, v.y);
    }
    if (valid) fin[m] = r;
    const bool sure = valid && (double)r.e <= sp.e_bar - dlt && (double)r.slack >= dlt;
    const bool poss = valid && (double)r.e <= sp.e_bar + dlt && (double)r.slack >= -dlt;
    const unsigned long long bs = __ballot(sure), bp = __ballot(poss), bu = bp & ~bs;
    TileRec32 t;
    t.sure = t.poss = t.unc = -1;
    t.pad = 0;
    const int pct = __popc(tile);
    if (bp)
      for (int j = lb; j >= 0; --j) {
        const unsigned long long at = __ballot(pcl == j);
        if (t.sure < 0 && (bs & at)) t.sure = pct + j;
        if (t.poss < 0 && (bp & at)) t.poss = pct + j;
        if (t.unc < 0 && (bu & at)) t.unc = pct + j;
      }
    if (lane == 0) tiles[tile] = t;
  }
}

}  // namespace okr
