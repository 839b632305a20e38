// Candidate scoring kernels: every mask of a segment (FP64, and the FP32
// difference-form screen of the mixed-precision search) and FP64 rescoring of
// a mask list.  Built with NaNs excluded (no input or intermediate here is
// NaN), which lets max/min compile to single instructions.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_internal.h"

namespace okr {

// ---------------------------------------------------------------- scoring --
// Tile record of one wave's 64 masks (lane q holds mask
// tile_mask(lanebits, tile, q, k), final score r): highest feasible level,
// smallest error at that level, highest level of a mask near the e_bar /
// band boundary.
__device__ __forceinline__ int tile_record(const MaskScore& r, uint32_t m, uint32_t tile, bool valid,
                                           const SelParams& sp, TileRec* __restrict__ tiles) {
  const int pc = __popc(m);
  const bool feas = valid && feasible(r, sp.e_bar);
  int best = feas ? pc : -1;
  int nearl = (valid && near_boundary(r, sp.e_bar, sp.amb)) ? pc : -1;
  for (int o = 32; o > 0; o >>= 1) {
    best = max(best, __shfl_xor(best, o, 64));
    nearl = max(nearl, __shfl_xor(nearl, o, 64));
  }
  double em = (feas && pc == best) ? r.e : INFINITY;
  for (int o = 32; o > 0; o >>= 1) em = fmin(em, __shfl_xor(em, o, 64));
  if ((threadIdx.x & 63) == 0) {
    TileRec t;
    t.best = best;
    t.near = nearl;
    t.emin = em;
    tiles[tile] = t;
  }
  return best;
}

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
    // members: every node of Omega_g contributes |V^| to the cluster of its
    // current super-node (a slot, a zone target, or a head outside Omega_g,
    // whose error is mask-independent and folds into the constant error)
    const int* rg = tab + H.o_range;
    auto fold = [](TargetRec* r, double v) {
      atomicMin((unsigned long long*)&r->lo, (unsigned long long)__double_as_longlong(v));
      atomicMax((unsigned long long*)&r->hi, (unsigned long long)__double_as_longlong(v));
    };
    for (int q = on ? tid : INT_MAX; q < H.nomega; q += kTermsBlock) {
      int r = 0;
      while (r + 1 < H.nrange && rg[3 * (r + 1) + 2] <= q) ++r;
      const int i = rg[3 * r] + (q - rg[3 * r + 2]);
      const int sp = St.sup[i];
      const unsigned ph = T.phase[i];
      if (T.segment[sp] == g) {
        const int s = St.slot_of[sp];
        if (s < 0 || s >= H.nslots) continue;
#pragma unroll
        for (int p = 0; p < 3; ++p)
          if (ph >> p & 1u) fold(&sS[s * 3 + p], av[(size_t)i * 3 + p]);
      } else {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          if (!(ph >> p & 1u)) continue;
          const double a = av[(size_t)i * 3 + p];
          const int zi = St.zent_of[sp * 3 + p];
          if (zi >= H.nz) continue;
          if (zi >= 0) {
            if (zi < zst) fold(&sZ[zi], a);
            else fold(&gZ[zi], a);
          } else {
            const double2 v = Vl[(size_t)sp * 3 + p];
            atomicMax((unsigned long long*)&s_ec,
                      (unsigned long long)__double_as_longlong(fabs(sqrt(v.x * v.x + v.y * v.y) - a)));
          }
        }
      }
    }
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
// k_build_struct).
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
      const uint32_t mm[1] = {list[q]};
      double el[1] = {ec}, qn[1] = {INFINITY}, qx[1] = {0.0};
      score_chain<true, 1>(chains, nest, c, sP, sS, sH, (const double*)nullptr, sZ, zst, zrec + (size_t)l * H.nz,
                           mm, el, qn, qx);
      unsigned long long* a = s_acc + 3 * (q - q0);
      atomicMax(&a[0], (unsigned long long)__double_as_longlong(el[0]));
      if (qn[0] < INFINITY) atomicMin(&a[1], (unsigned long long)__double_as_longlong(qn[0]));
      if (qx[0] > 0.0) atomicMax(&a[2], (unsigned long long)__double_as_longlong(qx[0]));
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

// Every mask's score from the pattern table (one thread per mask): the
// largest constant error and each chain's entry for the mask's bits, then
// the band slack; per-mask scores and 64-mask tile records as the per-mask
// scoring kernel writes them.
constexpr int kPatLds = 1024;  // pattern-table entries staged in LDS

__global__ __launch_bounds__(256) void k_fac_combine(const SegHdr* __restrict__ hdrs, const int* __restrict__ segs,
                                                     size_t lstride, const int* __restrict__ tab,
                                                     const unsigned long long* __restrict__ pat,
                                                     const unsigned long long* __restrict__ ecmax, SelParams sp,
                                                     MaskScore* __restrict__ fin, TileRec* __restrict__ tiles,
                                                     const int* __restrict__ gates) {
  __shared__ int s_pm[kMaxK], s_pb[kMaxK];
  __shared__ double s_pat[3 * kPatLds];
  const int g = *as_cint(segs + blockIdx.z);
  const SegHdr H = load_hdr_g(hdrs, g);
  if (!H.valid || (gates && gates[g] == 0)) return;
  if ((uint64_t)blockIdx.x * blockDim.x >= ((uint64_t)1 << H.k)) return;  // past this segment's masks
  tab = lane_ptr(tab, lstride);
  pat = lane_ptr(pat, lstride);
  ecmax = lane_ptr(ecmax, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  const int tid = threadIdx.x;
  const int nch = H.nchains;
  if (tid < nch) {
    s_pm[tid] = tab[H.o_chain + tid * kChainInts + C_PMASK];
    s_pb[tid] = tab[H.o_chain + tid * kChainInts + C_PBASE];
  }
  const int np = min(H.npat, kPatLds);
  for (int i = tid; i < 3 * np; i += blockDim.x) s_pat[i] = __longlong_as_double((long long)pat[i]);
  __syncthreads();
  const uint32_t nmask = 1u << H.k;
  const uint32_t L = (uint32_t)H.lanebits;
  const uint32_t tile = (blockIdx.x * blockDim.x + tid) / kScoreBlock;
  const uint32_t m = tile_mask(L, tile, (uint32_t)(tid & (kScoreBlock - 1)), H.k);
  const bool tile_ok = (tile << __popc(L)) < nmask;
  const bool valid = tile_ok && ((uint32_t)(tid & (kScoreBlock - 1)) >> __popc(L)) == 0;
  double e = __longlong_as_double((long long)*ecmax), qn = INFINITY, qx = 0.0;
  for (int c = 0; c < nch; ++c) {
    uint32_t pm = (uint32_t)__builtin_amdgcn_readfirstlane(s_pm[c]);
    const int pb = __builtin_amdgcn_readfirstlane(s_pb[c]);
    uint32_t u = 0;
    int j = 0;
    while (pm) {  // gather the mask's bits at C_PMASK's positions, run by run
      const int b = __builtin_ctz(pm);
      const int run = __builtin_ctz(~(pm >> b));
      const uint32_t ones = (1u << run) - 1u;
      u |= ((m >> b) & ones) << j;
      j += run;
      pm &= ~(ones << b);
    }
    const int idx = pb + (int)u;
    double pe, pn, px;
    if (idx < kPatLds) {
      pe = s_pat[3 * idx];
      pn = s_pat[3 * idx + 1];
      px = s_pat[3 * idx + 2];
    } else {
      pe = __longlong_as_double((long long)pat[3 * idx]);
      pn = __longlong_as_double((long long)pat[3 * idx + 1]);
      px = __longlong_as_double((long long)pat[3 * idx + 2]);
    }
    e = fmax(e, pe);
    qn = fmin(qn, pn);
    qx = fmax(qx, px);
  }
  MaskScore r;
  r.e = e;
  r.slack = band_slack(qn, qx, sp.vmin, sp.vmax);
  if (valid) fin[m] = r;
  if (tile_ok) tile_record(r, m, tile, valid, sp, tiles);
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

// FP32 chain walk for M masks per lane (as walk_chain): d is the difference
// |W + S| - |W| of a slot's voltage; a non-nested head is unaffected (d = 0).
template <bool ERR, int M>
__device__ __forceinline__ void walk32(const int* __restrict__ cr, const Pair32* Ps, const Rec32* Ss,
                                       const Head32* Hs, int c, const uint32_t (&m)[M], float2 (&B)[M][3],
                                       float (&el)[M], float (&slack)[M]) {
  float2 S[M][3];
  float dd[M][3];  // d of the current super on each phase
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      S[i][p] = B[i][p];
      dd[i][p] = 0.f;
    }
  if (ERR && cr[C_OUTER] >= 0) {
    const int hph = cr[C_PHASE];
    const Head32* hv = Hs + c * 3;
#pragma unroll
    for (int p = 0; p < 3; ++p)
      if (hph >> p & 1) {
        const Head32 h = hv[p];
#pragma unroll
        for (int i = 0; i < M; ++i) dd[i][p] = diff32(h.W, h.w, B[i][p]);
      }
  }
  const int ns = cr[C_NSLOT], s0 = cr[C_SLOT0], pair0 = cr[C_PAIR0], bit0 = cr[C_BIT0];
  const int phw0 = cr[C_PHW0], phw1 = cr[C_PHW1], phw2 = cr[C_PHW2];
  int sidx[M];
#pragma unroll
  for (int i = 0; i < M; ++i) sidx[i] = 0;
  for (int r = 0; r < ns; ++r) {
    const int w = r < 8 ? phw0 : (r < 16 ? phw1 : phw2);
    const int ph = (w >> (3 * (r & 7))) & 7;
    const int prow = pair0 + ((r * (r + 1)) >> 1);
    const Rec32* tr = Ss + (s0 + r) * 3;
    bool red[M];
    float rf[M];
    const Pair32* pp[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
      red[i] = (m[i] >> (bit0 + r)) & 1u;
      rf[i] = red[i] ? 1.f : 0.f;
      pp[i] = Ps + (prow + sidx[i]) * 3;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (!(ph >> p & 1)) continue;
      Rec32 t;
      if (ERR) t = tr[p];
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const Pair32 q = pp[i][p];
        S[i][p].x = fmaf(rf[i], q.P.x, S[i][p].x);
        S[i][p].y = fmaf(rf[i], q.P.y, S[i][p].y);
        if (ERR) {
          const float d = diff32(t.W, t.w, S[i][p]);
          const float ek = fmaxf(t.a + d, t.b - d);
          const float er = fmaxf(q.a + dd[i][p], q.b - dd[i][p]);
          el[i] = fmaxf(el[i], red[i] ? er : ek);
          slack[i] = red[i] ? slack[i] : fminf(slack[i], fminf(t.bmin + d, t.bmax - d));
          dd[i][p] = red[i] ? dd[i][p] : d;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < M; ++i) sidx[i] = red[i] ? sidx[i] : r + 1;
  }
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int p = 0; p < 3; ++p) B[i][p] = S[i][p];
}

// FP32 screen of every mask (M masks per lane, layout as in k_score_fp64):
// tile records of sure / possible / uncertain feasibility.
template <int M>
__global__ __launch_bounds__(kScoreThreads) void k_score_fp32(
    const SegHdr* __restrict__ hdrs, const int* __restrict__ segs, size_t lstride, const int* __restrict__ tab,
    const Pair32* __restrict__ P32, const Rec32* __restrict__ S32, const Head32* __restrict__ H32,
    const Rec32* __restrict__ Z32, const double* __restrict__ econst, int snaps_per_group, int SG, SelParams sp,
    MaskScore32* __restrict__ part, MaskScore32* __restrict__ fin, TileRec32* __restrict__ tiles,
    int* __restrict__ tickets) {
  __shared__ Pair32 Ps[kMaxPairs * 3];
  __shared__ Rec32 Ts[kMaxK * 3];
  __shared__ Head32 Hv[kMaxK * 3];
  __shared__ Rec32 Zs[kZoneLds];
  __shared__ double s_ec;
  __shared__ int ticket;
  const SegHdr H = load_hdr(hdrs, segs);
  if (!H.valid) return;
  // blocks past this segment's masks (a chunk's launch covers its largest segment)
  if ((uint64_t)blockIdx.x * (kScoreThreads * M) >= ((uint64_t)1 << H.k)) return;
  tab = lane_ptr(tab, lstride);
  P32 = lane_ptr(P32, lstride);
  S32 = lane_ptr(S32, lstride);
  H32 = lane_ptr(H32, lstride);
  Z32 = lane_ptr(Z32, lstride);
  econst = lane_ptr(econst, lstride);
  part = lane_ptr(part, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  tickets = lane_ptr(tickets, lstride);
  const int tid = threadIdx.x;
  // lane set i of the block: tile x[i] / 64 (tile_mask over the segment's lane bits)
  const uint32_t L = (uint32_t)H.lanebits;
  uint32_t x[M], m[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    x[i] = blockIdx.x * (kScoreThreads * M) + i * kScoreThreads + tid;
    m[i] = tile_mask(L, x[i] / kScoreBlock, x[i] % kScoreBlock, H.k);
  }
  const int sg = blockIdx.y;
  const int l0 = sg * snaps_per_group;
  const int l1 = min(H.S, l0 + snaps_per_group);
  const int* chains = tab + H.o_chain;
  const int* nest = tab + H.o_nest;
  const Stage z = stage_sizes(H);
  float e[M], slack[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    e[i] = 0.f;
    slack[i] = INFINITY;
  }
  for (int l = l0; l < l1; ++l) {
    {
      const uint4* P_l = (const uint4*)(P32 + (size_t)l * H.npairs * 3);
      const uint4* S_l = (const uint4*)(S32 + (size_t)l * H.nslots * 3);
      const uint4* H_l = (const uint4*)(H32 + (size_t)l * H.nchains * 3);
      const uint4* Z_l = (const uint4*)(Z32 + (size_t)l * H.nz);
      for (int i = tid; i < z.total; i += kScoreThreads)
        stage_put(z, i, stage_src(z, i, P_l, S_l, H_l, Z_l), (uint4*)Ps, (uint4*)Ts, (uint4*)Hv, (double*)nullptr,
                  (uint4*)Zs);
      if (tid == 0) s_ec = econst[l];
      __syncthreads();
    }
    const Rec32* Zl = Z32 + (size_t)l * H.nz;
    float el[M];
    const float ec = (float)s_ec;
#pragma unroll
    for (int i = 0; i < M; ++i) el[i] = ec;
    for (int c = 0; c < H.nchains; ++c) {
      const int* cr = chains + c * kChainInts;
      if (!(cr[C_PMASK] & L)) continue;  // the same for the wave's lanes: below
      float2 B[M][3];
#pragma unroll
      for (int i = 0; i < M; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p) B[i][p] = make_float2(0.f, 0.f);
      const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
      for (int q = 0; q + 1 < nl; ++q) {
        const int oc = nest[no + q];
        walk32<false, M>(chains + oc * kChainInts, Ps, Ts, Hv, oc, m, B, el, slack);
      }
      walk32<true, M>(cr, Ps, Ts, Hv, c, m, B, el, slack);
#pragma unroll
      for (int p = 0; p < 3; ++p)
        for (int q = cr[C_ZOFF0 + p], qe = q + cr[C_ZCNT0 + p]; q < qe; ++q) {
          Rec32 t;
          if (q < kZoneLds) t = Zs[q];
          else t = Zl[q];
#pragma unroll
          for (int i = 0; i < M; ++i) {
            const float d = diff32(t.W, t.w, B[i][p]);
            el[i] = fmaxf(el[i], fmaxf(t.a + d, t.b - d));
            slack[i] = fminf(slack[i], fminf(t.bmin + d, t.bmax - d));
          }
        }
    }
#pragma unroll
    for (int i = 0; i < M; ++i) e[i] = fmaxf(e[i], el[i]);
    __syncthreads();
  }
  // Chains none of whose bits is among the lane bits (the 6 that vary across
  // a wave's lanes) have the same terms for the wave's 64 masks of each of
  // its M mask sets:
  // evaluated once per wave and mask set, one snapshot per lane, from the
  // tables in global memory, folded across the lanes.
  {
    const int lane = tid & 63;
    for (int c = 0; c < H.nchains; ++c) {
      const int* cr = chains + c * kChainInts;
      if (cr[C_PMASK] & L) continue;
      const int nl = cr[C_NEST_LEN], no = cr[C_NEST_OFF];
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const uint32_t mi[1] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)m[i])};
        float ue = 0.f, us = INFINITY;
        for (int l = l0 + lane; l < l1; l += 64) {
          const Pair32* P_l = P32 + (size_t)l * H.npairs * 3;
          const Rec32* S_l = S32 + (size_t)l * H.nslots * 3;
          const Head32* H_l = H32 + (size_t)l * H.nchains * 3;
          const Rec32* Z_l = Z32 + (size_t)l * H.nz;
          float2 B[1][3];
#pragma unroll
          for (int p = 0; p < 3; ++p) B[0][p] = make_float2(0.f, 0.f);
          float el1[1] = {0.f}, sl1[1] = {INFINITY};
          for (int q = 0; q + 1 < nl; ++q) {
            const int oc = nest[no + q];
            walk32<false, 1>(chains + oc * kChainInts, P_l, S_l, H_l, oc, mi, B, el1, sl1);
          }
          walk32<true, 1>(cr, P_l, S_l, H_l, c, mi, B, el1, sl1);
#pragma unroll
          for (int p = 0; p < 3; ++p)
            for (int q = cr[C_ZOFF0 + p], qe = q + cr[C_ZCNT0 + p]; q < qe; ++q) {
              const Rec32 t = Z_l[q];
              const float d = diff32(t.W, t.w, B[0][p]);
              el1[0] = fmaxf(el1[0], fmaxf(t.a + d, t.b - d));
              sl1[0] = fminf(sl1[0], fminf(t.bmin + d, t.bmax - d));
            }
          ue = fmaxf(ue, el1[0]);
          us = fminf(us, sl1[0]);
        }
        for (int o = 32; o > 0; o >>= 1) {
          ue = fmaxf(ue, __shfl_xor(ue, o, 64));
          us = fminf(us, __shfl_xor(us, o, 64));
        }
        e[i] = fmaxf(e[i], ue);
        slack[i] = fminf(slack[i], us);
      }
    }
  }
  const uint32_t nmask = 1u << H.k;
#pragma unroll
  for (int i = 0; i < M; ++i)
    if (x[i] < nmask) {
      MaskScore32 r;
      r.e = e[i];
      r.slack = slack[i];
      part[(size_t)sg * nmask + m[i]] = r;
    }
  // every wave's partial scores are written and visible before the block
  // takes its ticket (the last block to take one reads them all)
  __threadfence();
  __syncthreads();
  if (tid == 0) ticket = atomicAdd(&tickets[blockIdx.x], 1);
  __syncthreads();
  if (ticket != SG - 1) return;
  __threadfence();
  const double dlt = sp.delta + sp.amb;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const bool valid = x[i] < nmask;
    MaskScore32 r;
    r.e = 0.f;
    r.slack = INFINITY;
    if (valid) {
      for (int q = 0; q < SG; ++q) {
        const volatile MaskScore32* x = part + (size_t)q * nmask + m[i];
        r.e = fmaxf(r.e, x->e);
        r.slack = fminf(r.slack, x->slack);
      }
      fin[m[i]] = r;
    }
    const bool sure = valid && (double)r.e <= sp.e_bar - dlt && (double)r.slack >= dlt;
    const bool poss = valid && (double)r.e <= sp.e_bar + dlt && (double)r.slack >= -dlt;
    const int pc = __popc(m[i]);
    int a = sure ? pc : -1, b = poss ? pc : -1, c = (poss && !sure) ? pc : -1;
    for (int o = 32; o > 0; o >>= 1) {
      a = max(a, __shfl_xor(a, o, 64));
      b = max(b, __shfl_xor(b, o, 64));
      c = max(c, __shfl_xor(c, o, 64));
    }
    const uint32_t tile = x[i] / kScoreBlock;
    if ((tid & 63) == 0 && tile * kScoreBlock < nmask) {
      TileRec32 t;
      t.sure = a;
      t.poss = b;
      t.unc = c;
      t.pad = 0;
      tiles[tile] = t;
    }
  }
  if (tid == 0) tickets[blockIdx.x] = 0;
}

#define OKR_SCORE32_INST(M_)                                                                                   \
  template __global__ void k_score_fp32<M_>(const SegHdr*, const int*, size_t, const int*, const Pair32*, const Rec32*,       \
                                            const Head32*, const Rec32*, const double*, int, int, SelParams,  \
                                            MaskScore32*, MaskScore32*, TileRec32*, int*);
OKR_SCORE32_INST(1)
OKR_SCORE32_INST(2)
OKR_SCORE32_INST(4)
#undef OKR_SCORE32_INST

}  // namespace okr
