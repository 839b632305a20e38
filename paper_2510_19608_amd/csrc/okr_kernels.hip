// gfx950 kernels of the segment-exhaustive Kron-reduction search.
//
// Data layout in HBM (complex values as double2 = (re, im)):
//   z[n][9]            branch impedance of node i's upstream edge (restricted)
//   Vhat               [S][n][3]: scenario voltages by the caller's node ids
//   Vcur, A            [S][n][3] by label (DFS preorder position): current
//                      candidate-state voltages of kept nodes, aggregated load
//                      current of kept nodes (consumed current, = -I^ moved by
//                      the assignment); every other per-node array goes by
//                      label too
//   absV[S][n][3]      |Vhat|
//   per segment        P[S][npairs][3], slot/zone TargetRec[S][..][3], headV
//   scores             MaskScore[2^k]
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_flow.h"
#include "okr_internal.h"
#include "okr_kron.h"

namespace okr {

// Largest |A_q| (one square root: it is monotone).
__device__ __forceinline__ double blk_maxabs(const double2* A) {
  double mx = 0.0;
  for (int q = 0; q < 9; ++q) mx = fmax(mx, cabs2(A[q]));
  return sqrt(mx);
}

// ---------------------------------------------------------- validation + z --
// Branch impedances z_i = (-Y_{i,parent})^+ and checks of the admittance input
// (symmetry, zero absent-phase entries, no shunts).  ext maps the labels of the
// tree arrays and z to the input's node ids.  With a search state it also resets
// every node's (kept and its own super-node, the maps empty).
// status bits: 1 singular, 2 absent-phase entry, 4 asymmetric, 8 shunt.
// The first nz blocks take a node per thread (inverse, symmetry, reset), the
// others the row sums, 16 lanes per node (9 entries; the children's ids loaded
// by a lane each).  Bound by latency; the comparisons take one square root each,
// of the largest square.  1000 nodes 8.7 us, 30 nodes 6.0 (14.3 and 8.8 with both
// in one thread, the children's blocks one after the other).
__global__ __launch_bounds__(64) void k_branch_z(int n, int nz, const uint8_t* __restrict__ phase,
                                                 const int* __restrict__ ch_off, const int* __restrict__ ch,
                                                 const int* __restrict__ ext, const double2* __restrict__ Ydiag,
                                                 const double2* __restrict__ Yoff, double2* __restrict__ z,
                                                 int* __restrict__ status, State St) {
  const int tid = threadIdx.x;
  int bad = 0;
  if ((int)blockIdx.x < nz) {
    const int i = blockIdx.x * 64 + tid;
    if (i >= n) return;
    if (St.kept) {
      St.kept[i] = 1;
      St.sup[i] = i;
      St.slot_of[i] = -1;
      for (int p = 0; p < 3; ++p) St.zent_of[i * 3 + p] = -1;
    }
    if (i == 0) {
      for (int q = 0; q < 9; ++q) z[q] = make_double2(0.0, 0.0);
      return;
    }
    const unsigned ph = phase[i];
    const double2* Yo = Yoff + (size_t)ext[i] * 9;
    const double oscale = blk_maxabs(Yo);
    double asym = 0.0;
    double2 y[9];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        asym = fmax(asym, cabs2(csub(Yo[r * 3 + c], Yo[c * 3 + r])));
        const bool absent = !((ph >> r) & 1u) || !((ph >> c) & 1u);
        if (absent && cabs2(Yo[r * 3 + c]) != 0.0) bad |= 2;
        y[r * 3 + c] = make_double2(-Yo[r * 3 + c].x, -Yo[r * 3 + c].y);
      }
    if (sqrt(asym) > 1e-12 * oscale) bad |= 4;
    if (!inv_restricted(y, ph, z + (size_t)i * 9)) bad |= 1;
  } else {
    // Laplacian row: Y_ii + Y_{i,p} + sum_c Y_{i,c} = 0, with Y_{i,c} = Y_{c,i}^T
    const int i = ((int)blockIdx.x - nz) * 4 + (tid >> 4), k = tid & 15;
    const bool in = i < n, on = in && k < 9;
    const int r = k / 3, c = k - 3 * r;
    const int x = in ? ext[i] : 0, e0 = in ? ch_off[i] : 0, nc = in ? ch_off[i + 1] - e0 : 0;
    const unsigned ph = in ? phase[i] : 0u;
    double2 acc = make_double2(0.0, 0.0);
    if (on) acc = Ydiag[(size_t)x * 9 + k];
    double dmax = cabs2(acc);
    const bool absent = !((ph >> r) & 1u) || !((ph >> c) & 1u);
    if (on && absent && dmax != 0.0) bad |= 2;
    if (on && i > 0) acc = cadd(acc, Yoff[(size_t)x * 9 + k]);
    for (int b = 0; __ballot(b < nc); b += 16) {
      const int id = b + k < nc ? ext[ch[e0 + b + k]] : 0;
      for (int j = 0; j < 16 && __ballot(b + j < nc); ++j) {
        const int y = __shfl(id, (tid & 48) + j, 64);
        if (on && b + j < nc) acc = cadd(acc, Yoff[(size_t)y * 9 + c * 3 + r]);
      }
    }
    double amax = cabs2(acc);
    for (int o = 8; o > 0; o >>= 1) {
      dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
      amax = fmax(amax, __shfl_xor(amax, o, 64));
    }
    if (on && k == 0 && sqrt(amax) > 1e-9 * fmax(sqrt(dmax), 1e-300)) bad |= 8;
  }
  if (bad) atomicOr(status, bad);
}

// ------------------------------------------------------------- load flow --
// Scenario library (Section III): constant-PQ wye loads, backward/forward
// sweep on the radial tree, one block per snapshot, level-synchronous.
// status bit 16: not converged; bit 32: base network outside the band.
// The tree arrays, V, J, A and absV go by label, Sload by the caller's node
// ids (ext[label]); Vext, where given, takes the voltages by the caller's ids.
// Forward-sweep update of node i: V(i) = V(parent) - z(i) J(i) on its
// present phases, and the largest change into dmax (NaN-propagating).
__device__ __forceinline__ void forward_node(int i, const int* __restrict__ parent, const uint8_t* __restrict__ phase,
                                             const double2 (&zi)[9], const double2* Jl, double2* Vl, double& dmax) {
  const int pv = parent[i];
  const double2 j0 = Jl[i * 3], j1 = Jl[i * 3 + 1], j2 = Jl[i * 3 + 2];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (!(phase[i] >> p & 1u)) continue;
    const double2 d = cadd(cadd(cmul(zi[p * 3], j0), cmul(zi[p * 3 + 1], j1)), cmul(zi[p * 3 + 2], j2));
    const double2 nv = csub(Vl[pv * 3 + p], d);
    const double dd = sqrt(cabs2(csub(nv, Vl[i * 3 + p])));
    dmax = nan_max(dmax, dd);
    Vl[i * 3 + p] = nv;
  }
}

// Level by level from global memory, for feeders beyond the other forms.
__global__ __launch_bounds__(256) void k_powerflow(
    int n, const int* __restrict__ parent, const uint8_t* __restrict__ phase,
    const int* __restrict__ lvl_off, const int* __restrict__ lvl_nodes, int nlev,
    const int* __restrict__ ch_off, const int* __restrict__ ch, const double2* __restrict__ z,
    const double2* __restrict__ Sload, double2 v0a, double2 v0b, double2 v0c, double tol, int maxit,
    double vmin, double vmax, double2* __restrict__ V, double2* __restrict__ J,
    double2* __restrict__ A, double* __restrict__ absV, int* __restrict__ iters, int* __restrict__ status,
    const int* __restrict__ ext, double2* __restrict__ Vext) {
  __shared__ double shd[16];
  const int l = blockIdx.x;
  const size_t base = (size_t)l * n * 3;
  double2* Vl = V + base;
  double2* Jl = J + base;
  const double2* Sl = Sload + base;
  const double2 v0[3] = {v0a, v0b, v0c};
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    for (int p = 0; p < 3; ++p) Vl[i * 3 + p] = (phase[i] >> p & 1u) ? v0[p] : make_double2(0.0, 0.0);
  __syncthreads();
  int it = 0;
  bool conv = false;
  const int tid = threadIdx.x, bd = blockDim.x;
  for (it = 1; it <= maxit; ++it) {
    // load currents conj(S/V) of every node in one pass (off the level
    // steps' latency chain), then the backward sweep adds each level's
    // children into their parents, deepest level first
    for (int i = tid; i < n; i += bd) {
      const int x = ext[i];
      for (int p = 0; p < 3; ++p)
        Jl[i * 3 + p] = (i > 0 && (phase[i] >> p & 1u)) ? cconj(cdiv(Sl[x * 3 + p], Vl[i * 3 + p]))
                                                        : make_double2(0.0, 0.0);
    }
    __syncthreads();
    for (int lev = nlev - 2; lev >= 0; --lev) {
      for (int q = lvl_off[lev] + tid; q < lvl_off[lev + 1]; q += bd) {
        const int i = lvl_nodes[q];
        double2 s0 = Jl[i * 3], s1 = Jl[i * 3 + 1], s2 = Jl[i * 3 + 2];
        for (int e = ch_off[i]; e < ch_off[i + 1]; ++e) {
          const int c = ch[e];
          s0 = cadd(s0, Jl[c * 3]);
          s1 = cadd(s1, Jl[c * 3 + 1]);
          s2 = cadd(s2, Jl[c * 3 + 2]);
        }
        Jl[i * 3] = s0; Jl[i * 3 + 1] = s1; Jl[i * 3 + 2] = s2;
      }
      __syncthreads();
    }
    double dmax = 0.0;
    // the branch impedance of this thread's first node on the next level is
    // loaded while the current level is computed (the impedances are the
    // only global reads of the sweep; a thread with no node there loads the
    // root's, unused)
    double2 zn[9];
    {
      const int q1 = nlev > 1 ? lvl_off[1] + tid : 0;
      const double2* zz = z + (size_t)((nlev > 1 && q1 < lvl_off[2]) ? lvl_nodes[q1] : 0) * 9;
#pragma unroll
      for (int e = 0; e < 9; ++e) zn[e] = zz[e];
    }
    for (int lev = 1; lev < nlev; ++lev) {
      double2 zc[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) zc[e] = zn[e];
      {
        const int qn = lev + 1 < nlev ? lvl_off[lev + 1] + tid : 0;
        const double2* zz = z + (size_t)((lev + 1 < nlev && qn < lvl_off[lev + 2]) ? lvl_nodes[qn] : 0) * 9;
#pragma unroll
        for (int e = 0; e < 9; ++e) zn[e] = zz[e];
      }
      const int q0 = lvl_off[lev] + tid, q1 = lvl_off[lev + 1];
      if (q0 < q1) forward_node(lvl_nodes[q0], parent, phase, zc, Jl, Vl, dmax);
      for (int q = q0 + bd; q < q1; q += bd) {  // (levels wider than the block)
        const int i = lvl_nodes[q];
        double2 zi[9];
#pragma unroll
        for (int e = 0; e < 9; ++e) zi[e] = z[(size_t)i * 9 + e];
        forward_node(i, parent, phase, zi, Jl, Vl, dmax);
      }
      __syncthreads();
    }
    dmax = block_reduce(dmax, [](double a, double b) { return nan_max(a, b); }, shd);
    if (!(dmax <= 1e3)) break;
    if (dmax <= tol) { conv = true; break; }
  }
  double vlo = 1e300, vhi = -1e300;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int x = ext[i];
    for (int p = 0; p < 3; ++p) {
      const bool pr = (phase[i] >> p & 1u);
      const double2 v = Vl[i * 3 + p];
      if (Vext) Vext[base + x * 3 + p] = v;
      A[base + i * 3 + p] = (i > 0 && pr) ? cconj(cdiv(Sl[x * 3 + p], v)) : make_double2(0.0, 0.0);
      const double m = pr ? sqrt(cabs2(v)) : 0.0;
      absV[base + i * 3 + p] = m;
      if (pr) { vlo = fmin(vlo, m); vhi = fmax(vhi, m); }
    }
  }
  vlo = block_reduce(vlo, [](double a, double b) { return fmin(a, b); }, shd);
  vhi = block_reduce(vhi, [](double a, double b) { return fmax(a, b); }, shd);
  if (threadIdx.x == 0) {
    iters[l] = it;
    if (!conv) atomicOr(status, 16);
    if (vlo < vmin || vhi > vmax) atomicOr(status, 32);
  }
}

// Breadth-first storage, for feeders beyond the prefix sums' LDS (n < 65536): every
// per-node quantity of the sweep is stored by breadth-first queue position
// (each level a contiguous run, the children of position q at positions
// cf[q] .. cf[q+1]-1 in child-list order, pp[q] the parent's position), so
// each level step reads and writes contiguous records and a node's children
// are one contiguous run.  The queue tables (16-bit) sit in dynamic LDS; the
// snapshot's loads and voltages in queue order use the V and A slices as
// scratch until the end, the branch currents the J slice.  Each node's
// arithmetic, and the order of every sum, is that of the node-order form.
__global__ __launch_bounds__(512) void k_powerflow_bfs(
    int n, const uint8_t* __restrict__ phase, const int* __restrict__ glvl_off, const int* __restrict__ glvl_nodes,
    int nlev, const int* __restrict__ gcf, const int* __restrict__ gpp, const double2* __restrict__ z,
    const double2* __restrict__ Sload, double2 v0a, double2 v0b, double2 v0c, double tol, int maxit,
    double vmin, double vmax, double2* __restrict__ V, double2* __restrict__ J,
    double2* __restrict__ A, double* __restrict__ absV, int* __restrict__ iters, int* __restrict__ status,
    const int* __restrict__ ext, double2* __restrict__ Vext) {
  extern __shared__ double2 pf_lds[];
  __shared__ double shd[16];
  const int l = blockIdx.x, tid = threadIdx.x, bd = blockDim.x;
  const size_t base = (size_t)l * n * 3;
  int* lvl_off = (int*)pf_lds;
  uint16_t* node = (uint16_t*)(lvl_off + nlev + 1);
  uint16_t* cf = node + n;
  uint16_t* pp = cf + n + 1;
  uint8_t* ph = (uint8_t*)(pp + n);
  for (int i = tid; i <= nlev; i += bd) lvl_off[i] = glvl_off[i];
  for (int q = tid; q <= n; q += bd) cf[q] = (uint16_t)gcf[q];
  for (int q = tid; q < n; q += bd) {
    const int i = glvl_nodes[q];
    node[q] = (uint16_t)i;
    pp[q] = (uint16_t)gpp[q];
    ph[q] = phase[i];
  }
  const double2* Sl = Sload + base;
  double2* Sb = V + base;
  double2* Vb = A + base;
  double2* Jb = J + base;
  __syncthreads();
  const double2 v0[3] = {v0a, v0b, v0c};
  for (int q = tid; q < n; q += bd) {
    const int x = ext[node[q]];
    const unsigned m = ph[q];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      Sb[q * 3 + p] = Sl[x * 3 + p];
      Vb[q * 3 + p] = (m >> p & 1u) ? v0[p] : make_double2(0.0, 0.0);
    }
  }
  __syncthreads();
  int it = 0;
  bool conv = false;
  for (it = 1; it <= maxit; ++it) {
    // backward sweep, deepest level first: branch current = own load
    // current conj(S/V) on present phases + the children's branch currents
    // (finished on the previous step), added in child order after all of
    // them are loaded; the root's is never read and is not formed
    for (int lev = nlev - 1; lev >= 1; --lev) {
      for (int q = lvl_off[lev] + tid; q < lvl_off[lev + 1]; q += bd) {
        const unsigned m = ph[q];
        const int c0 = cf[q], c1 = cf[q + 1];
        double2 s[3], v[3], a[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) { s[p] = Sb[q * 3 + p]; v[p] = Vb[q * 3 + p]; }
        for (int c = c0; c < c1; c += 2) {
          double2 t0[3], t1[3];
          const int cc = c + 1 < c1 ? c + 1 : c;
#pragma unroll
          for (int p = 0; p < 3; ++p) { t0[p] = Jb[c * 3 + p]; t1[p] = Jb[cc * 3 + p]; }
          if (c == c0) {
#pragma unroll
            for (int p = 0; p < 3; ++p) a[p] = (m >> p & 1u) ? cconj(cdiv(s[p], v[p])) : make_double2(0.0, 0.0);
          }
#pragma unroll
          for (int p = 0; p < 3; ++p) a[p] = cadd(a[p], t0[p]);
          if (c + 1 < c1) {
#pragma unroll
            for (int p = 0; p < 3; ++p) a[p] = cadd(a[p], t1[p]);
          }
        }
        if (c0 == c1) {
#pragma unroll
          for (int p = 0; p < 3; ++p) a[p] = (m >> p & 1u) ? cconj(cdiv(s[p], v[p])) : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) Jb[q * 3 + p] = a[p];
      }
      __syncthreads();
    }
    // forward sweep: V(q) = V(parent) - z J(q) on present phases, the
    // largest change into dmax (NaN-propagating)
    double dmax = 0.0;
    for (int lev = 1; lev < nlev; ++lev) {
      for (int q = lvl_off[lev] + tid; q < lvl_off[lev + 1]; q += bd) {
        const int i = node[q], pq = pp[q];
        const unsigned m = ph[q];
        double2 zi[9], j[3], vp[3], vo[3];
#pragma unroll
        for (int e = 0; e < 9; ++e) zi[e] = z[(size_t)i * 9 + e];
#pragma unroll
        for (int p = 0; p < 3; ++p) { j[p] = Jb[q * 3 + p]; vp[p] = Vb[pq * 3 + p]; vo[p] = Vb[q * 3 + p]; }
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          if (!(m >> p & 1u)) continue;
          const double2 d = cadd(cadd(cmul(zi[p * 3], j[0]), cmul(zi[p * 3 + 1], j[1])), cmul(zi[p * 3 + 2], j[2]));
          const double2 nv = csub(vp[p], d);
          const double dd = sqrt(cabs2(csub(nv, vo[p])));
          dmax = nan_max(dmax, dd);
          Vb[q * 3 + p] = nv;
        }
      }
      __syncthreads();
    }
    dmax = block_reduce(dmax, [](double a, double b) { return nan_max(a, b); }, shd);
    if (!(dmax <= 1e3)) break;
    if (dmax <= tol) { conv = true; break; }
  }
  // voltages back to label order (over the loads, no longer read), then the
  // load currents and magnitudes at the final voltages
  for (int q = tid; q < n; q += bd) {
    const int i = node[q];
#pragma unroll
    for (int p = 0; p < 3; ++p) V[base + i * 3 + p] = Vb[q * 3 + p];
  }
  __syncthreads();
  double vlo = 1e300, vhi = -1e300;
  for (int i = tid; i < n; i += bd) {
    const int x = ext[i];
    for (int p = 0; p < 3; ++p) {
      const bool pr = (phase[i] >> p & 1u);
      const double2 v = V[base + i * 3 + p];
      Vext[base + x * 3 + p] = v;
      A[base + i * 3 + p] = (i > 0 && pr) ? cconj(cdiv(Sl[x * 3 + p], v)) : make_double2(0.0, 0.0);
      const double m = pr ? sqrt(cabs2(v)) : 0.0;
      absV[base + i * 3 + p] = m;
      if (pr) { vlo = fmin(vlo, m); vhi = fmax(vhi, m); }
    }
  }
  vlo = block_reduce(vlo, [](double a, double b) { return fmin(a, b); }, shd);
  vhi = block_reduce(vhi, [](double a, double b) { return fmax(a, b); }, shd);
  if (tid == 0) {
    iters[l] = it;
    if (!conv) atomicOr(status, 16);
    if (vlo < vmin || vhi > vmax) atomicOr(status, 32);
  }
}

// Cumulative impedances by a launch of their own (one block; see zroot_block).
__global__ __launch_bounds__(1024) void k_zroot(int n, const int* __restrict__ parent,
                                                const int* __restrict__ lvl_off, const int* __restrict__ lvl_nodes,
                                                int nlev, const double2* __restrict__ z, double2* __restrict__ Zroot) {
  zroot_block(n, parent, lvl_off, lvl_nodes, nlev, z, Zroot);
}

// Given V^ (caller supplied, by the caller's node ids ext[label]): load currents
// and magnitudes, band check; with Vlab the voltages by label too.
__global__ void k_from_vhat(int n, int S, const uint8_t* __restrict__ phase, const double2* __restrict__ Sload,
                            const double2* __restrict__ V, double vmin, double vmax, double2* __restrict__ A,
                            double* __restrict__ absV, int* __restrict__ status, const int* __restrict__ ext,
                            double2* __restrict__ Vlab) {
  const size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= (size_t)S * n * 3) return;
  const int p = q % 3, i = (q / 3) % n;
  const size_t x = q + ((long)ext[i] - i) * 3;
  const bool pr = (phase[i] >> p & 1u);
  const double2 v = V[x];
  if (Vlab) Vlab[q] = v;
  A[q] = (i > 0 && pr) ? cconj(cdiv(Sload[x], v)) : make_double2(0.0, 0.0);
  const double m = pr ? sqrt(cabs2(v)) : 0.0;
  absV[q] = m;
  if (pr && (m < vmin || m > vmax)) atomicOr(status, 32);
}

// ----------------------------------------------------------------- argmin --
// Lexicographic selection over the tile records: most reduced nodes among
// feasible masks, then the smallest error, masks within tie_tol of that error
// tie and the lowest wins.  Only tiles whose record can hold the winner (or a
// mask within amb of the tie threshold) are rescanned mask by mask.
// Ambiguous when a mask at the chosen level or above lies within amb of the
// e_bar / band boundary, or a feasible mask at the chosen level lies within
// amb of e_min + tie_tol.  With tab the decision is final and the state's
// structure is updated.  With slist (SMICE as the key) it also lists mask 0
// and then every feasible mask of the chosen level, in any order (the listed
// masks are a few hundred of 65,536 on the 1000-node workload; scoring them
// from a dense list keeps every lane busy).
// One block per segment, bound by latency: the tile records in one round of
// loads, level and error in one reduction, what the state update reads loaded
// before the decision.  Per chunk 8.3 us at 1000 nodes (10.2 with the records
// read in three rounds of 1024 and the update's loads after the decision), 8.4
// at 6000 (11.9), 9.5 at 8400 (19.8).
__global__ __launch_bounds__(1024) void k_argmin(const SegHdr* __restrict__ hdrs, const int* __restrict__ segs,
                                                 size_t lstride, const MaskScore* __restrict__ fin,
                                                 const TileRec* __restrict__ tiles, SelParams sp,
                                                 const int* __restrict__ status, DevDecision* __restrict__ decs,
                                                 const int* __restrict__ gates, uint32_t* __restrict__ slist,
                                                 int* __restrict__ scount, const int* __restrict__ tab, Topo T,
                                                 State St, SmicePrep pp) {
  // one slot per wave for each reduction (each its own array, so no
  // reduction's slots are written while another's are still being read)
  __shared__ int s_best[16], s_near[16], s_amb[16];
  __shared__ double s_emin[16], s_run[16];
  __shared__ unsigned s_pick[16];
  __shared__ int ncand, nlist;
  __shared__ int cand[1024];
  __shared__ StateUpdate su;
  const int g = segs[blockIdx.z];
  const SegHdr H = load_hdr_g(hdrs, g);
  if (blockIdx.x == 1) {  // (SMICE as the key: the segment's tables for it)
    smice_prep(H, lane_ptr(pp.tab, lstride), T, St, lane_ptr(pp.stab, lstride));
    return;
  }
  if (blockIdx.x > 1) {  // (the fixed errors of its heads, a snapshot per block)
    smice_hconst(H, lane_ptr(pp.tab, lstride), T, St, pp.Vcur, pp.absV, lane_ptr(pp.hK, lstride), pp.S,
                 (int)blockIdx.x - 2);
    return;
  }
  tab = lane_ptr(tab, lstride);
  const int tid = threadIdx.x, bd = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = bd >> 6;
  const bool upd = tab && H.valid;
  int ui = -1, us = -1, uj = -1;
  if (gates && gates[g] == 0) {  // decided without the full enumeration
    if (upd) {
      su.load(H, tab, T, St, ui, us, uj);
      __syncthreads();
      su.store(H, tab, St, decs[g].mask, ui, us, uj);
    }
    return;
  }
  slist = lane_ptr(slist, lstride);
  scount = lane_ptr(scount, lstride);
  fin = lane_ptr(fin, lstride);
  tiles = lane_ptr(tiles, lstride);
  DevDecision* dec = decs + g;
  // nothing is reduced when the full network violates the band, the load
  // flow failed, or the segment's tables are inconsistent
  if (!H.valid || (*status & (16 | 32))) {
    if (upd) {
      su.load(H, tab, T, St, ui, us, uj);
      __syncthreads();
      su.store(H, tab, St, 0u, ui, us, uj);
    }
    if (tid == 0) {
      DevDecision d;
      d.mask = 0; d.popcount = 0; d.e_loc = 0.0; d.e_min = 0.0; d.ambiguous = 0; d.found = 0;
      d.key_gap = INFINITY;
      d.smice_rise = 0.0;
      *dec = d;
      if (slist) *scount = 0;
    }
    return;
  }
  const int k = H.k;
  const uint32_t nm = 1u << k;
  const int lb = tile_bits(k);
  const int ntiles = (int)(nm >> lb);
  // the first kTileRegs tiles of each thread (all of them for segments of up
  // to 20 nodes) are read once, together, and kept in registers
  constexpr int kTileRegs = 16;
  TileRec rt[kTileRegs];
#pragma unroll
  for (int u = 0; u < kTileRegs; ++u) {
    if (u * bd >= ntiles) break;
    if (tid + u * bd < ntiles) rt[u] = tiles[tid + u * bd];
    else rt[u] = TileRec{-1, -1, INFINITY};
  }
  auto each_tile = [&](auto f) {
#pragma unroll
    for (int u = 0; u < kTileRegs; ++u) {
      if (u * bd >= ntiles) break;
      if (tid + u * bd < ntiles) f(rt[u], tid + u * bd);
    }
    for (int t = tid + kTileRegs * bd; t < ntiles; t += bd) f(tiles[t], t);
  };
  if (tid == 0) ncand = 0;
  // the best level, the smallest error there, and the best level near the boundary
  int best = -1, near = -1;
  double emin = INFINITY;
  auto join = [&](int b, double e, int c) {
    emin = b > best ? e : b == best ? fmin(emin, e) : emin;
    best = max(best, b);
    near = max(near, c);
  };
  each_tile([&](const TileRec& r, int) { join(r.best, r.emin, r.near); });
  for (int o = 32; o > 0; o >>= 1) join(__shfl_xor(best, o, 64), __shfl_xor(emin, o, 64), __shfl_xor(near, o, 64));
  if (lane == 0) {
    s_best[wv] = best;
    s_emin[wv] = emin;
    s_near[wv] = near;
  }
  if (upd) su.load(H, tab, T, St, ui, us, uj);
  __syncthreads();
  {
    const int w = lane & (nw - 1);
    best = s_best[w];
    emin = s_emin[w];
    near = s_near[w];
    for (int o = nw / 2; o > 0; o >>= 1)
      join(__shfl_xor(best, o, 64), __shfl_xor(emin, o, 64), __shfl_xor(near, o, 64));
  }
  int amb = best >= 0 && near >= best;
  unsigned pick = 0xffffffffu;
  const double thr = emin + sp.tie;
  // runner-up: the smallest error above the tie window at the chosen level
  // (a tile not rescanned holds it at its own minimum)
  double runner = INFINITY;
  auto rescan = [&](int nc) {
    for (int q = tid; q < nc * 64; q += bd) {
      if ((q & 63) >> lb) continue;
      const uint32_t mm = (uint32_t)cand[q >> 6] << lb | (uint32_t)(q & 63);
      if (__popc(mm) != best) continue;  // (only these masks' scores are stored)
      const MaskScore r = fin[mm];
      if (!feasible(r, sp.e_bar)) continue;
      if (fabs(r.e - thr) <= sp.amb) amb = 1;
      if (r.e <= thr) pick = min(pick, mm);
      else runner = fmin(runner, r.e);
    }
  };
  if (best >= 0) {
    // candidate tiles: all of them at once, or (more than the list holds) one
    // tile per thread at a time
    each_tile([&](const TileRec& r, int t) {
      if (r.best != best) return;
      if (r.emin <= thr + sp.amb) {
        const int at = atomicAdd(&ncand, 1);
        if (at < 1024) cand[at] = t;
      } else {
        runner = fmin(runner, r.emin);
      }
    });
    __syncthreads();
    const int nc = ncand;
    if (nc <= 1024) {
      rescan(nc);
    } else {
      for (int base = 0; base < ntiles; base += bd) {
        __syncthreads();
        if (tid == 0) ncand = 0;
        __syncthreads();
        if (base + tid < ntiles) {
          const TileRec r = tiles[base + tid];
          if (r.best == best && r.emin <= thr + sp.amb) cand[atomicAdd(&ncand, 1)] = base + tid;
        }
        __syncthreads();
        rescan(ncand);
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    pick = min(pick, (unsigned)__shfl_xor((int)pick, o, 64));
    amb |= __shfl_xor(amb, o, 64);
    runner = fmin(runner, __shfl_xor(runner, o, 64));
  }
  if (lane == 0) {
    s_pick[wv] = pick;
    s_amb[wv] = amb;
    s_run[wv] = runner;
  }
  __syncthreads();
  {
    const int w = lane & (nw - 1);
    pick = s_pick[w];
    for (int o = nw / 2; o > 0; o >>= 1) pick = min(pick, (unsigned)__shfl_xor((int)pick, o, 64));
  }
  if (upd) su.store(H, tab, St, best < 0 ? 0u : pick, ui, us, uj);  // this decision is final
  if (tid == 0) {
    for (int w = 0; w < nw; ++w) {
      amb |= s_amb[w];
      runner = fmin(runner, s_run[w]);
    }
    DevDecision d;
    if (best < 0) {
      d.mask = 0; d.popcount = 0; d.e_loc = fin[0].e; d.e_min = fin[0].e; d.ambiguous = 1; d.found = 0;
      d.key_gap = INFINITY;
      d.smice_rise = 0.0;
    } else {
      d.mask = pick; d.popcount = best; d.e_loc = fin[pick].e; d.e_min = emin; d.ambiguous = amb; d.found = 1;
      d.key_gap = runner - emin;
      d.smice_rise = 0.0;
    }
    *dec = d;
  }
  if (!slist) return;
  if (tid == 0) {
    nlist = best >= 0 ? 1 : 0;
    slist[0] = 0;
  }
  for (int base = 0; base < ntiles && best > 0; base += bd) {  // (at level 0 the list is mask 0)
    if (tid == 0) ncand = 0;
    __syncthreads();
    const int t = base + tid;
    if (t < ntiles && tiles[t].best == best) cand[atomicAdd(&ncand, 1)] = t;
    __syncthreads();
    const int nc = ncand;
    for (int q = tid; q < nc * 64; q += bd) {
      if ((q & 63) >> lb) continue;
      const uint32_t mm = (uint32_t)cand[q >> 6] << lb | (uint32_t)(q & 63);
      if (__popc(mm) == best && feasible(fin[mm], sp.e_bar)) slist[atomicAdd(&nlist, 1)] = mm;
    }
    __syncthreads();
  }
  __syncthreads();
  if (tid == 0) *scount = nlist;
}

// Self-test hook: sqrt_nr on an array (host compares with the libm result).
__global__ void k_sqrt_selftest(const double* __restrict__ x, double* __restrict__ y, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = sqrt_nr(x[i]);
}

__global__ void k_copy2(const double2* __restrict__ a, double2* __restrict__ b, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    b[i] = a[i];
}

// ---------------------------------------------------------- final outputs --
// Final outputs: the first nd blocks form the diagonal blocks of the reduced
// network (and the status word joins the results), each other block one
// snapshot's largest error of the final reduction over every node-phase.
// Y_Kron(x,x) = y_eq of x's own branch plus those of its reduced-network
// children, found by following each tree child down through reduced nodes
// (which have at most one child) to the first kept node.  (As
// launches of their own 11 and 7.4 us at 1000 nodes; the errors with 256 threads
// a block 42 us at 6000 nodes.)
__global__ __launch_bounds__(512) void k_final(Topo T, State St, int nd, const double2* __restrict__ yeq,
                                               double2* __restrict__ Yk_diag, const int* __restrict__ status,
                                               int* __restrict__ status_out, int nstatus,
                                               const double2* __restrict__ Vcur, const double* __restrict__ absV,
                                               double* __restrict__ err) {
  __shared__ double shd[16];
  if ((int)blockIdx.x < nd) {
    const int x = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x >= 64) return;
    if (x < nstatus) status_out[x] = status[x];
    if (x >= T.n) return;
    double2 D[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) D[q] = make_double2(0.0, 0.0);
    if (St.kept[x]) {
      if (x > 0)
#pragma unroll
        for (int q = 0; q < 9; ++q) D[q] = yeq[(size_t)x * 9 + q];
      for (int e = T.ch_off[x]; e < T.ch_off[x + 1]; ++e) {
        int v = T.ch[e];
        while (!St.kept[v] && T.ch_off[v + 1] > T.ch_off[v]) v = T.ch[T.ch_off[v]];
        if (St.kept[v])
#pragma unroll
          for (int q = 0; q < 9; ++q) D[q] = cadd(D[q], yeq[(size_t)v * 9 + q]);
      }
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) Yk_diag[(size_t)T.ext[x] * 9 + q] = D[q];
    return;
  }
  const int l = blockIdx.x - nd, n = T.n;
  double e = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const unsigned ph = T.phase[i];
    const size_t at = ((size_t)l * n + i) * 3, as = ((size_t)l * n + St.sup[i]) * 3;
#pragma unroll
    for (int p = 0; p < 3; ++p)
      if (ph >> p & 1u) e = fmax(e, fabs(sqrt(cabs2(Vcur[as + p])) - absV[at + p]));
  }
  e = block_reduce(e, [](double a, double b) { return fmax(a, b); }, shd);
  if (threadIdx.x == 0) err[l] = e;
}

}  // namespace okr
