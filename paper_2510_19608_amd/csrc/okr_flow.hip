// Load flow (Section III's scenario library) and fixed-current solve by prefix
// sums.
//
// Nodes are labelled by depth-first position, so with load currents I the
// current of the branch above q is the sum of I over its subtree, a run of
// labels: J(q) = P(end(q)) - P(q) with P the prefix sums of I.  With branch
// drops d = z J, the voltage is V(q) = V0 - D(q), D(q) the sum of d over q's
// root path: the prefix sum, at the place where the tour enters q, of the tour
// that enters (+d) and leaves (-d) every node in depth-first order.  One sweep
// is two block-wide prefix sums whatever the depth of the tree, where a sweep
// level by level waits for two barriers and dependent loads per level.
// Accuracy: D's partial sums are differences of voltage drops, so their
// rounding is below that of adding up |V| ~ 1 level by level.  P's are of the
// size of the feeder's whole current, and the current of a light branch would
// keep only the bits above the rounding of that (a load 1e5 times smaller than
// the others behind an impedance 1e5 times larger: voltages off by 2e-13), so
// the currents are summed in two parts (see Split), whose differences are exact
// to about 2^-90 of the whole current.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "okr_device.h"
#include "okr_flow.h"

namespace okr {

namespace {

constexpr int kFlowThreads = 1024;
constexpr int kFlowWaves = kFlowThreads / 64;
constexpr int kFlowAhead = 4;  // entries whose loads a thread issues together
constexpr int kFlowEntries = 9600;       // nodes a phase that the second form's LDS holds
constexpr size_t kFlowLds = 156 * 1024;  // bound on the dynamic LDS

// A copy shifted along the lanes (DPP control); lanes without a source get 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, ROWS == 0xf);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, ROWS == 0xf);
  return __hiloint2double(hi, lo);
}

// Inclusive prefix sums over rows of 16 lanes, and over the wave (the rows'
// last lanes broadcast).
__device__ __forceinline__ double row_scan(double v) {
  v += dpp<0x111, 0xf>(v);
  v += dpp<0x112, 0xf>(v);
  v += dpp<0x114, 0xf>(v);
  v += dpp<0x118, 0xf>(v);
  return v;
}
__device__ __forceinline__ double wave_scan(double v) {
  v = row_scan(v);
  v += dpp<0x142, 0xa>(v);
  v += dpp<0x143, 0xc>(v);
  return v;
}
__device__ __forceinline__ double2 wave_scan(double2 v) { return make_double2(wave_scan(v.x), wave_scan(v.y)); }

// The value of the lane before (0 in the first).
__device__ __forceinline__ double lane_before(double v) { return dpp<0x138, 0xf>(v); }

__device__ __forceinline__ double read_lane(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ __forceinline__ double last_lane(double v) { return read_lane(v, 63); }

// Sum of the waves' totals before wave wv (t: a total per wave, written before
// the last barrier).
__device__ __forceinline__ double2 waves_before(const double2* t, int wv) {
  const int lane = threadIdx.x & 15;
  double2 v = lane < (int)(blockDim.x >> 6) ? t[lane] : make_double2(0.0, 0.0);
  v = make_double2(row_scan(v.x), row_scan(v.y));
  return wv > 0 ? make_double2(read_lane(v.x, wv - 1), read_lane(v.y, wv - 1)) : make_double2(0.0, 0.0);
}

// The same for three sums at once (t: three totals per wave), a row of lanes
// each: one scan instead of three.
__device__ __forceinline__ void waves_before(const double2 (*t)[3], int wv, double2 (&sum)[3]) {
  const int lane = threadIdx.x & 15, row = (threadIdx.x & 63) >> 4;
  double2 v = row < 3 && lane < (int)(blockDim.x >> 6) ? t[lane][row] : make_double2(0.0, 0.0);
  v = make_double2(row_scan(v.x), row_scan(v.y));
#pragma unroll
  for (int p = 0; p < 3; ++p)
    sum[p] = wv > 0 ? make_double2(read_lane(v.x, 16 * p + wv - 1), read_lane(v.y, 16 * p + wv - 1))
                    : make_double2(0.0, 0.0);
}

// The parts of a current: hi, its multiple of a grid that is fine enough for
// every partial sum of hi's to be exact (up to 128 times the sum `total` of the
// magnitudes that the grid is made for; beyond, they round like plain sums), and
// lo = c - hi, below 2^-46 of total, whose sums round at 2^-53 of that.
struct Split {
  double m;  // 1.5 * 2^e: adding and subtracting it rounds to multiples of 2^(e - 52)
  __device__ __forceinline__ explicit Split(double total) {
    m = total > 1e-280 && total < 1e280 ? ldexp(1.5, ilogb(total) + 7) : 0.0;  // (0: no parts)
  }
  __device__ __forceinline__ double2 hi(double2 c) const { return make_double2((c.x + m) - m, (c.y + m) - m); }
};
__device__ __forceinline__ double l1(double2 a) { return fabs(a.x) + fabs(a.y); }
// Bound on the magnitude of the current that load s draws at voltage v.
__device__ __forceinline__ double current_bound(double2 s, double2 v) { return l1(s) / fmax(fabs(v.x), fabs(v.y)); }

// NaN-propagating maximum of non-negative values over the block (every thread
// gets it); s holds a value per wave and must not be in use.
__device__ __forceinline__ double block_nan_max(double v, double* s) {
  v = nan_max(v, dpp<0x111, 0xf>(v));
  v = nan_max(v, dpp<0x112, 0xf>(v));
  v = nan_max(v, dpp<0x114, 0xf>(v));
  v = nan_max(v, dpp<0x118, 0xf>(v));
  v = nan_max(v, dpp<0x142, 0xa>(v));
  v = nan_max(v, dpp<0x143, 0xc>(v));
  if ((threadIdx.x & 63) == 63) s[threadIdx.x >> 6] = v;
  __syncthreads();
  const int lane = threadIdx.x & 15;
  v = lane < (int)(blockDim.x >> 6) ? s[lane] : 0.0;
  v = nan_max(v, dpp<0x111, 0xf>(v));
  v = nan_max(v, dpp<0x112, 0xf>(v));
  v = nan_max(v, dpp<0x114, 0xf>(v));
  v = nan_max(v, dpp<0x118, 0xf>(v));
  return read_lane(v, 15);
}

// Load currents and magnitudes at the final voltages, and the band check.
__device__ __forceinline__ void flow_finish(const FlowArgs& a, int n, size_t base, const uint8_t* __restrict__ phase,
                                            bool conv, int it, double* shd) {
  double vlo = 1e300, vhi = -1e300;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int x = a.ext[i];
    for (int p = 0; p < 3; ++p) {
      const bool pr = (phase[i] >> p & 1u);
      const double2 v = a.V[base + i * 3 + p];
      if (a.Vext) a.Vext[base + x * 3 + p] = v;
      a.A[base + i * 3 + p] = (i > 0 && pr) ? cconj(cdiv(a.Sload[base + x * 3 + p], v)) : make_double2(0.0, 0.0);
      const double m = pr ? sqrt(cabs2(v)) : 0.0;
      a.absV[base + i * 3 + p] = m;
      if (pr) {
        vlo = fmin(vlo, m);
        vhi = fmax(vhi, m);
      }
    }
  }
  vlo = block_reduce(vlo, [](double x, double y) { return fmin(x, y); }, shd);
  vhi = block_reduce(vhi, [](double x, double y) { return fmax(x, y); }, shd);
  if (threadIdx.x == 0) {
    a.iters[blockIdx.x] = it;
    if (!conv) atomicOr(a.status, 16);
    if (vlo < a.vmin || vhi > a.vmax) atomicOr(a.status, 32);
  }
}

}  // namespace

// Form 1: a node per thread (n <= 1024), a node's impedance and voltage in
// registers, the prefix sums, drops and loads in LDS (X, Y, L: n x 3 each; with
// the loads in registers too the kernel spills); one block per snapshot, one
// more for the cumulative impedances.  kFixed: one sweep at the currents Sload,
// given by label.  kEval: after the load flow, one sweep at the currents
// aggregated over the clusters of an assignment, and each snapshot's largest
// difference of |V^| to the super-node's |V|; besides only the status and |V^|
// are written.  The currents' low parts use Y until the drops need it.  Seven
// barriers and three scans of six doubles per sweep, whatever the depth; bound
// by FP64 and DPP instructions on one CU per snapshot.  1000 nodes, 24
// snapshots, 8 sweeps: 84 us with the cumulative impedances (72 with the
// currents in one part; 96 with one scan of the waves' totals per phase; 228 +
// 20 level by level in LDS); 168 snapshots and the evaluation 99 (80 in one
// part; 417 + 20 level by level in global memory, and three launches).
enum { kLoadFlow = 0, kFixed = 1, kEval = 2 };

template <int MODE>
__global__ __launch_bounds__(kFlowThreads) void k_flow_node(int n, int S, const int* __restrict__ end,
                                                            const int* __restrict__ tour, FlowArgs a, FlowEval ev) {
  constexpr bool FIXED = MODE == kFixed;
  extern __shared__ double2 flow_lds[];
  __shared__ double2 s_tot[3][kFlowWaves][3];  // currents' parts, drops
  __shared__ double s_red[16];
  if (MODE == kLoadFlow && (int)blockIdx.x == S) {
    zroot_block(n, a.parent, a.lvl_off, a.lvl_nodes, a.nlev, a.z, a.Zroot);
    return;
  }
  double2 *X = flow_lds, *Y = flow_lds + 3 * n, *L = flow_lds + 6 * n + 3 * threadIdx.x;
  const int q = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(q >> 6);
  const size_t base = (size_t)blockIdx.x * n * 3;
  const bool on = q < n, last = (q & 63) == 63;
  const unsigned ph = on ? a.phase[q] : 0u;
  const int x = on ? (FIXED ? q : a.ext[q]) : 0;
  const int e = on ? end[q] : 1, t0 = on ? tour[2 * q] : 0, t1 = on ? tour[2 * q + 1] : 0;
  double2 z[9], v[3];
#pragma unroll
  for (int k = 0; k < 9; ++k) z[k] = on ? a.z[(size_t)q * 9 + k] : make_double2(0.0, 0.0);
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (on) L[p] = a.Sload[base + x * 3 + p];
    v[p] = (ph >> p & 1u) ? a.v0[p] : make_double2(0.0, 0.0);
  }
  double total = 0.0;
  if (on)
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (FIXED) total += l1(L[p]);
      else if (q > 0 && (ph >> p & 1u)) total += current_bound(L[p], v[p]);
    }
  const Split parts(block_reduce(total, [](double x, double y) { return x + y; }, s_red));
  // X and Y: prefix sums of the parts of c, a current per thread and phase
  auto prefix_sums = [&](double2(&c)[3]) {
    double2 h[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      h[p] = parts.hi(c[p]);
      c[p] = wave_scan(csub(c[p], h[p]));
      h[p] = wave_scan(h[p]);
      if (last) {
        s_tot[0][wv][p] = h[p];
        s_tot[1][wv][p] = c[p];
      }
    }
    __syncthreads();
    double2 before[3];
    waves_before(s_tot[0], wv, before);
    if (on)
#pragma unroll
      for (int p = 0; p < 3; ++p) X[q * 3 + p] = cadd(h[p], before[p]);
    waves_before(s_tot[1], wv, before);
    if (on)
#pragma unroll
      for (int p = 0; p < 3; ++p) Y[q * 3 + p] = cadd(c[p], before[p]);
    __syncthreads();
  };
  // the sum of c over the threads i0 .. i1 - 1
  auto range_sum = [&](int i0, int i1, int p) {
    double2 hb = make_double2(0.0, 0.0), lb = hb, ha = hb, la = hb;
    if (i1 > 0) {
      hb = X[(i1 - 1) * 3 + p];
      lb = Y[(i1 - 1) * 3 + p];
    }
    if (i0 > 0) {
      ha = X[(i0 - 1) * 3 + p];
      la = Y[(i0 - 1) * 3 + p];
    }
    return cadd(csub(hb, ha), csub(lb, la));
  };
  int it = 0;
  bool conv = false, fixed = FIXED;  // fixed: at the currents L
  for (it = 1; fixed || it <= a.maxit; ++it) {
    double2 c[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      c[p] = make_double2(0.0, 0.0);
      if (fixed) {
        if (on) c[p] = L[p];
      } else if (q > 0 && (ph >> p & 1u)) {
        c[p] = cconj(cdiv(L[p], v[p]));
      }
    }
    prefix_sums(c);
    // branch currents and drops
#pragma unroll
    for (int p = 0; p < 3; ++p) c[p] = range_sum(on ? q : 0, e, p);
    __syncthreads();  // (Y is read)
    if (on)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        Y[q * 3 + p] = cadd(cadd(cmul(z[p * 3], c[0]), cmul(z[p * 3 + 1], c[1])), cmul(z[p * 3 + 2], c[2]));
    __syncthreads();
    // prefix sums of the tour, two steps per thread (read again after the
    // barrier rather than held in registers)
    const double f0 = on ? (t0 & 1 ? -1.0 : 1.0) : 0.0, f1 = on ? (t1 & 1 ? -1.0 : 1.0) : 0.0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const double2 y0 = Y[(t0 >> 1) * 3 + p], y1 = Y[(t1 >> 1) * 3 + p];
      const double2 i = wave_scan(make_double2(f0 * y0.x + f1 * y1.x, f0 * y0.y + f1 * y1.y));
      if (last) s_tot[2][wv][p] = i;
      c[p] = make_double2(lane_before(i.x), lane_before(i.y));
    }
    __syncthreads();
    double2 before[3];
    waves_before(s_tot[2], wv, before);
#pragma unroll
    for (int p = 0; p < 3; ++p) c[p] = cadd(c[p], before[p]);
    if (on) {
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const double2 y0 = Y[(t0 >> 1) * 3 + p], y1 = Y[(t1 >> 1) * 3 + p];
        const double2 d0 = make_double2(c[p].x + f0 * y0.x, c[p].y + f0 * y0.y);
        if (!(t0 & 1)) X[(t0 >> 1) * 3 + p] = d0;
        if (!(t1 & 1)) X[(t1 >> 1) * 3 + p] = make_double2(d0.x + f1 * y1.x, d0.y + f1 * y1.y);
      }
    }
    __syncthreads();
    double dmax = 0.0;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (!(ph >> p & 1u)) continue;
      const double2 nv = csub(a.v0[p], X[q * 3 + p]);
      dmax = nan_max(dmax, cabs2(csub(nv, v[p])));
      v[p] = nv;
    }
    if (fixed) break;
    dmax = sqrt(block_nan_max(dmax, s_red));  // (squares up to here)
    conv = dmax <= a.tol;
    const bool stop = !(dmax <= 1e3) || conv;
    if (MODE != kEval) {
      if (stop) break;
      continue;
    }
    if (!stop && it < a.maxit) continue;
    // the load currents and magnitudes at the final voltages, and the currents
    // summed over the clusters: prefix sums over the member list
    if (q == 0 && !conv) atomicOr(a.status, 16);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const bool pr = ph >> p & 1u;
      if (on) L[p] = q > 0 && pr ? cconj(cdiv(L[p], v[p])) : make_double2(0.0, 0.0);
      if (on) a.absV[base + q * 3 + p] = pr ? sqrt(cabs2(v[p])) : 0.0;  // (in registers to the end it spills)
    }
    __syncthreads();
    const int mq = on ? ev.mem[q] : 0;
#pragma unroll
    for (int p = 0; p < 3; ++p) c[p] = on ? flow_lds[6 * n + 3 * mq + p] : make_double2(0.0, 0.0);
    prefix_sums(c);
    const int m0 = on ? ev.moff[q] : 0, m1 = on ? ev.moff[q + 1] : 0;
    if (on)
#pragma unroll
      for (int p = 0; p < 3; ++p) L[p] = range_sum(m0, m1, p);
    fixed = true;  // (a barrier precedes the next writes of X and Y)
  }
  if (MODE == kEval) {
    double e = 0.0;
    if (on) {
      const int s = ev.sup[q];
#pragma unroll
      for (int p = 0; p < 3; ++p)
        if (ph >> p & 1u) e = fmax(e, fabs(a.absV[base + q * 3 + p] - sqrt(cabs2(csub(a.v0[p], X[s * 3 + p])))));
    }
    e = block_reduce(e, [](double x, double y) { return fmax(x, y); }, s_red);
    if (q == 0) ev.err[blockIdx.x] = e;
    return;
  }
  if (on)
#pragma unroll
    for (int p = 0; p < 3; ++p) a.V[base + q * 3 + p] = v[p];
  if (FIXED) return;
  __syncthreads();
  flow_finish(a, n, base, a.phase, conv, it, s_red);
}

// Form 1 for small feeders (n <= kFlowSmall): a thread per node and phase, so
// that a node's three phases run in three waves side by side instead of one
// after the other (a single wave issues one FP64 instruction in about 8 cycles
// here).  The load flow and the cumulative impedances.  30 nodes: 17.6 us a
// launch (15.4 with the currents in one part; 25 with a thread per node).
constexpr int kFlowSmall = 320;
__global__ __launch_bounds__(kFlowThreads) void k_flow_small(int n, int S, const int* __restrict__ end,
                                                             const int* __restrict__ tour, FlowArgs a) {
  __shared__ double2 X[3][kFlowSmall], Y[3][kFlowSmall], W[3][kFlowSmall];  // (W: the currents' low parts)
  __shared__ double2 s_tot[3][16];
  __shared__ double s_red[16];
  if ((int)blockIdx.x == S) {
    zroot_block(n, a.parent, a.lvl_off, a.lvl_nodes, a.nlev, a.z, a.Zroot);
    return;
  }
  const int nw = (n + 63) >> 6, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = wv / nw, w0 = p * nw, q = (wv - w0) * 64 + (threadIdx.x & 63);
  const size_t base = (size_t)blockIdx.x * n * 3;
  const bool on = q < n, last = (threadIdx.x & 63) == 63;
  const unsigned ph = on ? a.phase[q] : 0u;
  const bool pr = ph >> p & 1u;
  const int e = on ? end[q] : 1, t0 = on ? tour[2 * q] : 0, t1 = on ? tour[2 * q + 1] : 0;
  double2 z[3], s = make_double2(0.0, 0.0), v = pr ? a.v0[p] : s;
#pragma unroll
  for (int c = 0; c < 3; ++c) z[c] = on ? a.z[(size_t)q * 9 + p * 3 + c] : make_double2(0.0, 0.0);
  if (on) s = a.Sload[base + (size_t)a.ext[q] * 3 + p];
  const double f0 = on ? (t0 & 1 ? -1.0 : 1.0) : 0.0, f1 = on ? (t1 & 1 ? -1.0 : 1.0) : 0.0;
  const double bound = q > 0 && pr ? current_bound(s, v) : 0.0;
  const Split parts(block_reduce(bound, [](double x, double y) { return x + y; }, s_red));
  int it = 0;
  bool conv = false;
  for (it = 1; it <= a.maxit; ++it) {
    double2 c = q > 0 && pr ? cconj(cdiv(s, v)) : make_double2(0.0, 0.0);
    double2 h = parts.hi(c);
    c = wave_scan(csub(c, h));
    h = wave_scan(h);
    if (last) {
      s_tot[0][wv] = h;
      s_tot[1][wv] = c;
    }
    __syncthreads();
    for (int w = w0; w < wv; ++w) {
      h = cadd(h, s_tot[0][w]);
      c = cadd(c, s_tot[1][w]);
    }
    if (on) {
      X[p][q] = h;
      W[p][q] = c;
    }
    __syncthreads();
    double2 d = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double2 hi = X[k][e - 1], lo = W[k][e - 1];
      if (on && q > 0) {
        hi = csub(hi, X[k][q - 1]);
        lo = csub(lo, W[k][q - 1]);
      }
      const double2 j = cmul(z[k], cadd(hi, lo));
      d = k ? cadd(d, j) : j;
    }
    if (on) Y[p][q] = d;
    __syncthreads();
    const double2 y0 = Y[p][t0 >> 1], y1 = Y[p][t1 >> 1];
    const double2 g = wave_scan(make_double2(f0 * y0.x + f1 * y1.x, f0 * y0.y + f1 * y1.y));
    if (last) s_tot[2][wv] = g;
    c = make_double2(lane_before(g.x), lane_before(g.y));
    __syncthreads();
    for (int w = w0; w < wv; ++w) c = cadd(c, s_tot[2][w]);
    if (on) {
      const double2 d0 = make_double2(c.x + f0 * y0.x, c.y + f0 * y0.y);
      if (!(t0 & 1)) X[p][t0 >> 1] = d0;
      if (!(t1 & 1)) X[p][t1 >> 1] = make_double2(d0.x + f1 * y1.x, d0.y + f1 * y1.y);
    }
    __syncthreads();
    double dmax = 0.0;
    if (pr) {
      const double2 nv = csub(a.v0[p], X[p][q]);
      dmax = nan_max(dmax, cabs2(csub(nv, v)));
      v = nv;
    }
    dmax = sqrt(block_nan_max(dmax, s_red));
    if (!(dmax <= 1e3)) break;
    if (dmax <= a.tol) {
      conv = true;
      break;
    }
  }
  if (on) a.V[base + q * 3 + p] = v;
  __syncthreads();
  flow_finish(a, n, base, a.phase, conv, it, s_red);
}

struct FlowPhases {
  const int *lab[3], *ende[3], *tour[3], *idx;
  int cnt[3], most;  // entries of each phase's list, and the most of them
};

// Form 2: phase by phase, over the list of the nodes that have the phase (a
// subtree, in label order), so that one phase's prefix sums or drops fit in LDS
// (X) for up to 9600 nodes a phase and absent phases cost nothing.  Loads and
// voltages lie by phase and list entry in the V and A slices until the end,
// branch currents by phase and label in the J slice.  A wave takes a run of
// rows of 64 entries, or of the tour.  The list's rows are scanned each by
// itself, in the two parts of the currents: a subtree that ends in its first
// entry's row is the difference of two lanes; a longer one is the rest of that
// row, the rows between (from the prefix sums of the rows' parts, R) and the
// beginning of the row that it ends in, none of which cancels.  Of the tour, a
// wave's total is formed first, then the run is scanned from the sum of the
// waves before it.  6000 nodes, 96 snapshots, 9 sweeps: 780 us with the cumulative
// impedances (700 with the currents in one part, a wave's rows in one scan;
// 1100 + 88 level by level in breadth-first storage), bound by latency on 96 CUs.
// 8400 nodes, 288 snapshots, 12 sweeps: 2.55 ms in blocks of 512, two on a
// compute unit (2.30 in one part; 3.99 + 0.12 level by level).
template <bool FIXED, int BT>
__global__ __launch_bounds__(BT) void k_flow_phase(int n, int S, FlowPhases t, FlowArgs a) {
  extern __shared__ double2 flow_lds[];
  __shared__ double2 s_tot[BT / 64];
  __shared__ double s_red[16];
  if (!FIXED && (int)blockIdx.x == S) {
    zroot_block(n, a.parent, a.lvl_off, a.lvl_nodes, a.nlev, a.z, a.Zroot);
    return;
  }
  double2* X = flow_lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t base = (size_t)blockIdx.x * n * 3;
  double2 *Sb = a.V + base, *Vb = a.A + base, *Jb = a.J + base;
  const double2* Sl = a.Sload + base;
  double total = 0.0;
  for (int p = 0; p < 3; ++p)
    for (int k = tid; k < t.cnt[p]; k += BT) {
      const int i = t.lab[p][k] >> 3;
      if (FIXED) {
        total += l1(Sl[(size_t)i * 3 + p]);
        continue;
      }
      const double2 s = Sl[(size_t)a.ext[i] * 3 + p];
      Sb[p * n + k] = s;
      Vb[p * n + k] = a.v0[p];
      if (k > 0) total += current_bound(s, a.v0[p]);
    }
  const Split parts(block_reduce(total, [](double x, double y) { return x + y; }, s_red));  // (and a barrier)
  double2 *Rh = X + t.most, *Rl = Rh + (t.most + 63) / 64;  // prefix sums over the rows, in parts
  int it = 0;
  bool conv = false;
  for (it = 1; it <= a.maxit; ++it) {
    for (int p = 0; p < 3; ++p) {
      const int cnt = t.cnt[p], C = (cnt + BT - 1) / BT, rows = (cnt + 63) / 64, r0 = wv * C;
      const double2 *Sp = Sb + (size_t)p * n, *Vp = Vb + (size_t)p * n;
      for (int i = 0; i < C && r0 + i < rows; i += kFlowAhead) {
        double2 sv[kFlowAhead], vv[kFlowAhead];
        int e[kFlowAhead], q[kFlowAhead];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          const int k = min((r0 + i + u) * 64 + lane, cnt - 1);
          e[u] = t.ende[p][k];
          q[u] = t.lab[p][k] >> 3;
          if (FIXED) {
            sv[u] = Sl[(size_t)q[u] * 3 + p];
          } else {
            sv[u] = Sp[k];
            vv[u] = Vp[k];
          }
        }
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          const int r = r0 + i + u, k = r * 64 + lane;
          if (i + u >= C || r >= rows) break;
          double2 c = make_double2(0.0, 0.0);
          if (k < cnt) {
            if (FIXED) c = sv[u];
            else if (k > 0) c = cconj(cdiv(sv[u], vv[u]));  // (entry 0 is the root)
          }
          double2 h = parts.hi(c);
          c = wave_scan(csub(c, h));
          h = wave_scan(h);
          if (lane == 63) {
            Rh[r] = h;
            Rl[r] = c;
          }
          // the subtree's part in this row
          const int to = k < cnt ? min(e[u] - 1 - r * 64, 63) : lane;
          const double2 J =
              make_double2((__shfl(h.x, to, 64) - lane_before(h.x)) + (__shfl(c.x, to, 64) - lane_before(c.x)),
                           (__shfl(h.y, to, 64) - lane_before(h.y)) + (__shfl(c.y, to, 64) - lane_before(c.y)));
          if (k < cnt) {
            X[k] = cadd(h, c);
            Jb[(size_t)p * n + q[u]] = J;
          }
        }
      }
      __syncthreads();
      if (wv == 0) {
        double2 h0 = make_double2(0.0, 0.0), l0 = h0;
        for (int r = lane; r - lane < rows; r += 64) {
          double2 h = r < rows ? Rh[r] : make_double2(0.0, 0.0), l = r < rows ? Rl[r] : make_double2(0.0, 0.0);
          h = cadd(h0, wave_scan(h));
          l = cadd(l0, wave_scan(l));
          if (r < rows) {
            Rh[r] = h;
            Rl[r] = l;
          }
          h0 = make_double2(last_lane(h.x), last_lane(h.y));
          l0 = make_double2(last_lane(l.x), last_lane(l.y));
        }
      }
      __syncthreads();
      for (int k1 = tid; k1 < cnt; k1 += kFlowAhead * BT) {
        int e[kFlowAhead];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) e[u] = t.ende[p][min(k1 + u * BT, cnt - 1)];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          const int k = k1 + u * BT, ra = k >> 6, rb = (e[u] - 1) >> 6;
          if (k >= cnt) break;
          if (ra == rb) continue;
          double2* J = Jb + (size_t)p * n + (t.lab[p][k] >> 3);
          double2 c = cadd(*J, X[e[u] - 1]);
          if (rb > ra + 1) c = cadd(c, cadd(csub(Rh[rb - 1], Rh[ra]), csub(Rl[rb - 1], Rl[ra])));
          *J = c;
        }
      }
      __syncthreads();
    }
    double dmax = 0.0;
    for (int p = 0; p < 3; ++p) {
      const int cnt = t.cnt[p];
      for (int k1 = tid; k1 < cnt; k1 += 2 * BT) {
        int q[2];
        double2 d[2], zz[2][3], jj[2][3];
#pragma unroll
        for (int u = 0; u < 2; ++u) q[u] = t.lab[p][min(k1 + u * BT, cnt - 1)];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            zz[u][c] = a.z[(size_t)(q[u] >> 3) * 9 + p * 3 + c];
            jj[u][c] = Jb[(size_t)c * n + (q[u] >> 3)];
          }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          d[u] = make_double2(0.0, 0.0);
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (q[u] >> c & 1) d[u] = cadd(d[u], cmul(zz[u][c], jj[u][c]));
          if (k1 + u * BT < cnt) X[k1 + u * BT] = d[u];
        }
      }
      __syncthreads();
      const int C = (2 * cnt + BT - 1) / BT, k0 = wv * 64 * C + lane;
      double2 acc = make_double2(0.0, 0.0);
      for (int i = 0; i < C; i += kFlowAhead) {
        int s[kFlowAhead];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) s[u] = t.tour[p][min(k0 + (i + u) * 64, 2 * cnt - 1)];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          if (i + u >= C || k0 + (i + u) * 64 >= 2 * cnt) break;
          acc = s[u] & 1 ? csub(acc, X[s[u] >> 1]) : cadd(acc, X[s[u] >> 1]);
        }
      }
      acc = wave_scan(acc);
      if (lane == 63) s_tot[wv] = acc;
      __syncthreads();
      double2 run = waves_before(s_tot, wv);
      for (int i = 0; i < C; i += kFlowAhead) {
        int s[kFlowAhead];
        double2 old[kFlowAhead];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          const int k = k0 + (i + u) * 64;
          s[u] = t.tour[p][min(k, 2 * cnt - 1)];
          if (i + u >= C || k >= 2 * cnt) s[u] = 1;  // (nothing)
        }
        if (!FIXED)
#pragma unroll
          for (int u = 0; u < kFlowAhead; ++u)
            if (!(s[u] & 1)) old[u] = Vb[(size_t)p * n + (s[u] >> 1)];
#pragma unroll
        for (int u = 0; u < kFlowAhead; ++u) {
          if (i + u >= C) break;
          double2 g = k0 + (i + u) * 64 < 2 * cnt ? X[s[u] >> 1] : make_double2(0.0, 0.0);
          if (s[u] & 1) g = make_double2(-g.x, -g.y);
          g = wave_scan(g);
          if (!(s[u] & 1)) {
            const double2 nv = csub(a.v0[p], cadd(run, g));
            if (FIXED) {
              a.V[base + (size_t)(t.lab[p][s[u] >> 1] >> 3) * 3 + p] = nv;
            } else {
              dmax = nan_max(dmax, cabs2(csub(nv, old[u])));
              Vb[(size_t)p * n + (s[u] >> 1)] = nv;
            }
          }
          run = make_double2(run.x + last_lane(g.x), run.y + last_lane(g.y));
        }
      }
      __syncthreads();
    }
    if (FIXED) break;
    dmax = sqrt(block_nan_max(dmax, s_red));  // (squares up to here)
    if (!(dmax <= 1e3)) break;
    if (dmax <= a.tol) {
      conv = true;
      break;
    }
  }
  // voltages by label (over the loads, no longer read)
  for (int k = tid; k < n * 3; k += BT) {
    const int p = k % 3, i = t.idx[p * n + k / 3];
    if (FIXED) {
      if (i < 0) a.V[base + k] = make_double2(0.0, 0.0);
    } else {
      a.V[base + k] = i >= 0 ? Vb[(size_t)p * n + i] : make_double2(0.0, 0.0);
    }
  }
  if (FIXED) return;
  __syncthreads();
  flow_finish(a, n, base, a.phase, conv, it, s_red);
}

// ---- host ----

namespace {

// The tour of a tree given by label (or list entry): 2 q where q is entered,
// 2 q + 1 where it is left.
void append_tour(const std::vector<int>& end, std::vector<int>& out) {
  const int n = (int)end.size();
  std::vector<int> open;
  for (int q = 0; q < n; ++q) {
    while (!open.empty() && end[open.back()] <= q) {
      out.push_back(2 * open.back() + 1);
      open.pop_back();
    }
    out.push_back(2 * q);
    open.push_back(q);
  }
  for (; !open.empty(); open.pop_back()) out.push_back(2 * open.back() + 1);
}

int most_entries(const FlowPlan& p) {
  int m = 1;
  for (int c : p.cnt) m = c > m ? c : m;
  return m;
}

FlowPhases phases(const FlowPlan& p, const int* tab) {
  FlowPhases t;
  for (int c = 0; c < 3; ++c) {
    t.lab[c] = tab + p.lab[c];
    t.ende[c] = tab + p.ende[c];
    t.tour[c] = tab + p.ptour[c];
    t.cnt[c] = p.cnt[c];
  }
  t.idx = tab + p.idx;
  t.most = most_entries(p);
  return t;
}

size_t node_lds(int n) { return sizeof(double2) * 9 * (size_t)n; }
// (a phase's prefix sums or drops, and the rows' two parts)
size_t phase_lds(const FlowPlan& p) {
  const size_t m = most_entries(p);
  return sizeof(double2) * (m + 2 * ((m + 63) / 64));
}

// Blocks of 512 threads, two on a compute unit, where blocks of 1024 would leave
// a second round of them (more snapshots than compute units) and two blocks' sums
// fit in a unit's LDS.
constexpr int kComputeUnits = 256;
bool pairs_of_blocks(const FlowPlan& p, int S) { return S > kComputeUnits && phase_lds(p) <= 79 * 1024; }

}  // namespace

FlowPlan flow_tables(int n, const int* end, const uint8_t* phase, std::vector<int>& out) {
  FlowPlan p;
  p.n = n;
  if (n <= kFlowThreads) {
    p.form = 1;
    const std::vector<int> e(end, end + n);
    p.end = out.size();
    out.insert(out.end(), e.begin(), e.end());
    p.tour = out.size();
    append_tour(e, out);
    return p;
  }
  std::vector<int> lab[3], idx(3 * (size_t)n, -1);
  for (int c = 0; c < 3; ++c) {
    for (int q = 0; q < n; ++q)
      if (phase[q] >> c & 1) {
        idx[(size_t)c * n + q] = (int)lab[c].size();
        lab[c].push_back(q);
      }
    p.cnt[c] = (int)lab[c].size();
  }
  if (most_entries(p) > kFlowEntries) return p;
  p.form = 2;
  for (int c = 0; c < 3; ++c) {
    std::vector<int> e(lab[c].size());
    std::vector<int> below(n + 1, 0);  // list entries with a smaller label
    for (int q = 0; q < n; ++q) below[q + 1] = below[q] + (phase[q] >> c & 1);
    for (size_t k = 0; k < e.size(); ++k) e[k] = below[end[lab[c][k]]];
    p.lab[c] = out.size();
    for (int q : lab[c]) out.push_back(q << 3 | phase[q]);
    p.ende[c] = out.size();
    out.insert(out.end(), e.begin(), e.end());
    p.ptour[c] = out.size();
    append_tour(e, out);
  }
  p.idx = out.size();
  out.insert(out.end(), idx.begin(), idx.end());
  return p;
}

hipError_t flow_prepare(const FlowPlan& p) {
  const void* f[3] = {nullptr, nullptr, nullptr};
  if (p.form == 1 && node_lds(p.n) > 60 * 1024) {
    f[0] = reinterpret_cast<const void*>(&k_flow_node<kLoadFlow>);
    f[1] = reinterpret_cast<const void*>(&k_flow_node<kFixed>);
    f[2] = reinterpret_cast<const void*>(&k_flow_node<kEval>);
  } else if (p.form == 2 && phase_lds(p) > 60 * 1024) {
    f[0] = reinterpret_cast<const void*>(&k_flow_phase<false, kFlowThreads>);
    f[1] = reinterpret_cast<const void*>(&k_flow_phase<true, kFlowThreads>);
    f[2] = reinterpret_cast<const void*>(&k_flow_phase<false, kFlowThreads / 2>);
  }
  for (const void* k : f)
    if (k) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFlowLds);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

void flow_launch(const FlowPlan& p, const FlowArgs& a, int S, hipStream_t st) {
  if (p.form == 1 && p.n <= kFlowSmall)
    hipLaunchKernelGGL(k_flow_small, dim3(S + 1), dim3((p.n + 63) / 64 * 192), 0, st, p.n, S, a.tab + p.end,
                       a.tab + p.tour, a);
  else if (p.form == 1)
    hipLaunchKernelGGL(k_flow_node<kLoadFlow>, dim3(S + 1), dim3((p.n + 63) / 64 * 64), node_lds(p.n), st, p.n, S,
                       a.tab + p.end, a.tab + p.tour, a, FlowEval{});
  else
    hipLaunchKernelGGL((pairs_of_blocks(p, S) ? k_flow_phase<false, kFlowThreads / 2> : k_flow_phase<false, kFlowThreads>),
                       dim3(S + 1), dim3(pairs_of_blocks(p, S) ? kFlowThreads / 2 : kFlowThreads), phase_lds(p), st, p.n,
                       S, phases(p, a.tab), a);
}

void flow_eval_launch(const FlowPlan& p, const FlowArgs& a, const FlowEval& e, int S, hipStream_t st) {
  hipLaunchKernelGGL(k_flow_node<kEval>, dim3(S), dim3((p.n + 63) / 64 * 64), node_lds(p.n), st, p.n, S,
                     a.tab + p.end, a.tab + p.tour, a, e);
}

void flow_fixed_launch(const FlowPlan& p, const int* tab, const uint8_t* phase, const double2* z, const double2* v0,
                       const double2* I, double2* J, double2* V, int S, hipStream_t st) {
  FlowArgs a{};
  a.phase = phase;
  a.z = z;
  a.Sload = I;
  for (int c = 0; c < 3; ++c) a.v0[c] = v0[c];
  a.maxit = 1;
  a.V = V;
  a.J = J;
  if (p.form == 1)
    hipLaunchKernelGGL(k_flow_node<kFixed>, dim3(S), dim3((p.n + 63) / 64 * 64), node_lds(p.n), st, p.n, S,
                       tab + p.end, tab + p.tour, a, FlowEval{});
  else
    hipLaunchKernelGGL((k_flow_phase<true, kFlowThreads>), dim3(S), dim3(kFlowThreads), phase_lds(p), st, p.n, S, phases(p, tab), a);
}

}  // namespace okr
