// Inverse of a phase-restricted 3x3 block and the Kron-reduced branch of a kept
// node.
#pragma once

#include <hip/hip_runtime.h>

#include "okr_device.h"
#include "okr_internal.h"

namespace okr {

// Restricted inverse of a 3x3 block on the phases in `mask` (zero-padded):
// for blocks supported on the present-phase principal submatrix this is the
// Moore-Penrose pseudo-inverse (Section II.B footnote).  Closed forms for
// 1x1, 2x2 (adjugate) and 3x3 (cofactors), with constant indices so that the
// blocks stay in registers.  Returns false if singular.
template <int I>
__device__ __forceinline__ bool inv_one(const double2* A, double2* out) {
  const double2 a = A[I * 4];
  if (cabs2(a) == 0.0) return false;
  out[I * 4] = cdiv(make_double2(1.0, 0.0), a);
  return true;
}
template <int I, int J>
__device__ __forceinline__ bool inv_two(const double2* A, double2* out) {
  const double2 a = A[I * 3 + I], b = A[I * 3 + J], c = A[J * 3 + I], d = A[J * 3 + J];
  const double2 det = csub(cmul(a, d), cmul(b, c));
  if (cabs2(det) == 0.0) return false;
  out[I * 3 + I] = cdiv(d, det);
  out[I * 3 + J] = cdiv(make_double2(-b.x, -b.y), det);
  out[J * 3 + I] = cdiv(make_double2(-c.x, -c.y), det);
  out[J * 3 + J] = cdiv(a, det);
  return true;
}
__device__ __forceinline__ bool inv_restricted(const double2* A, unsigned mask, double2* out) {
#pragma unroll
  for (int q = 0; q < 9; ++q) out[q] = make_double2(0.0, 0.0);
  if (mask == 1) return inv_one<0>(A, out);
  if (mask == 2) return inv_one<1>(A, out);
  if (mask == 4) return inv_one<2>(A, out);
  if (mask == 3) return inv_two<0, 1>(A, out);
  if (mask == 5) return inv_two<0, 2>(A, out);
  if (mask == 6) return inv_two<1, 2>(A, out);
  if (mask == 7) {
    double2 cof[9];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) {
        const int r1 = (r + 1) % 3, r2 = (r + 2) % 3, c1 = (c + 1) % 3, c2 = (c + 2) % 3;
        cof[r * 3 + c] = csub(cmul(A[r1 * 3 + c1], A[r2 * 3 + c2]), cmul(A[r1 * 3 + c2], A[r2 * 3 + c1]));
      }
    const double2 det = cadd(cadd(cmul(A[0], cof[0]), cmul(A[1], cof[1])), cmul(A[2], cof[2]));
    if (cabs2(det) == 0.0) return false;
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) out[r * 3 + c] = cdiv(cof[c * 3 + r], det);
    return true;
  }
  return mask == 0;
}

// Kron-reduced branch of every kept node: the eliminated path up to its kept
// parent is a series chain, so y_eq = (sum of z on the path, restricted to
// the node's phases)^-1 (eq. Y_kron for degree-2 and leaf eliminations).
__device__ __forceinline__ void kron_yeq(int x, const Topo& T, const State& St, const double2* __restrict__ z,
                                         double2* __restrict__ yeq, double2* __restrict__ Yk_off,
                                         int* __restrict__ kp_out, int* __restrict__ status) {
  const int xe = T.ext[x];  // (the outputs go by the caller's node ids)
  double2* yo = Yk_off + (size_t)xe * 9;
  double2* ye = yeq + (size_t)x * 9;
  for (int q = 0; q < 9; ++q) { yo[q] = make_double2(0.0, 0.0); ye[q] = yo[q]; }
  const int kp = (x > 0 && St.kept[x]) ? St.sup[T.parent[x]] : -1;
  kp_out[xe] = kp < 0 ? -1 : T.ext[kp];
  if (kp < 0) return;
  const unsigned ph = T.phase[x];
  double2 Z[9];
  for (int q = 0; q < 9; ++q) Z[q] = make_double2(0.0, 0.0);
  for (int v = x; v != kp; v = T.parent[v]) {
    const double2* zv = z + (size_t)v * 9;
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c)
        if ((ph >> r & 1u) && (ph >> c & 1u)) Z[r * 3 + c] = cadd(Z[r * 3 + c], zv[r * 3 + c]);
  }
  if (!inv_restricted(Z, ph, ye)) { atomicOr(status, 1); return; }
  for (int q = 0; q < 9; ++q) yo[q] = make_double2(-ye[q].x, -ye[q].y);
}

}  // namespace okr
