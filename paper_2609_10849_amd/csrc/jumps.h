// Jumps of the derivatives across a face, for the sensors of the oscillation-eliminating maps.
#pragma once
#include "common.h"
#include "xcd.h"

// jump of the derivative of order r across the face between the lines m (minus side) and q (plus side)
template <int P>
__device__ __forceinline__ double line_jump(const double* m, const double* q, int r, const HydroTab* __restrict__ T) {
  double j = 0.0;
#pragma unroll
  for (int k = 0; k <= P; ++k) j = fma(T->Dr0[r][k], r & 1 ? q[k] + m[P - k] : q[k] - m[P - k], j);
  return j;
}

// squared, weighted jumps of the derivatives of order r (eq. euler-oe-jump, eq. magnetic-oe-sensor) across a face between the
// elements at m (minus side) and q (plus side), normal direction D, as square roots.  On the symmetric GLL
// nodes d^r l_k (+1) = (-1)^r d^r l_{p-k} (-1), which the tables hold bit for bit, so the jump of order r is one
// sum over the differences (r even) or sums (r odd) of mirrored values.
template <int P, int D>
__device__ __forceinline__ void face_jumps(const double* m, const double* q, const HydroTab* __restrict__ T, double J[]) {
  constexpr int NP = P + 1;
#pragma unroll
  for (int r = 0; r < NP; ++r) J[r] = 0.0;
#pragma unroll
  for (int l = 0; l < NP; ++l) {
    double dif[NP], sum[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const double a = q[D ? k * NP + l : l * NP + k], b = m[D ? (P - k) * NP + l : l * NP + P - k];
      dif[k] = a - b;
      sum[k] = a + b;
    }
#pragma unroll
    for (int r = 0; r < NP; ++r) {
      double j = 0.0;
#pragma unroll
      for (int k = 0; k < NP; ++k) j = fma(T->Dr0[r][k], r & 1 ? sum[k] : dif[k], j);
      J[r] = fma(0.5 * T->w[l] * j, j, J[r]);
    }
    SCHED_FENCE();
  }
#pragma unroll
  for (int r = 0; r < NP; ++r) J[r] = sqrt(J[r]);
}
