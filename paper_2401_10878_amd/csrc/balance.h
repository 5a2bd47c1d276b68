// Zero-net-flux balance controller (balance mode 2).  The lattice blocks'
// (mass, momentum) sums are added in two fixed-order stages: BAL_PARTS
// wavefronts each sum one contiguous range of blocks (lane t takes entries
// t, t + 64, .. of the range, then a fixed tree), then one wavefront sums the
// BAL_PARTS results the same way, giving the lattice mass M and momentum P.
// init: M, P_{-1} = P, b_0 = -P / M.  Update after the collision of step t
// (which used b_t): C_t = P_t - P_{t-1} - b_t M, b_{t+1} = -(P_t + C_t) / M.
// The acceleration in use is a = fluid_accel + b.
//
// Between two steps of one call the first stage runs as extra workgroups of
// the contact treatment and the second as one of the motion kernel (both
// after the lattice pass that left the block sums, before the one that uses
// the result), which saves two launches of 4.6 us each; after the last step
// of a call the two stages are launches of their own.  Both ways run these
// functions, so they give the same bits.  (The second stage as a further
// workgroup of the detection had made that kernel slower by 11 of 78 us.)
#pragma once

#include "context.h"

namespace hlbm {

__device__ inline void balance_stage1(const double* part, unsigned nblocks, unsigned k,
                                      double* out) {
  const unsigned chunk = (nblocks + BAL_PARTS - 1) / BAL_PARTS;
  const unsigned b0 = k * chunk;
  const unsigned b1 = b0 + chunk < nblocks ? b0 + chunk : nblocks;
  const unsigned lane = threadIdx.x % WAVE;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (unsigned b = b0 + lane; b < b1; b += WAVE)
    for (int m = 0; m < 4; ++m) acc[m] += part[4 * (size_t)b + m];
  for (int m = 0; m < 4; ++m) {
    const double s = wave_sum(acc[m]);
    if (lane == 0) out[4 * k + m] = s;
  }
}

__device__ inline void balance_stage2(const double* parts, Counters* ctr, const Phys& ph,
                                      int init) {
#pragma clang fp contract(off)
  const unsigned lane = threadIdx.x % WAVE;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (unsigned b = lane; b < BAL_PARTS; b += WAVE)
    for (int m = 0; m < 4; ++m) acc[m] += parts[4 * (size_t)b + m];
  for (int m = 0; m < 4; ++m) acc[m] = wave_sum(acc[m]);
  if (lane != 0) return;
  if (init) ctr->bal_M = acc[0];
  const double M = ctr->bal_M;
  for (int k = 0; k < 3; ++k) {
    const double P = acc[1 + k];
    double b;
    if (init) {
      b = -P / M;
    } else {
      const double Ct = P - ctr->bal_P[k] - ctr->bal_b[k] * M;
      b = -(P + Ct) / M;
    }
    ctr->bal_b[k] = b;
    ctr->bal_P[k] = P;
    ctr->bal_a[k] = ph.a_ext[k] + b;
  }
}

}  // namespace hlbm
