// amh_proposal.h -- proposal randoms, schedule and trace helpers shared by the localized
// (amh_local.hip) and global (amh_global.hip) sweep kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amh_device.h"
#include "amh_kernels.h"

namespace amh {

// Parameters in constant memory.  cold() hides where a pointer came from, so that a field
// read through it is loaded where it is used instead of being kept in scalar registers.
typedef const __attribute__((address_space(4))) SweepParams CParams;
__device__ __forceinline__ CParams& cold(CParams& P) {
  CParams* p = &P;
  asm volatile("" : "+s"(p));
  return *p;
}

struct Batch {  // proposal randoms of 64 consecutive proposals, one per lane
  double delta, log_u, cd, sd;
};

// Proposal width of sweep t: constant, or reduced geometrically from sigma to
// sigma_end over the schedule (Sec. 2.3 and Sec. 3 reduce it from 10 to 4 degrees).
template <class Params>   // (SweepParams, in whichever address space)
__device__ __forceinline__ double sigma_at(Params& P, int64_t t) {
  if (P.sigma_end > 0.0 && P.sigma > 0.0 && P.S > 1)
    return P.sigma * pow(P.sigma_end / P.sigma, (double)t / (double)(P.S - 1));
  return P.sigma;
}

template <class Params>
__device__ __forceinline__ Batch fill_batch(Params& P, int kb, uint32_t t, uint32_t chain, int lane) {
  const int k = kb + lane;
  Batch b{0.0, 0.0, 1.0, 0.0};
  if (k < 2 * P.L) {
    const Draw d = proposal_draw((uint32_t)k, t, chain, P.key0, P.key1, sigma_at(P, t));
    b.delta = d.delta; b.log_u = d.log_u; b.cd = d.cd; b.sd = d.sd;
  }
  return b;
}

template <class Params>
__device__ __forceinline__ int trace_slot(Params& P, int chain) {
  int slot = -1;
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (m < P.n_trace && P.trace_chain[m] == chain) slot = m;
  return slot;
}

template <class Params>
__device__ __forceinline__ void trace_step(Params& P, int slot, int64_t t, int k,
                                           double dE, double delta, int acc) {
  if (slot < 0) return;
  const int64_t idx = (t - P.trace_t0) * (int64_t)(2 * P.L) + k;
  if (idx < 0 || idx >= P.trace_cap) return;
  P.tr_dE[slot * P.trace_cap + idx] = dE;
  P.tr_delta[slot * P.trace_cap + idx] = delta;
  P.tr_acc[slot * P.trace_cap + idx] = (uint8_t)acc;
}

// Inverse temperature of sweep t (a call, not inlined: the compiler would keep the constants
// of pow in registers throughout the loop over the sweeps).
[[maybe_unused]] static __device__ __attribute__((noinline)) double sweep_beta(CParams* P, int64_t t) {
  double T_t = P->T0;
  if (P->S > 1) T_t = P->T0 * pow(P->T1 / P->T0, (double)t / (double)(P->S - 1));
  return 1.0 / T_t;
}

}  // namespace amh
