// amh_grad.h -- parameter blocks of the gradient and L-BFGS kernels (amh_grad.hip),
// shared with the C ABI (amh_api.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "amh_kernels.h"

namespace amh {

constexpr unsigned int kErrGradEnergy = kErrEnergy;
constexpr int kReduceThreads = 256;   // of a workgroup, that sum over a chain's vectors
constexpr int kLbfgsMaxHistory = 64;
constexpr int kLbfgsMaxNonmonotone = 64;
// Fixed L-BFGS workspace of amh_minimize_noalloc: 8 Mi doubles (64 MiB) per device,
// e.g. 499 conformations of 400 residues with m = 8 (16,800 doubles each).
constexpr long long kNoallocScratchDoubles = 8LL << 20;
constexpr int kMaxDevices = 64;

struct GradParams {
  int L;
  const double* s;      // [B][2L]
  const float* table;   // padded -ln p rows
  int stride, nb;
  double d_min, bin_w;
  double vfar;          // sum of every row's no-contact value
  int ordered;          // V pair by pair (ordered_energies)
  int cap;              // pairs a wavefront's list holds
  double* V;            // [B] or null
  double* g;            // [B][2L] or null
  unsigned int* err;
};

struct LbfgsParams {
  int L;
  double* s;            // [B][2L] in/out
  const float* table;
  int stride, nb;
  double d_min, bin_w;
  double vfar;          // sum of every row's no-contact value
  int ordered;          // V pair by pair (ordered_energies)
  int cap;              // pairs a wavefront's list holds
  int n_iter, m, nonmonotone, max_ls;
  double c1, shrink, gtol, step0;
  double* work;         // [B][(5 + 2m) 2L]
  double* V;            // [B] or null
  int32_t* iters;       // [B] or null
  int32_t* status;      // [B] or null
  double* f_trace;      // [B][n_iter + 1] or null
  double* x_trace;      // [B][n_iter + 1][2L] or null (iterates, unwrapped)
  double* v_state;      // [B][2] (current V, best V) or null
  double* s_best;       // [B][2L], updated with v_state
  unsigned int* err;
};

// Whether a table whose entries deviate from their row's no-contact value by dev_max at most can
// have a pair outside the range of value_grad's integer energy sums (|deviation| < 2^16; a
// Catmull-Rom value is at most 1.25 times the largest of its four).
inline bool ordered_energies(float dev_max) { return !(1.3 * (double)dev_max < 65536.0); }

// A wavefront's list of cap pairs (a multiple of 8, 64 at least).
__host__ __device__ inline size_t grad_pair_bytes(int cap) { return 10 * (size_t)cap + 640; }
// Pairs of the one list that W wavefronts sharing ntile tiles make of theirs (beside 1152 bytes of
// marks and positions a tile).
__host__ __device__ inline int grad_shared_pairs(int W, int cap, int ntile) {
  return ((int)grad_pair_bytes(cap) * W - 1152 * ntile) / 10;
}
inline size_t grad_lds_bytes(int L, int W, int cap) {
  return 8 * (12 * (size_t)L + 6 * ((size_t)L + 1) + 3 * (kReduceThreads / 64)) + 16 * (size_t)((L + 7) / 8) +
         W * grad_pair_bytes(cap);
}
inline size_t lbfgs_lds_bytes(int L, int W, int cap, int m, int M) {
  return grad_lds_bytes(L, W, cap) + 8 * (2 * (size_t)m + (size_t)M);
}
inline size_t lbfgs_work_doubles(int L, int m) { return (5 + 2 * (size_t)m) * 2 * (size_t)L; }

template <bool FEW> __global__ void grad_kernel(GradParams P);
template <bool FEW> __global__ void lbfgs_kernel(LbfgsParams P);

}  // namespace amh
