// amh_kernels.hip -- HIP kernels of the Alternating Metropolis-Hastings sampler
// for MI355X (gfx950, wave64).
//
// Method (Ghantasala, Jaiswal, Datta, arXiv 2211.03193): single-torsion Gaussian
// proposals swept over k = 0 .. 2L-1 (Sec. 2.1, Algorithm 1), judged either by the
// full distogram energy V (global MH) or by the energy of the window of residues
// within d/2 of residue k/2 (localized MH, Sec. 2.3); global and localized sweeps
// alternate (Algorithm 1, Fig. 1); acceptance min(1, exp(-beta dE)) (Sec. 2.1).
//
// Mapping to the GPU (our design, not the paper's block-per-chain layout):
//   * a workgroup owns G chains that walk the same proposal index k in lockstep,
//     so every table row a global proposal needs is fetched once per workgroup
//     from L2 and shared by the G chains;
//   * localized sweeps are run by one wavefront per chain with no workgroup
//     barrier; residues beyond the window are brought up to date lazily with one
//     accumulated rigid transform (float64) when they enter the window;
//   * pair energies are handled as deviations from the pair's no-contact value
//     (a second copy of the table with that value subtracted), which are exactly
//     zero beyond the last knot: a pair farther apart than 20.25 A costs a
//     distance and a compare, no table access;
//   * global proposals use every wavefront of the workgroup; dE of pivot p is
//     D_new(p) - D(p), where D(p), the deviation energy of the pair rectangle
//     i < p <= j of the current conformation, is carried from proposal to
//     proposal (the new rectangle sum on accept, an O(L) row/column update when
//     p advances), so each global proposal evaluates one spline per changed near
//     pair instead of two;
//   * the rectangle is walked in 8 x 8 tiles (blocks of 8 residues); a tile whose
//     two bounding spheres lie farther apart than the last knot holds only pairs
//     that add zero and is skipped whole, a decision uniform over the wavefront;
//   * the proposal randoms come from Philox4x32-10 at counter (k, t, chain, 0),
//     the same stream the oracle replays, drawn 64 proposals at a time, one per lane;
//   * the master coordinates (N, CA, C, C-beta) live in LDS in float64 and are
//     rotated in float64; the O(L^2) pair loop reads float32 C-beta positions taken
//     relative to the pivot point, rounded once per proposal, so float32 never
//     accumulates error in the state (an extended 300-residue chain spans ~1000 A,
//     where float32 resolves only ~6e-5 A);
//   * after every anchor sweep the coordinates are rebuilt from the float64
//     torsions by NeRF and V is re-anchored in float64 with Neumaier summation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amh_device.h"
#include "amh_geom.h"
#include "amh_kernels.h"
#include "amh_proposal.h"

namespace amh {

// ---------------------------------------------------------------------------
// Table ingest: repack [P][nb] rows into padded rows [y1, y0..y_{nb-1}, y_{nb-2}, 0...]
// (`out`) and the same rows minus the row's no-contact value y_{nb-1} (`dev`, rounded
// once from float64), and flag non-finite entries.
__global__ void ingest_kernel(const float* __restrict__ y, int64_t P, int nb, int stride,
                              float* __restrict__ out, float* __restrict__ dev, unsigned int* err) {
  const int64_t n = P * (int64_t)stride;
  bool bad = false;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / stride;
    const int c = (int)(e - r * stride);
    float v = 0.0f;
    if (c == 0) v = y[r * nb + 1];
    else if (c <= nb) v = y[r * nb + (c - 1)];
    else if (c == nb + 1) v = y[r * nb + (nb - 2)];
    if (c <= nb && !isfinite(v)) bad = true;
    out[e] = v;
    dev[e] = c <= nb + 1 ? (float)((double)v - (double)y[r * nb + (nb - 1)]) : 0.0f;
  }
  if (bad) atomicOr(err, kErrTable);
}

// Noisy restart: s_k += amplitude (2u - 1) with u from Philox at (k, tag, chain, 1),
// wrapped into (-pi, pi]; one thread per torsion of every chain.
__global__ void perturb_kernel(double* __restrict__ s, int64_t n_total, int n, uint32_t chain_offset,
                               uint32_t tag, uint32_t k0, uint32_t k1, double amplitude) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n_total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e / n), k = (int)(e - (int64_t)c * n);
    const U4 r = philox10(U4{(uint32_t)k, tag, chain_offset + (uint32_t)c, 1u}, k0, k1);
    const double u = ((double)r.x + 0.5) * (1.0 / 4294967296.0);
    s[e] = wrap_angle(s[e] + amplitude * (2.0 * u - 1.0));
  }
}

__global__ void philox_kernel(const uint32_t* __restrict__ ctr, int64_t n, uint32_t k0, uint32_t k1,
                              uint32_t* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const U4 c{ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]};
    const U4 r = philox10(c, k0, k1);
    out[4 * i] = r.x; out[4 * i + 1] = r.y; out[4 * i + 2] = r.z; out[4 * i + 3] = r.w;
  }
}

// Float64 energy V = sum_{i<j} E_ij(|CB_i - CB_j|) of one conformation by the whole
// workgroup.  Beyond the last knot E_ij is the row's no-contact value E_ij(inf), so
// V = vfar + sum over the pairs inside it of (E_ij - E_ij(inf)), vfar the sum of every
// row's no-contact value.  The pairs inside are found as in a global proposal: bounding
// spheres of blocks of 8 residues (float32 centre and radius in sph) cull the 8 x 8 tiles
// whose spheres lie farther apart than the last knot plus 0.05 A; a surviving tile
// is one wavefront step, a pair per lane, tested in float64.  Each pair term is
// rounded to a multiple of 2^-40 (error < 5e-13 per pair) and summed as an integer,
// exactly and so in any order: V does not depend on the launch shape.  acc is one 64-bit
// integer in LDS; every thread returns V.
__device__ double energy64(const float* __restrict__ table, int stride, int nb, double d_min, double w,
                           double vfar, int L, const double* __restrict__ x, float4* __restrict__ sph,
                           long long* acc) {
  const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63;
  const double dfar = d_min + w * ((double)nb - 0.5), d2far = dfar * dfar;   // the last knot
  const double inv_w = 1.0 / w;
  const float rcut = (float)dfar + 0.05f;
  const int nb8 = (L + 7) >> 3, nres8 = 8 * nb8;
  if (tid == 0) *acc = 0;
  // spheres: the 8 residues of a block in 8 aligned lanes of one wavefront
  for (int e0 = 0; e0 < nres8; e0 += T) {
    const int r = e0 + tid;
    const bool real = r < L;
    float vx = 0.0f, vy = 0.0f, vz = 0.0f;
    if (real) {
      const double* q = atom(x, r, 3);
      vx = (float)q[0]; vy = (float)q[1]; vz = (float)q[2];
    }
    const float cnt = sum8(real ? 1.0f : 0.0f), inv = __builtin_amdgcn_rcpf(cnt > 1.0f ? cnt : 1.0f);
    const float cx = sum8(vx) * inv, cy = sum8(vy) * inv, cz = sum8(vz) * inv;
    const float rad = max8(real ? __builtin_amdgcn_sqrtf((vx - cx) * (vx - cx) + (vy - cy) * (vy - cy) +
                                                         (vz - cz) * (vz - cz))
                                : 0.0f);
    if (r < nres8 && (r & 7) == 0) sph[r >> 3] = make_float4(cx, cy, cz, rad);
  }
  __syncthreads();
  // candidate tiles (row block I, column block J), I <= J, one per thread
  long long part = 0;
  const int lr = lane >> 3, lc = lane & 7, per = nb8 * nb8;
  const float inv_nb8 = 1.0f / (float)nb8;
  for (int base = 0; base < per; base += T) {
    const int cand = base + tid;
    int code = 0;
    bool keep = false;
    if (cand < per) {
      const int I = (int)(((float)cand + 0.5f) * inv_nb8), J = cand - I * nb8;
      if (I <= J) {
        const float4 u = sph[I], v = sph[J];
        const float dx = u.x - v.x, dy = u.y - v.y, dz = u.z - v.z, lim = rcut + u.w + v.w;
        keep = dx * dx + dy * dy + dz * dz <= lim * lim;
      }
      code = (I << 10) | J;
    }
    unsigned long long m = __ballot(keep);
    while (m) {
      const int l = __builtin_ctzll(m);
      m &= m - 1;
      const int cd = __builtin_amdgcn_readlane(code, l);
      const int i = 8 * (cd >> 10) + lr, j = 8 * (cd & 1023) + lc;
      if (i < j && j < L) {
        const double* pa = atom(x, i, 3);
        const double* pb = atom(x, j, 3);
        const double dx = pb[0] - pa[0], dy = pb[1] - pa[1], dz = pb[2] - pa[2];
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (d2 < d2far) {
          const float* row = table + (size_t)pair_row(i, j, L) * stride;
          // distance through the hardware reciprocal square root and two Newton steps
          const double e = spline64(row, d2 * rsqrt64(d2), nb, d_min, w, inv_w) - (double)row[nb];
          part += (long long)rint(e * 1099511627776.0);   // e 2^40
        }
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
  if (lane == 0 && part != 0)
    atomicAdd(reinterpret_cast<unsigned long long*>(acc), (unsigned long long)part);
  __syncthreads();
  return vfar + (double)*acc * (1.0 / 1099511627776.0);
}

// ---------------------------------------------------------------------------
// Sum over the P rows of the table of their no-contact value row[nb] (the energy of
// a conformation whose pairs all lie beyond the last knot), float64 Neumaier in a
// fixed order: one workgroup; thread t takes rows t, t + T, ...; the partials are
// combined in thread order by thread 0.
__global__ void far_sum_kernel(const float* __restrict__ table, int64_t P, int stride, int nb,
                               double* __restrict__ out) {
  __shared__ double part[2 * 1024];
  const int tid = threadIdx.x, T = blockDim.x;
  double s = 0.0, c = 0.0;
  for (int64_t r = tid; r < P; r += T) neumaier_add(s, c, (double)table[r * stride + nb]);
  part[2 * tid] = s;
  part[2 * tid + 1] = c;
  __syncthreads();
  if (tid == 0) {
    double a = 0.0, b = 0.0;
    for (int t = 0; t < T; ++t) { neumaier_add(a, b, part[2 * t]); b += part[2 * t + 1]; }
    *out = a + b;
  }
}

// Conformation / energy kernel: one workgroup per conformation.
__global__ void conf_energy_kernel(ConfParams P) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int L = P.L, tid = threadIdx.x;
  const int b = blockIdx.x;
  double* s = reinterpret_cast<double*>(lds);   // [2L]
  double* x64 = s + 2 * L;                      // [12L]
  double* acc = x64 + 12 * L;                   // [2] (a 64-bit sum; 16-byte aligned)
  float4* sph = reinterpret_cast<float4*>(acc + 2);                          // [(L + 7) / 8]
  double* fr = reinterpret_cast<double*>(sph + ((L + 7) >> 3));              // [nerf_scratch(L)]
  const double* src = P.s_in ? P.s_in + (size_t)b * 2 * L : nullptr;
  int bad = 0;   // a non-finite torsion: V(s) is undefined and returned as NaN
  for (int m = tid; m < 2 * L; m += blockDim.x) {
    s[m] = src ? src[m] : kPi;
    bad |= !isfinite(s[m]);
  }
  bad = __syncthreads_or(bad);
  nerf_wg(s, L, x64, fr);
  if (P.atoms_out) {
    float* o = P.atoms_out + (size_t)b * L * 12;
    for (int e = tid; e < L * 12; e += blockDim.x) o[e] = (float)x64[e];
  }
  if (P.atoms64_out) {
    double* o = P.atoms64_out + (size_t)b * L * 12;
    for (int e = tid; e < L * 12; e += blockDim.x) o[e] = x64[e];
  }
  if (P.cb_out) {
    float* o = P.cb_out + (size_t)b * L * 3;
    for (int e = tid; e < L * 3; e += blockDim.x) o[e] = (float)atom(x64, e / 3, 3)[e % 3];
  }
  if (P.s_out)
    for (int m = tid; m < 2 * L; m += blockDim.x) P.s_out[(size_t)b * 2 * L + m] = s[m];
  if (P.table) {
    const double Vs = energy64(P.table, P.stride, P.nb, P.d_min, P.bin_w, P.vfar, L, x64, sph,
                               reinterpret_cast<long long*>(acc));
    const double V = bad ? __builtin_nan("") : Vs;
    // keep_best: V becomes the current energy and replaces the best one only if lower
    // (every thread decides from the old best before it is overwritten)
    const bool better = !(P.v_state && P.keep_best) || V < P.v_state[2 * b + 1];
    __syncthreads();
    if (tid == 0) {
      if (!isfinite(V)) atomicOr(P.err, kErrEnergy);
      if (P.V_out) P.V_out[b] = V;
      if (P.v_state) {
        P.v_state[2 * b] = V;
        if (better) P.v_state[2 * b + 1] = V;
      }
      if (P.counters) {
        P.counters[4 * b + 0] = 0; P.counters[4 * b + 1] = 0;
        P.counters[4 * b + 2] = -1; P.counters[4 * b + 3] = 0;
      }
    }
    if (P.s_best && better)
      for (int m = tid; m < 2 * L; m += blockDim.x) P.s_best[(size_t)b * 2 * L + m] = s[m];
  }
}

// Anchor of one chain after sweep P.t0 - 1 (one workgroup): rebuild the coordinates from
// the float64 torsions (NeRF), re-anchor V in float64 and update the best state and the
// time-to-target.
__device__ __forceinline__ void anchor_body(const SweepParams& P, const int chain) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int L = P.L, n = 2 * L, tid = threadIdx.x;
  double* s = reinterpret_cast<double*>(lds);   // laid out as in conf_energy_kernel
  double* x64 = s + n;
  double* acc = x64 + 12 * L;
  float4* sph = reinterpret_cast<float4*>(acc + 2);
  double* fr = reinterpret_cast<double*>(sph + ((L + 7) >> 3));
  for (int m = tid; m < n; m += blockDim.x) s[m] = P.s[(size_t)chain * n + m];
  const double best = P.v[2 * chain + 1];
  __syncthreads();
  nerf_wg(s, L, x64, fr);
  for (int e = tid; e < 12 * L; e += blockDim.x) P.atoms[(size_t)chain * L * 12 + e] = x64[e];
  const double v = energy64(P.table, P.stride, P.nb, P.d_min, P.bin_w, P.vfar, L, x64, sph,
                            reinterpret_cast<long long*>(acc));
  if (v < best)
    for (int m = tid; m < n; m += blockDim.x) P.s_best[(size_t)chain * n + m] = s[m];
  if (tid == 0) {   // (every thread has read the old best before the barriers above)
    if (!isfinite(v)) atomicOr(P.err, kErrEnergy);
    P.v[2 * chain] = v;
    if (v < best) P.v[2 * chain + 1] = v;
    if (P.counters[4 * chain + 2] < 0 && v <= P.target) P.counters[4 * chain + 2] = P.t0;
    P.counters[4 * chain + 3] += 1;
    const int slot = trace_slot(P, chain);
    if (slot >= 0) {
      const int64_t ai = P.t0 / P.anchor_every - P.trace_anchor0;
      if (ai >= 0 && ai < P.trace_anchor_cap) P.tr_anchor[slot * P.trace_anchor_cap + ai] = v;
    }
  }
}

__global__ __launch_bounds__(256) void anchor_kernel(SweepParams P) { anchor_body(P, blockIdx.x); }

// Several proteins: workgroup (b, q) anchors chain q of group map[b].y of its protein, of
// those whose descriptor asks for it (n_sweeps != 0).
__global__ __launch_bounds__(256) void anchor_batch_kernel(const SweepParams* __restrict__ descs,
                                                           const int2* __restrict__ map, int G) {
  const int2 wm = map[blockIdx.x];
  const SweepParams& P = descs[wm.x];
  const int chain = wm.y * G + (int)blockIdx.y;
  if (P.n_sweeps == 0 || chain >= P.C) return;
  anchor_body(P, chain);
}

// ---------------------------------------------------------------------------
// LDS layout of a localized-sweep workgroup: per chain the float64 atoms [L][4][3] and
// the torsions [2L] (112 L bytes, padded to 64 mod 256, so that the same residue of the
// G chains, read together, falls in different banks); then one progress counter per
// wavefront and the accept counts per wavefront and chain.
__host__ __device__ inline size_t chain_stride(int L) {
  const size_t b = 112 * (size_t)L;
  return b + ((64 + 256 - (b & 255)) & 255);
}

struct Lds {
  unsigned char* base;
  int L, G;
  __device__ size_t per() const { return chain_stride(L); }
  __device__ double* x64(int g) const { return reinterpret_cast<double*>(base + g * per()); }
  __device__ double* s(int g) const { return reinterpret_cast<double*>(base + g * per() + 96 * (size_t)L); }
  __device__ int* prog() const { return reinterpret_cast<int*>(base + G * per()); }
  __device__ long long* nacc(int W) const { return reinterpret_cast<long long*>(prog() + ((W + 1) & ~1)); }
};

size_t local_lds_bytes(int G, int L, int W) {
  return (size_t)G * chain_stride(L) + 4 * (size_t)((W + 1) & ~1) + 8 * (size_t)W * G;
}

// The LDS that bounds which shapes (chains and wavefronts per workgroup) a length admits:
// 128 L bytes a chain and its queues and partial sums.  The launches themselves need no
// more (local_lds_bytes, global_lds_bytes).
size_t sweep_lds_bytes(int G, int L, int W) {
  const size_t b = 128 * (size_t)L, per = b + ((64 + 256 - (b & 255)) & 255);
  return (size_t)G * per + 208 * (size_t)G + 16 * (size_t)W * G + 128 * (size_t)G + 8 * (size_t)G +
         4 * (size_t)((W + 1) & ~1) + 8 * (size_t)W * G + 64 + 16 + 512 * (size_t)W +
         16 * (size_t)G * ((L + 7) / 8) + 24 * (size_t)G;
}

__device__ __forceinline__ void axis_atoms(const double* x64, int k, D3& A, D3& B) {
  const int c = k >> 1;
  if (k & 1) { A = ld3(atom(x64, c, 1)); B = ld3(atom(x64, c, 2)); }  // psi_c: CA_c -> C_c
  else { A = ld3(atom(x64, c, 0)); B = ld3(atom(x64, c, 1)); }        // phi_c: N_c -> CA_c
}

// Window half-width of localized sweep t: window_d, then the cascade radii in turn
// (Sec. 2.2 allows several localization ranges).
__device__ __forceinline__ int half_window_at(const SweepParams& P, int64_t t) {
  if (P.n_cascade == 0) return P.half_window;
  const int r = (int)((uint32_t)t % (uint32_t)(1 + P.n_cascade));   // t < 2^32
  return r == 0 ? P.half_window : r == 1 ? P.cascade_hw[0] : r == 2 ? P.cascade_hw[1] : P.cascade_hw[2];
}

// Localized sweeps run all chains of a workgroup side by side in one wavefront:
// chain q owns the LW = 64 / G lanes [q LW, (q + 1) LW), and every chain is at the
// same proposal k of the same sweep, so the window bounds are uniform and only the
// geometry differs between the lane groups.  The wavefronts of a workgroup are
// consecutive sweeps of a block, pipelined.
//
// Pipelining: the m-th sweep of a block of consecutive localized sweeps publishes
// m * 4096 + (proposals done) in `publish`; sweep m+1 waits on that counter so that
// it runs proposal k' (residue c') only once sweep m stands at residue c'+2h+1 or
// beyond.  A localized dE depends only on the geometry of its window, and a
// rotation moves only residues downstream of its bond, so the two sweeps never
// touch the same residues and the results equal those of running them in turn.
struct Pipe {
  const int* wait_on;   // progress counter of the previous sweep, or null
  int* publish;         // this sweep's progress counter
  int m;                // index of the sweep in its block
};

// Waits until *ctr >= target and returns the value seen (bounded: on a stall the
// error word is flagged and the sweep goes on rather than hang).
__device__ __forceinline__ int wait_progress(const SweepParams& P, const int* ctr, int target,
                                             bool& stalled) {
  if (stalled) return 0x7fffffff;
  for (int spin = 0; spin < P.spin_limit; ++spin) {
    const int v = __hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (v >= target) return v;
    __builtin_amdgcn_s_sleep(2);
  }
  stalled = true;
  atomicOr(P.err, kErrStall);
  return 0x7fffffff;
}

// Value of lane (q LW + kl) for the lanes of chain group q (kl uniform).
template <int LW>
__device__ __forceinline__ double group_bcast(double v, int lane, int kl) {
  if constexpr (LW == 64) {
    return readlane_d(v, kl);
  } else {
    const int src = ((lane & ~(LW - 1)) + kl) << 2;
    const int lo = __builtin_amdgcn_ds_bpermute(src, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(src, __double2hiint(v));
    return __hiloint2double(hi, lo);
  }
}

// Sum over the LW lanes of each chain group; every lane of a group gets its group's
// sum.  The addends are multiples of 2^-30 below 2^23 in magnitude, so every partial
// sum is exact and the result does not depend on LW or on the order.
template <int LW>
__device__ __forceinline__ double group_sum(double v, int lane) {
  v += dpp_d<kDppXor1>(v);
  v += dpp_d<kDppXor2>(v);
  v += dpp_d<kDppRor4>(v);
  v += dpp_d<kDppRor8>(v);   // every lane: the sum of its row of 16
  if constexpr (LW == 16) {
    return v;
  } else if constexpr (LW == 32) {
    const double a = readlane_d(v, 0) + readlane_d(v, 16), b = readlane_d(v, 32) + readlane_d(v, 48);
    return lane < 32 ? a : b;
  } else {
    return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
  }
}

// One localized sweep of the workgroup's chains (G of them, nact active) by one
// wavefront, with no workgroup barrier inside.
template <int G>
__device__ void local_sweep(const SweepParams& P, const Lds& S, int nact, int c0, int64_t t,
                            double beta, int h, int h_prev, int lane, int slot, int64_t& n_acc,
                            const Pipe& pipe, bool& stalled) {
  constexpr int LW = 64 / G;   // lanes per chain
  constexpr int R = G > 2 ? 3 : G;   // pair slots per lane: LW R pairs per pass (48 at G = 4)
  const int L = P.L, n = 2 * L;
  const int q = lane / LW, ll = lane - q * LW;
  const bool act = q < nact;
  double* __restrict__ x64 = S.x64(q);
  double* __restrict__ s = S.s(q);
  const uint32_t chain = (uint32_t)(P.chain_offset + c0 + q);
  const Spline32 sp{P.inv_w, P.off, P.tmax};
  // accumulated rigid transform x -> A x + b of the residues that have not yet
  // entered the window (float64, uniform over the chain's lanes)
  double A[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, tb[3] = {0, 0, 0};
  bool moved = false;
  int entered = h < L - 1 ? h : L - 1;
  int seen = -1;   // progress of the previous sweep last read
  Batch bt{};
  for (int k = 0; k < n; ++k) {
    const int kl = k & (LW - 1);
    if (kl == 0) bt = fill_batch(P, k, (uint32_t)t, chain, ll);
    // this proposal's randoms from the lane of the chain that drew them
    const double cd = group_bcast<LW>(bt.cd, lane, kl), sd = group_bcast<LW>(bt.sd, lane, kl);
    const double log_u = group_bcast<LW>(bt.log_u, lane, kl), delta = group_bcast<LW>(bt.delta, lane, kl);
    const int c = k >> 1, p = (k & 1) ? c + 1 : c;
    const int lo = c - h > 0 ? c - h : 0, hi = c + h < L - 1 ? c + h : L - 1;
    if (pipe.wait_on) {
      // the previous sweep (half-width h_prev) must be done with every proposal whose
      // window reaches residue c + h, i.e. with all proposals up to c' = c + h + h_prev
      const int need = (pipe.m - 1) * 4096 +
                       (2 * (c + h + h_prev) + 2 < n ? 2 * (c + h + h_prev) + 2 : n);
      if (seen < need) seen = wait_progress(P, pipe.wait_on, need, stalled);
    }
    // residues entering the window take the transform accumulated so far
    while (entered < hi) {
      ++entered;
      if (moved && ll < 4) {
        double* qa = atom(x64, entered, ll);
        const double X = qa[0], Y = qa[1], Z = qa[2];
        qa[0] = A[0] * X + A[1] * Y + A[2] * Z + tb[0];
        qa[1] = A[3] * X + A[4] * Y + A[5] * Z + tb[1];
        qa[2] = A[6] * X + A[7] * Y + A[8] * Z + tb[2];
      }
      wave_sync();
    }
    const bool live = k != 0 && k != n - 1;
    const int nF = p - lo > 0 ? p - lo : 0, nM = hi - p + 1 > 0 ? hi - p + 1 : 0;
    const int npair = live ? nF * nM : 0;
    // hardware reciprocal (1 ulp): floor((x + 1/2) inv_nM) stays exact for x < 2^22
    const float inv_nM = __builtin_amdgcn_rcpf((float)(nM > 0 ? nM : 1));
    double part = 0.0;
    Rot Rk;
    // the changed pairs (lo + a, p + b), a in [0, nF), b in [0, nM), in passes of LW R:
    // pair x = a nM + b sits in slot (x mod LW R) / LW of lane x mod LW.  The stencils
    // of the current distances are fetched before the rotation is set up; only the
    // stencils stay in registers, the coordinates are read again afterwards
    for (int x0 = 0; x0 < npair || x0 == 0; x0 += LW * R) {
      // branch-free over the slots, so that all their loads are in flight together:
      // an unused slot reads atoms of the window and the zero row
      int pr[R];   // (row residue << 16) | column residue of the slot's pair
      float4 q0[R];
      float f0[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int x = x0 + r * LW + ll;
        // floor((x + 1/2) / nM) is exact through the float reciprocal for x < 2^22
        const int a = (int)(((float)x + 0.5f) * inv_nM);
        const bool use = x < npair;
        const int ii = use ? lo + a : lo, j = use ? p + (x - a * nM) : p;
        pr[r] = (ii << 16) | j;
        const float d2 = use ? dist2_64(ld3(atom(x64, ii, 3)), ld3(atom(x64, j, 3))) : __builtin_inff();
        const float* row = P.ydev + (size_t)pair_row(ii, j, L) * P.stride;
        q0[r] = ld_stencil(stencil_addr(row, P.zrow, d2, sp, P.d2far, f0[r]));
      }
      if (x0 == 0 && live) {
        D3 a, b;
        axis_atoms(x64, k, a, b);
        make_rot(a, b, cd, sd, Rk);
      }
      float4 q1[R];
      float f1[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int ii = pr[r] >> 16, j = pr[r] & 0xffff;
        const float d2 = x0 + r * LW + ll < npair
                             ? dist2_64(ld3(atom(x64, ii, 3)), apply_rot(Rk, ld3(atom(x64, j, 3))))
                             : __builtin_inff();
        const float* row = P.ydev + (size_t)pair_row(ii, j, L) * P.stride;
        q1[r] = ld_stencil(stencil_addr(row, P.zrow, d2, sp, P.d2far, f1[r]));
      }
#pragma unroll
      for (int r = 0; r < R; ++r)
        part += fixed30_units(catmull_rom(q1[r].x, q1[r].y, q1[r].z, q1[r].w, f1[r])) -
                fixed30_units(catmull_rom(q0[r].x, q0[r].y, q0[r].z, q0[r].w, f0[r]));
    }
    const double dE = npair > 0 ? group_sum<LW>(act ? part : 0.0, lane) * (1.0 / 1073741824.0) : 0.0;
    const int acc = (dE <= 0.0) || (log_u < -beta * dE);
    if (act && ll == 0 && !isfinite(dE)) atomicOr(P.err, kErrEnergy);
    trace_step(P, act && ll == 0 ? slot : -1, t, k, dE, delta, acc);
    if (act && acc) {
      if (ll == 0) s[k] = wrap_angle(s[k] + delta);
      ++n_acc;
      if (live) {
        // rotate the atoms of the entered residues p..entered that the torsion moves,
        // two per lane at a time (both read before either is written)
        const int nat = 4 * (entered - p + 1);
        for (int x0 = 0; x0 < nat; x0 += 2 * LW) {
          const int xa = x0 + ll, xb = xa + LW;
          const int ya = xa < nat ? xa : nat - 1, yb = xb < nat ? xb : nat - 1;
          // phi_c leaves N_c and CA_c in place
          const bool va = xa < nat && ((k & 1) || xa >= 2), vb = xb < nat && ((k & 1) || xb >= 2);
          double* qa = atom(x64, p + (ya >> 2), ya & 3);
          double* qb = atom(x64, p + (yb >> 2), yb & 3);
          const D3 ra = apply_rot(Rk, ld3(qa)), rb = apply_rot(Rk, ld3(qb));
          if (va) st3(qa, ra);
          if (vb) st3(qb, rb);
        }
        // compose the pending transform: x -> R (x - a) + a after (A, b)
        double nA[9], nb[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
          for (int qq = 0; qq < 3; ++qq)
            nA[3 * r + qq] = Rk.r[3 * r] * A[qq] + Rk.r[3 * r + 1] * A[3 + qq] + Rk.r[3 * r + 2] * A[6 + qq];
          nb[r] = Rk.r[3 * r] * (tb[0] - Rk.a[0]) + Rk.r[3 * r + 1] * (tb[1] - Rk.a[1]) +
                  Rk.r[3 * r + 2] * (tb[2] - Rk.a[2]) + Rk.a[r];
        }
#pragma unroll
        for (int qq = 0; qq < 9; ++qq) A[qq] = nA[qq];
        tb[0] = nb[0]; tb[1] = nb[1]; tb[2] = nb[2];
        moved = true;
      }
    }
    wave_sync();
    if (pipe.publish && lane == 0)
      __hip_atomic_store(pipe.publish, pipe.m * 4096 + k + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// The localized sweeps [P.t0, P.t0 + P.n_sweeps) of one workgroup: chains group G ..
// group G + G - 1 of the protein that P describes.  Every wavefront runs all chains of
// the workgroup (64 / G lanes each); the W wavefronts run the consecutive sweeps in turn,
// pipelined.
template <int G>
__device__ __forceinline__ void local_body(const SweepParams& P, const int group) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, W = T >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = P.L, n = 2 * L;
  const int c0 = group * G;
  const int nact = P.C - c0 < G ? P.C - c0 : G;
  const Lds S{lds, L, G};

  // load chain state
  for (int e = tid; e < nact * L * 12; e += T) {
    const int g = e / (12 * L), q = e - g * 12 * L;
    S.x64(g)[q] = P.atoms[(size_t)(c0 + g) * L * 12 + q];
  }
  for (int e = tid; e < nact * n; e += T) {
    const int g = e / n, m = e % n;
    S.s(g)[m] = P.s[(size_t)(c0 + g) * n + m];
  }
  // the slots of absent chains (a last workgroup with nact < G) hold zeros: their
  // lanes compute on them without any effect
  for (int e = tid; e < (G - nact) * L * 12; e += T) {
    const int g = nact + e / (12 * L);
    S.x64(g)[e - (g - nact) * 12 * L] = 0.0;
  }
  const int lslot = (lane / (64 / G)) < nact ? trace_slot(P, c0 + lane / (64 / G)) : -1;
  int64_t acc_stage = 0;   // accepted proposals of this lane's chain
  bool stalled = false;
  // blocks of at most 4096 sweeps (the progress counters' range)
  for (int64_t t = P.t0, t_end = P.t0 + P.n_sweeps; t < t_end;) {
    const int nblk = t_end - t < 4096 ? (int)(t_end - t) : 4096;
    for (int e = tid; e < W; e += T) S.prog()[e] = 0;
    __syncthreads();
    for (int m = wave; m < nblk; m += W) {
      const int64_t tm = t + m;
      double Tm = P.T0;
      if (P.S > 1) Tm = P.T0 * pow(P.T1 / P.T0, (double)tm / (double)(P.S - 1));
      Pipe pipe;
      pipe.m = m;
      pipe.publish = S.prog() + wave;
      pipe.wait_on = m > 0 ? S.prog() + ((m - 1) % W) : nullptr;
      local_sweep<G>(P, S, nact, c0, tm, 1.0 / Tm, half_window_at(P, tm),
                     tm > 0 ? half_window_at(P, tm - 1) : 0, lane, lslot, acc_stage, pipe, stalled);
    }
    __syncthreads();
    t += nblk;
  }
  // store chain state; the accept counts of a chain's wavefronts are summed
  if ((lane & (64 / G - 1)) == 0) S.nacc(W)[wave * G + lane / (64 / G)] = acc_stage;
  __syncthreads();
  if (tid < nact) {
    long long a = 0;
    for (int v = 0; v < W; ++v) a += S.nacc(W)[v * G + tid];
    P.counters[4 * (c0 + tid)] += a;
  }
  for (int e = tid; e < nact * L * 12; e += T) {
    const int g = e / (12 * L), q = e - g * 12 * L;
    P.atoms[(size_t)(c0 + g) * L * 12 + q] = S.x64(g)[q];
  }
  for (int e = tid; e < nact * n; e += T) {
    const int g = e / n, m = e % n;
    P.s[(size_t)(c0 + g) * n + m] = S.s(g)[m];
  }
}

template <int G>
__global__ __launch_bounds__(768) void local_kernel(SweepParams P) {
  local_body<G>(P, blockIdx.x);
}

// Several proteins in one launch: workgroup b runs chain group map[b].y of the
// protein described by descs[map[b].x] (the grid is ordered by decreasing work).
template <int G>
__global__ __launch_bounds__(768) void local_batch_kernel(const SweepParams* __restrict__ descs,
                                                          const int2* __restrict__ map) {
  const int2 wm = map[blockIdx.x];
  if (descs[wm.x].n_sweeps == 0) return;
  local_body<G>(descs[wm.x], wm.y);
}

template __global__ void local_kernel<1>(SweepParams);
template __global__ void local_kernel<2>(SweepParams);
template __global__ void local_kernel<4>(SweepParams);
template __global__ void local_batch_kernel<1>(const SweepParams*, const int2*);
template __global__ void local_batch_kernel<2>(const SweepParams*, const int2*);
template __global__ void local_batch_kernel<4>(const SweepParams*, const int2*);

}  // namespace amh
