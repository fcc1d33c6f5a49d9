// amh_kernels.hip -- HIP kernels of the Alternating Metropolis-Hastings sampler
// for MI355X (gfx950, wave64).
//
// Method (Ghantasala, Jaiswal, Datta, arXiv 2211.03193): single-torsion Gaussian
// proposals swept over k = 0 .. 2L-1 (Sec. 2.1, Algorithm 1), judged either by the
// full distogram energy V (global MH) or by the energy of the window of residues
// within d/2 of residue k/2 (localized MH, Sec. 2.3); global and localized sweeps
// alternate (Algorithm 1, Fig. 1); acceptance min(1, exp(-beta dE)) (Sec. 2.1).
//
// The localized sweeps are in amh_local.hip, the global ones in amh_global.hip, the gradient
// and L-BFGS in amh_grad.hip.  Here: the table's repacking, energies and coordinates of given
// conformations, and anchors.  After every anchor sweep the coordinates are rebuilt from the
// float64 torsions by NeRF and V is re-anchored in float64, so that neither the sweeps'
// rotations nor their float32 distances accumulate an error in the state (an extended
// 300-residue chain spans ~1000 A, where float32 resolves only ~6e-5 A).
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
// once from float64), flag non-finite entries, and leave each workgroup's largest magnitude in
// `dev` to far_sum_kernel (an atomic maximum of all wavefronts on one word took 65 us more).
__global__ void ingest_kernel(const float* __restrict__ y, int64_t P, int nb, int stride,
                              float* __restrict__ out, float* __restrict__ dev, float* __restrict__ most,
                              unsigned int* err) {
  __shared__ float wave_most[4];
  const int64_t n = P * (int64_t)stride;
  bool bad = false;
  float m = 0.0f;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / stride;
    const int c = (int)(e - r * stride);
    float v = 0.0f;
    if (c == 0) v = y[r * nb + 1];
    else if (c <= nb) v = y[r * nb + (c - 1)];
    else if (c == nb + 1) v = y[r * nb + (nb - 2)];
    if (c <= nb && !isfinite(v)) bad = true;
    const float d = c <= nb + 1 ? (float)((double)v - (double)y[r * nb + (nb - 1)]) : 0.0f;
    out[e] = v;
    dev[e] = d;
    m = fmaxf(m, fabsf(d));
  }
  if (bad) atomicOr(err, kErrTable);
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) wave_most[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) most[blockIdx.x] = fmaxf(fmaxf(wave_most[0], wave_most[1]), fmaxf(wave_most[2], wave_most[3]));
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
// is one wavefront step, a pair per lane, tested in float64; the pairs inside go to the
// wavefront's queue, which is evaluated 64 at a time (about one lane in five of a tile holds
// one, and a spline takes three times the instructions of a test).  Each pair term is
// rounded to a multiple of 2^-40 (error < 5e-13 per pair) and summed as an integer,
// exactly and so in any order: V does not depend on the launch shape.  acc is one 64-bit
// integer in LDS, queue EnergyQueue[wavefronts]; every thread returns V.
// Evaluated tile by tile, under the test's mask, 1024 conformations of 300 residues took
// 195 us with their coordinates, now 160; alone (16 wavefronts) 42 us above its coordinates',
// now 13.
__device__ double energy64(const float* __restrict__ table, int stride, int nb, double d_min, double w,
                           double vfar, int L, const double* __restrict__ x, float4* __restrict__ sph,
                           long long* acc, EnergyQueue* __restrict__ queue) {
  const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, wave = tid >> 6, W = T >> 6;
  const double dfar = d_min + w * ((double)nb - 0.5), d2far = dfar * dfar;   // the last knot
  const double inv_w = 1.0 / w;
  const float rcut = (float)dfar + 0.05f;
  const int nb8 = (L + 7) >> 3;
  if (tid == 0) *acc = 0;
  block_spheres(x, L, sph);
  __syncthreads();
  long long part = 0;
  int fill = 0;   // pairs in the wavefront's queue (uniform)
  EnergyQueue& q = queue[wave];
  auto flush = [&](int nq) {   // evaluate the queue's last nq pairs, one per lane
    fill -= nq;
    wave_sync();
    if (lane < nq) {
      const double d2 = q.d2[fill + lane];
      const unsigned int c = q.code[fill + lane];
      const float* row = table + (size_t)pair_row((int)(c >> 10), (int)(c & 1023u), L) * stride;
      // distance through the hardware reciprocal square root and two Newton steps
      const double e = spline64(row, d2 * rsqrt64(d2), nb, d_min, w, inv_w) - (double)row[nb];
      part += (long long)rint(e * 1099511627776.0);   // e 2^40
    }
    wave_sync();
  };
  // candidate tiles (row block I, column block J), I <= J, one per thread, dealt to the
  // wavefronts in turn: row blocks r and nb8 - 1 - r together have nb8 + 1
  const int lr = lane >> 3, lc = lane & 7, cols = nb8 + 1, ncand = cols * ((nb8 + 1) >> 1);
  const float inv_cols = 1.0f / (float)cols;
  for (int base = 0; base < ncand; base += T) {
    const int cand = base + lane * W + wave;
    const int r = (int)(((float)cand + 0.5f) * inv_cols), c = cand - r * cols;
    const bool low = c < nb8 - r;
    const int I = low ? r : nb8 - 1 - r, J = low ? r + c : c - 1;
    bool keep = cand < ncand && (low || I > r);
    if (keep) {
      const float4 u = sph[I], v = sph[J];
      const float dx = u.x - v.x, dy = u.y - v.y, dz = u.z - v.z, lim = rcut + u.w + v.w;
      keep = dx * dx + dy * dy + dz * dz <= lim * lim;
    }
    const int code = (I << 10) | J;
    unsigned long long m = __ballot(keep);
    while (m) {
      const int l = __builtin_ctzll(m);
      m &= m - 1;
      const int cd = __builtin_amdgcn_readlane(code, l);
      const int i = 8 * (cd >> 10) + lr, j = 8 * (cd & 1023) + lc;
      bool near = false;
      double d2 = 0.0;
      if (i < j && j < L) {
        const double* pa = atom(x, i, 3);
        const double* pb = atom(x, j, 3);
        const double dx = pb[0] - pa[0], dy = pb[1] - pa[1], dz = pb[2] - pa[2];
        d2 = dx * dx + dy * dy + dz * dz;
        near = d2 < d2far;
      }
      const unsigned long long bal = __ballot(near);
      if (near) {
        const unsigned at = __builtin_amdgcn_mbcnt_hi((unsigned int)(bal >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((unsigned int)bal, (unsigned)fill));
        q.d2[at] = d2;
        q.code[at] = (unsigned)((i << 10) | j);
      }
      fill += (int)__popcll(bal);
      if (fill >= 64) flush(64);
    }
  }
  if (fill > 0) flush(fill);
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
// combined in thread order by thread 0.  And the largest of ingest_kernel's n_most maxima.
__global__ void far_sum_kernel(const float* __restrict__ table, int64_t P, int stride, int nb,
                               const float* __restrict__ most, int n_most, double* __restrict__ out,
                               float* __restrict__ dev_max) {
  __shared__ double part[2 * 1024];
  __shared__ float wave_most[16];
  const int tid = threadIdx.x, T = blockDim.x;
  double s = 0.0, c = 0.0;
  for (int64_t r = tid; r < P; r += T) neumaier_add(s, c, (double)table[r * stride + nb]);
  part[2 * tid] = s;
  part[2 * tid + 1] = c;
  float m = 0.0f;
  for (int q = tid; q < n_most; q += T) m = fmaxf(m, most[q]);
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((tid & 63) == 0) wave_most[tid >> 6] = m;
  __syncthreads();
  if (tid == 0) {
    double a = 0.0, b = 0.0;
    for (int t = 0; t < T; ++t) { neumaier_add(a, b, part[2 * t]); b += part[2 * t + 1]; }
    *out = a + b;
    for (int w = 1; w < T >> 6; ++w) m = fmaxf(m, wave_most[w]);
    *dev_max = m;
  }
}

// Conformation / energy kernel: one workgroup per conformation.
__global__ __launch_bounds__(1024) void conf_energy_kernel(ConfParams P) {
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
                               reinterpret_cast<long long*>(acc), reinterpret_cast<EnergyQueue*>(fr));
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
                            reinterpret_cast<long long*>(acc), reinterpret_cast<EnergyQueue*>(fr));
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

__global__ __launch_bounds__(1024) void anchor_kernel(SweepParams P) { anchor_body(P, blockIdx.x); }

// Several proteins: workgroup (b, q) anchors chain q of group map[b].y of its protein, of
// those whose descriptor asks for it (n_sweeps != 0).
__global__ __launch_bounds__(1024) void anchor_batch_kernel(const SweepParams* __restrict__ descs,
                                                           const int2* __restrict__ map, int G) {
  const int2 wm = map[blockIdx.x];
  const SweepParams& P = descs[wm.x];
  const int chain = wm.y * G + (int)blockIdx.y;
  if (P.n_sweeps == 0 || chain >= P.C) return;
  anchor_body(P, chain);
}

// ---------------------------------------------------------------------------
// The rule for which shapes (chains and wavefronts per workgroup) a length admits, kept so that what
// was accepted and refused stays so: 128 L bytes a chain and queues and partial sums, as much as
// a kernel needs that holds all atoms of its chains for localized and global sweeps alike.  It
// is no bound of what the launches take (a global one of a short chain takes more, for its
// queues and its helper): that is checked by itself (local_lds_bytes, global_lds_bytes).
size_t sweep_lds_bytes(int G, int L, int W) {
  const size_t b = 128 * (size_t)L, per = b + ((64 + 256 - (b & 255)) & 255);
  return (size_t)G * per + 208 * (size_t)G + 16 * (size_t)W * G + 128 * (size_t)G + 8 * (size_t)G +
         4 * (size_t)((W + 1) & ~1) + 8 * (size_t)W * G + 64 + 16 + 512 * (size_t)W +
         16 * (size_t)G * ((L + 7) / 8) + 24 * (size_t)G;
}

}  // namespace amh
