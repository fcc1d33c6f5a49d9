// amh_geom.h -- float64 chain geometry shared by the sweep, energy and gradient
// kernels: the atom layout [L][4][3] (N, CA, C, C-beta) and the NeRF build of a
// chain from its torsions.
#pragma once
#include <hip/hip_runtime.h>

#include "amh_device.h"

namespace amh {

constexpr double kDeg = kPi / 180.0;

__device__ __forceinline__ double* atom(double* x64, int r, int a) { return x64 + (4 * r + a) * 3; }
__device__ __forceinline__ const double* atom(const double* x64, int r, int a) {
  return x64 + (4 * r + a) * 3;
}

// ---------------------------------------------------------------------------
// Float64 NeRF of one chain by a whole workgroup, in parallel over the atoms
// (Parsons et al. 2005 placement; the parallel form of AlQuraishi's pNeRF).  Backbone
// atom a_k (k >= 3: N, CA, C of residue k/3) is placed from a_{k-3}, a_{k-2}, a_{k-1}
// in the frame (e1 = unit(a_{k-1} - a_{k-2}), n = unit((a_{k-2} - a_{k-3}) x e1),
// m = n x e1) at a_{k-1}: a_k = a_{k-1} + F (l (-cos t, sin t cos x, sin t sin x)),
// F = [e1 m n], with bond l, angle t and torsion x of atom k.  The frame of atom k+1
// is then F R_k with
//   R_k = [[-cos t, -sin t, 0], [sin t cos x, -cos t cos x, -sin x],
//          [sin t sin x, -cos t sin x, cos x]],
// which depends only on (t, x), so every frame is a prefix product of the rigid
// transforms (R_k, l R_k e_1) (composition (R, u) o (R', u') = (R R', u + R u')).  The
// transforms go 64 to a block, one per lane, and each block is scanned across its
// wavefront's lanes (Hillis-Steele, six steps), the blocks dealt to the wavefronts in
// turn; one wavefront then carries the frame from block to block (one composition
// each), and every atom follows from its block's frame; C-beta follows per residue from
// its N, CA, C.  The scan is nearly all of the work (72 lane exchanges and six dependent
// 3x3 products a block), so it is shared by the wavefronts; the values do not depend on
// how many there are.  The rounding differs from a serial build only at the last bits
// (about 1e-13 of the chain's extent).
//
// x64 [12L] and fr [nerf_scratch(L)] are in LDS, s [2L] anywhere; s is complete (a barrier
// if the workgroup wrote it) and nobody uses fr; ends with a barrier of the workgroup.
__host__ __device__ inline int nerf_scratch(int L) { return 12 * ((3 * (L - 1) + 63) / 64); }

__device__ __forceinline__ void nerf_wg(const double* __restrict__ s, int L, double* __restrict__ x64,
                               double* __restrict__ fr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
  const double ct_cacn = cos(kAngCACN * kDeg), st_cacn = sin(kAngCACN * kDeg);
  const double ct_cnca = cos(kAngCNCA * kDeg), st_cnca = sin(kAngCNCA * kDeg);
  const double ct_ncac = cos(kAngNCAC * kDeg), st_ncac = sin(kAngNCAC * kDeg);
  const double ct_ncacb = cos(kAngNCACB * kDeg), st_ncacb = sin(kAngNCACB * kDeg);
  const double co = cos(kTorOmega * kDeg), so = sin(kTorOmega * kDeg);
  const double ccb = cos(kTorCB * kDeg), scb = sin(kTorCB * kDeg);
  // residue 0: N at the origin, CA on +x, C in the xy-plane
  const double N0[3] = {0.0, 0.0, 0.0};
  const double CA0[3] = {kBondNCA, 0.0, 0.0};
  const double C0[3] = {kBondNCA - kBondCAC * ct_ncac, kBondCAC * st_ncac, 0.0};
  if (wave == 0 && lane < 9)
    atom(x64, 0, lane / 3)[lane % 3] = lane < 3 ? N0[lane] : lane < 6 ? CA0[lane - 3] : C0[lane - 6];
  const int nt = 3 * (L - 1), nblk = (nt + 63) >> 6;   // placed backbone atoms and their blocks
  for (int blk = wave; blk < nblk; blk += W) {
    const int k0 = 64 * blk, j = k0 + lane, k = 3 + j, kind = k % 3, c = k / 3;
    // this lane's transform (absent lanes: the identity)
    double ct = 1.0, st = 0.0, l = 0.0, cx = 1.0, sx = 0.0;
    if (j < nt) {
      if (kind == 1) {
        ct = ct_cnca; st = st_cnca; l = kBondNCA; cx = co; sx = so;
      } else {
        ct = kind == 0 ? ct_cacn : ct_ncac;
        st = kind == 0 ? st_cacn : st_ncac;
        l = kind == 0 ? kBondCN : kBondCAC;
        sincos(s[kind == 0 ? 2 * c - 1 : 2 * c], &sx, &cx);
      }
    }
    double R[9], u[3];
    if (j < nt) {
      R[0] = -ct;      R[1] = -st;      R[2] = 0.0;
      R[3] = st * cx;  R[4] = -ct * cx; R[5] = -sx;
      R[6] = st * sx;  R[7] = -ct * sx; R[8] = cx;
    } else {
      R[0] = 1.0; R[1] = 0.0; R[2] = 0.0; R[3] = 0.0; R[4] = 1.0; R[5] = 0.0; R[6] = 0.0; R[7] = 0.0; R[8] = 1.0;
    }
    u[0] = l * R[0]; u[1] = l * R[3]; u[2] = l * R[6];
    // inclusive scan over the lanes: (R, u) <- (R, u) of lane - off  o  (R, u)
    for (int off = 1; off < 64; off <<= 1) {
      double Rp[9], up[3];
#pragma unroll
      for (int q = 0; q < 9; ++q) Rp[q] = __shfl_up(R[q], off, 64);
#pragma unroll
      for (int q = 0; q < 3; ++q) up[q] = __shfl_up(u[q], off, 64);
      if (lane >= off) {
        double Rn[9], un[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
          for (int q = 0; q < 3; ++q) Rn[3 * r + q] = row3(Rp + 3 * r, R[q], R[3 + q], R[6 + q]);
          un[r] = row3(up[r], Rp + 3 * r, u[0], u[1], u[2]);
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) R[q] = Rn[q];
        u[0] = un[0]; u[1] = un[1]; u[2] = un[2];
      }
    }
    // the atom in its block's frame, and the block's transform
    if (j < nt) {
      double* x = atom(x64, c, kind);
      x[0] = u[0]; x[1] = u[1]; x[2] = u[2];
    }
    if (lane == 63 || j == nt - 1) {
      double* o = fr + 12 * blk;
#pragma unroll
      for (int q = 0; q < 9; ++q) o[q] = R[q];
      o[9] = u[0]; o[10] = u[1]; o[11] = u[2];
    }
  }
  __syncthreads();
  if (wave == 0) {
    // frame of atom 3 (N_1): from N_0, CA_0, C_0, origin C_0 (uniform over the lanes)
    double F[9], o[3];
    double bx = C0[0] - CA0[0], by = C0[1] - CA0[1], bz = C0[2] - CA0[2];
    const double ib = 1.0 / sqrt(bx * bx + by * by + bz * bz);
    bx *= ib; by *= ib; bz *= ib;
    const double ax = CA0[0] - N0[0], ay = CA0[1] - N0[1], az = CA0[2] - N0[2];
    double nx = ay * bz - az * by, ny = az * bx - ax * bz, nz = ax * by - ay * bx;
    const double in = 1.0 / sqrt(nx * nx + ny * ny + nz * nz);
    nx *= in; ny *= in; nz *= in;
    const double mx = ny * bz - nz * by, my = nz * bx - nx * bz, mz = nx * by - ny * bx;
    F[0] = bx; F[1] = mx; F[2] = nx;
    F[3] = by; F[4] = my; F[5] = ny;
    F[6] = bz; F[7] = mz; F[8] = nz;
    o[0] = C0[0]; o[1] = C0[1]; o[2] = C0[2];
    double T[12], Tn[12];   // the block's transform and the next block's, read one ahead
#pragma unroll
    for (int q = 0; q < 12; ++q) T[q] = fr[q];
    for (int blk = 0; blk < nblk; ++blk) {
      if (blk + 1 < nblk) {
#pragma unroll
        for (int q = 0; q < 12; ++q) Tn[q] = fr[12 * (blk + 1) + q];
      }
      wave_sync();
      if (lane == 0) {   // the block's frame takes the transform's place
        double* w = fr + 12 * blk;
#pragma unroll
        for (int q = 0; q < 9; ++q) w[q] = F[q];
        w[9] = o[0]; w[10] = o[1]; w[11] = o[2];
      }
      double Fn[9], on[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int q = 0; q < 3; ++q) Fn[3 * r + q] = row3(F + 3 * r, T[q], T[3 + q], T[6 + q]);
        on[r] = row3(o[r], F + 3 * r, T[9], T[10], T[11]);
      }
#pragma unroll
      for (int q = 0; q < 9; ++q) F[q] = Fn[q];
      o[0] = on[0]; o[1] = on[1]; o[2] = on[2];
#pragma unroll
      for (int q = 0; q < 12; ++q) T[q] = Tn[q];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nt; j += blockDim.x) {
    const double* F = fr + 12 * (j >> 6);
    double* x = atom(x64, (3 + j) / 3, j % 3);
    const double u0 = x[0], u1 = x[1], u2 = x[2];
#pragma unroll
    for (int r = 0; r < 3; ++r) x[r] = row3(F[9 + r], F + 3 * r, u0, u1, u2);
  }
  __syncthreads();
  // C-beta of residue c from C_c, N_c, CA_c (one residue per thread)
  for (int c = threadIdx.x; c < L; c += blockDim.x) {
    const double* pN = atom(x64, c, 0);
    const double* pCA = atom(x64, c, 1);
    const double* pC = atom(x64, c, 2);
    const double Nc[3] = {pN[0], pN[1], pN[2]}, CAc[3] = {pCA[0], pCA[1], pCA[2]}, Cc[3] = {pC[0], pC[1], pC[2]};
    double B[3];
    nerf_place(Cc, Nc, CAc, kBondCACB, ct_ncacb, st_ncacb, ccb, scb, B);
    double* pB = atom(x64, c, 3);
    pB[0] = B[0]; pB[1] = B[1]; pB[2] = B[2];
  }
  __syncthreads();
}

// Bounding spheres (centroid, radius; float32) of the C-betas of every block of 8 residues,
// by the workgroup: a block in 8 aligned lanes of one wavefront.  x64 is complete; the
// caller's next barrier publishes sph.
__device__ __forceinline__ void block_spheres(const double* __restrict__ x64, int L, float4* __restrict__ sph) {
  const int nres8 = 8 * ((L + 7) >> 3);
  for (int r0 = 0; r0 < nres8; r0 += blockDim.x) {
    const int r = r0 + threadIdx.x;
    const bool real = r < L;
    float vx = 0.0f, vy = 0.0f, vz = 0.0f;
    if (real) {
      const double* q = atom(x64, r, 3);
      vx = (float)q[0]; vy = (float)q[1]; vz = (float)q[2];
    }
    const float cnt = sum8(real ? 1.0f : 0.0f), inv = __builtin_amdgcn_rcpf(cnt > 1.0f ? cnt : 1.0f);
    const float cx = sum8(vx) * inv, cy = sum8(vy) * inv, cz = sum8(vz) * inv;
    const float rad = max8(real ? __builtin_amdgcn_sqrtf((vx - cx) * (vx - cx) + (vy - cy) * (vy - cy) +
                                                         (vz - cz) * (vz - cz))
                                : 0.0f);
    if (r < nres8 && (r & 7) == 0) sph[r >> 3] = make_float4(cx, cy, cz, rad);
  }
}

}  // namespace amh
