// amh_global.hip -- global sweeps of the Alternating Metropolis-Hastings sampler for
// MI355X (gfx950, wave64): every proposal is judged by the full distogram energy
// (global MH, Sec. 2.1 and Algorithm 1 of arXiv 2211.03193).
//
// A proposal is a serial step (its rotation axis and its energy depend on the previous
// decision), so a sweep is a chain of 2L short phases, bound by the latency of each phase
// (LDS reads, dependent float64 operations, gathers), not by bandwidth: the kernel keeps
// the phases few and several independent steps in flight in each.
//   * NW wavefronts advance one chain, two workgroup barriers a proposal:
//       B  the trial conformation (float32 C-beta, bounding spheres) is written to LDS;
//       C  the changed pairs i < p <= j are scored, the partial sums written to LDS;
//          one wavefront, the helper, prepares the next proposal's rotation, for both
//          outcomes of this one
//       D  every wavefront takes the same decision from the same sums, reads the next
//          rotation and commits the C-betas it owns; B follows at once.
//   * LDS holds only what the pair loop reads: float64 and float32 C-betas, spheres,
//     queues.  N, CA and C are not rotated at every accepted move: the helper carries the
//     composition x -> A x + b of the moves accepted so far in the sweep, applies it to
//     the backbone atoms of the residues the sweep has reached (read from HBM, 21 residues
//     at a time, one atom per lane) and writes them back once final.
//   * pair energies are deviations from the pair's no-contact value, exactly zero beyond
//     the last knot; dE of pivot p is D_new(p) - D(p), where D(p), the deviation energy
//     of the pair rectangle i < p <= j, is carried from proposal to proposal (the new
//     sum on accept, an O(L) row and column when p advances).
//   * the rectangle is walked in 8 x 8 tiles; a tile whose two bounding spheres lie
//     farther apart than the last knot (plus a margin far above float32 rounding) holds
//     only pairs that add exactly zero and is skipped whole.
//   * every pair term is rounded to a multiple of 2^-30 and summed in float64 as an
//     integer count of these, exactly and so in any order: the sums do not depend on the
//     launch shape.
// Measured against global sweeps that rotated all atoms in LDS (128 bytes a residue), took
// one tile at a time and wrote the next rotation after the decision, with a third barrier:
// 1024 chains of 300 residues (2 chains and 4 wavefronts a workgroup) 6.8 -> 4.5 ms a
// sweep; 128 chains of 300 (8 wavefronts a chain) 2.9 -> 2.0 ms; 64 of 800 27.7 -> 18.9 ms;
// one of 64 residues 370 -> 242 us.  Most of it is instructions: a tile took 55 issued
// instructions of one wavefront at a time, now 25.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amh_device.h"
#include "amh_geom.h"
#include "amh_kernels.h"
#include "amh_proposal.h"

namespace amh {

typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

constexpr int kQueue = 320;       // near pairs a wavefront's queue holds (63 + four tiles at most)
constexpr int kList = 68;         // surviving tiles a wavefront's list holds (3 + one per lane at most)
constexpr int kWindowAtoms = 63;  // backbone atoms in the helper's window (21 residues)

// What the helper prepares for the next proposal: its rotation (matrix and point on the
// axis) if the current one is rejected and if it is accepted, and its randoms.
struct Slot {
  double rot[2][12];
  double log_u, delta;
};
static_assert(sizeof(Slot) == 208, "Slot layout");

// LDS of one chain: float64 C-betas (x, y, z arrays), float32 C-betas of the trial
// conformation (with two more blocks of 8: the fixed rows of the pivot's block, and one
// that is far from everything), spheres, the slot, partial sums, near-pair queues and
// tile lists.
__host__ __device__ inline size_t global_chain_bytes(int L, int NW) {
  const size_t nb8 = (size_t)((L + 7) >> 3);
  return nb8 * (8 * 24 + 8 * 16 + 16) + (16 * 16 + 16) + sizeof(Slot) + 8 * 64 + (8 * (size_t)kQueue + 4 * kList) * NW;
}

size_t global_lds_bytes(int G, int L, int NW) { return (size_t)G * global_chain_bytes(L, NW); }

// acc (lanes 0-31) and tr (lanes 32-63) halves added across the wavefront: lane l < 32
// gets acc[l] + acc[l + 32], lane l >= 32 gets tr[l - 32] + tr[l].
__device__ __forceinline__ double fold_halves(double acc, double tr) {
  const uint2v lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(acc), (unsigned)__double2loint(tr),
                                                     false, false);
  const uint2v hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(acc), (unsigned)__double2hiint(tr),
                                                     false, false);
  return __hiloint2double((int)hi.x, (int)lo.x) + __hiloint2double((int)hi.y, (int)lo.y);
}

// Workgroup barrier that orders LDS only: loads and stores of global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The global sweeps [P.t0, P.t0 + P.n_sweeps) of chains group G .. group G + G - 1 of the
// protein that P describes, NW wavefronts a chain.
template <int NW>
__device__ __forceinline__ void global_body(const SweepParams& P, const int group, const int G) {
  extern __shared__ __align__(16) unsigned char lds[];
  // From four wavefronts on the helper leaves the tiles to the others and takes the
  // transitions; below, the first wavefront takes them.
  constexpr int TW = NW >= 4 ? NW - 1 : NW;
  constexpr int kTransWave = NW >= 4 ? NW - 1 : 0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gi = wave / NW, wl = wave % NW;
  const int L = P.L, n = 2 * L, nb8 = (L + 7) >> 3, nres8 = 8 * nb8, nchunk = (L + 63) >> 6;
  const int chain = group * G + gi;
  const int64_t t_end = P.t0 + P.n_sweeps;
  if (gi >= G || chain >= P.C) {   // a wavefront without a chain only keeps the barriers
    for (int64_t t = P.t0; t < t_end; ++t) {
      lds_barrier();
      for (int k = 0; k < n; ++k) { lds_barrier(); lds_barrier(); }
      lds_barrier();
    }
    return;
  }
  unsigned char* const base = lds + (size_t)gi * global_chain_bytes(L, NW);
  double* const xb = reinterpret_cast<double*>(base);                  // [3][nres8]
  float4* const w32 = reinterpret_cast<float4*>(xb + 3 * nres8);       // [nres8 + 16]
  float4* const sph = w32 + nres8 + 16;                                // [nb8 + 1]
  Slot* const slot = reinterpret_cast<Slot*>(sph + nb8 + 1);
  double* const part = reinterpret_cast<double*>(slot + 1);            // [64]
  uint2* const qb = reinterpret_cast<uint2*>(part + 64) + kQueue * wl;
  unsigned int* const list = reinterpret_cast<unsigned int*>(reinterpret_cast<uint2*>(part + 64) + kQueue * NW) +
                             kList * wl;
  auto ldx = [&](int r) { return D3{xb[r], xb[nres8 + r], xb[2 * nres8 + r]}; };

  const Spline32 sp{P.inv_w, P.off, P.tmax};
  const bool helper = wl == NW - 1;
  double* const gatoms = P.atoms + (size_t)chain * L * 12;
  double* const gs = P.s + (size_t)chain * n;
  const int slot_id = trace_slot(P, chain);
  const float rcut = __builtin_amdgcn_sqrtf(P.d2far) + 0.05f;
  // absent columns and the columns before the pivot stand at kFar, absent rows at -kFar
  constexpr float kFar = 1e18f;
  // a step's four tiles take 16 lanes each; a lane has one row and four columns
  const unsigned int lane_pair = (unsigned int)((lane >> 1) & 7) | ((unsigned int)(4 * (lane & 1)) << 11);
  const unsigned int far_tile = (unsigned int)(nres8 + 8);   // (the far block's rows, the first columns)
  const bool count = P.work != nullptr;
  // sums of a wavefront's rows of 16 lanes: rows 0 and 1 the rectangle's, 2 and 3 the
  // transition's; part holds the former in its first half, the latter in its second
  constexpr int kHalf = NW == 16 ? 32 : 16;
  int n_acc = 0;
  unsigned int wk_tiles = 0, wk_tests = 0, wk_near = 0;   // executed work (tests: of this lane)

  for (int r = lane + 64 * wl; r < nres8; r += 64 * NW) {
    if (r < L) {
      const double* q = atom(gatoms, r, 3);
      xb[r] = q[0]; xb[nres8 + r] = q[1]; xb[2 * nres8 + r] = q[2];
    }
    w32[r] = make_float4(kFar, kFar, kFar, 0.0f);
  }
  if (wl == 0 && lane < 16) w32[nres8 + lane] = make_float4(-kFar, -kFar, -kFar, 0.0f);
  if (wl == 0) part[lane] = 0.0;
  for (int64_t t = P.t0; t < t_end; ++t) {
    double T_t = P.T0;
    if (P.S > 1) T_t = P.T0 * pow(P.T1 / P.T0, (double)t / (double)(P.S - 1));
    const double beta = 1.0 / T_t;
    double rp = 0.0;                                           // D(p) in units of 2^-30
    double A[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, tb[3] = {0, 0, 0};   // helper: accepted moves composed
    double bx = 0.0, by = 0.0, bz = 0.0;                       // helper: backbone atom of this lane
    int b0 = 0;                                                // first residue of the window
    double sv = 0.0;                                           // helper: torsion (k & ~63) + lane
    Batch bt{};
    Rot R;                                                     // of the current proposal
    double log_u = 0.0, delta = 0.0;                           // its randoms
    auto load_window = [&](int r0) {
      b0 = r0;
      const int m = 3 * r0 + lane;
      if (lane < kWindowAtoms && m < 3 * L) {
        const double* q = atom(gatoms, m / 3, m % 3);
        bx = q[0]; by = q[1]; bz = q[2];
      }
    };
    auto put = [&](double* o, const Rot& r) {
#pragma unroll
      for (int q = 0; q < 9; ++q) o[q] = r.r[q];
      o[9] = r.a[0]; o[10] = r.a[1]; o[11] = r.a[2];
    };
    auto get = [&](const double* o) {
#pragma unroll
      for (int q = 0; q < 9; ++q) R.r[q] = o[q];
      R.a[0] = o[9]; R.a[1] = o[10]; R.a[2] = o[11];
    };
    // proposal kn for the slot: (tx, ty, tz) hold the window's atoms in the conformation
    // that proposal kn - 1 starts from; `both`: also the rotation if kn - 1 (R) is accepted
    auto prepare = [&](int kn, double tx, double ty, double tz, bool both) {
      if ((kn & 63) == 0) bt = fill_batch(P, kn, (uint32_t)t, (uint32_t)(P.chain_offset + chain), lane);
      const int m = 3 * ((kn >> 1) - b0) + (kn & 1), kl = kn & 63;
      D3 a{readlane_d(tx, m), readlane_d(ty, m), readlane_d(tz, m)};
      const D3 e{readlane_d(tx, m + 1), readlane_d(ty, m + 1), readlane_d(tz, m + 1)};
      D3 u = unit(a, e);
      const double cd = readlane_d(bt.cd, kl), sd = readlane_d(bt.sd, kl);
      Rot q;
      make_rot_u(a, u, cd, sd, q);
      if (lane == 0) {
        put(slot->rot[0], q);
        slot->log_u = readlane_d(bt.log_u, kl);
        slot->delta = readlane_d(bt.delta, kl);
      }
      if (both) {
        // an accepted rotation turns the next bond rigidly: psi_c moves both atoms of
        // phi_{c+1}'s, phi_c the far atom of psi_c's (whose near atom CA_c is on its axis)
        if (!(kn & 1)) a = apply_rot(R, a);
        u = rot_dir(R, u);
        make_rot_u(a, u, cd, sd, q);
        if (lane == 0) put(slot->rot[1], q);
      }
    };
    if (helper) {
      load_window(0);
      prepare(0, bx, by, bz, false);
      if (lane < n) sv = gs[lane];
    }
    lds_barrier();
    // origin of the float32 work array for this sweep: the middle C-beta
    const D3 org = ldx(L / 2);
    get(slot->rot[0]);
    log_u = slot->log_u;
    delta = slot->delta;
    int pprev = 0;   // pivot of the previous proposal (0: refresh every residue)
    // the previous proposal's outcome, for the helper's bookkeeping
    double dE_prev = 0.0, delta_prev = 0.0;
    bool acc_prev = false;
    auto book = [&](int k) {   // of proposal k, by the helper
      if (acc_prev && lane == (k & 63)) sv = wrap_angle(sv + delta_prev);
      if (lane == 0) {
        if (!isfinite(dE_prev)) atomicOr(P.err, kErrEnergy);
        if (slot_id >= 0) trace_step(P, slot_id, t, k, dE_prev, delta_prev, acc_prev);
      }
      n_acc += acc_prev;
      if ((k & 63) == 63 || k == n - 1) {
        const int m = (k & ~63) + lane;
        if (m < n) gs[m] = sv;
        if (m + 64 < n) sv = gs[m + 64];
      }
    };
    unsigned int code0 = 0;       // this lane's first candidate tile, for blocks (I_code, J_code)
    int I_code = -1, J_code = -1;
    for (int k = 0; k < n; ++k) {
      const int c = k >> 1, odd = k & 1, p = c + odd;
      // [B] float32 C-beta of the trial conformation relative to the origin (residues
      // below the pivot as they are, the others rotated) and a bounding sphere (centroid,
      // radius) of every block of 8 residues, in chunks of 64 residues dealt to the
      // chain's wavefronts.  Residues below the previous pivot hold their committed
      // position already, so only the chunks from that of the previous pivot on.
      {
        const int c0 = pprev >> 6;
        for (int ch = c0 + ((wl - c0) & (NW - 1)); ch < nchunk; ch += NW) {
          const int r = 64 * ch + lane;
          const bool real = r < L;
          float vx = 0.0f, vy = 0.0f, vz = 0.0f;
          if (real) {
            D3 x = ldx(r);
            if (r >= p) x = apply_rot(R, x);
            vx = (float)(x.x - org.x); vy = (float)(x.y - org.y); vz = (float)(x.z - org.z);
          }
          if (ch == p >> 6 && (r >> 3) == p >> 3) {
            // the pivot's block: its fixed rows have a block of their own
            const bool row = r < p && real, col = r >= p && real;
            w32[nres8 + (r & 7)] = row ? make_float4(vx, vy, vz, 0.0f) : make_float4(-kFar, -kFar, -kFar, 0.0f);
            w32[r] = col ? make_float4(vx, vy, vz, 0.0f) : make_float4(kFar, kFar, kFar, 0.0f);
          } else if (real) {
            w32[r] = make_float4(vx, vy, vz, 0.0f);
          }
          // any centre will do (the radius is measured from it); the 0.05 A margin of the
          // tile test covers the 1-ulp hardware square root
          const float cnt = sum8(real ? 1.0f : 0.0f), inv = __builtin_amdgcn_rcpf(cnt > 1.0f ? cnt : 1.0f);
          const float cx = sum8(vx) * inv, cy = sum8(vy) * inv, cz = sum8(vz) * inv;
          const float rad = max8(real ? __builtin_amdgcn_sqrtf((vx - cx) * (vx - cx) + (vy - cy) * (vy - cy) +
                                                               (vz - cz) * (vz - cz))
                                      : 0.0f);
          if ((r & 7) == 0 && r < nres8) {
            sph[r >> 3] = make_float4(cx, cy, cz, rad);
            if ((r >> 3) == p >> 3) sph[nb8] = make_float4(cx, cy, cz, rad);
          }
        }
      }
      pprev = p;
      lds_barrier();
      // [C] the changed pairs of the trial conformation, and for odd k the row and column
      // that carry D from pivot p - 1 to p (current conformation): residue x against p - 1
      double acc = 0.0, tr = 0.0;
      const bool pairs = p > 0 && p < L;
      if (helper) {
        if (k > 0) book(k - 1);
        if (!odd && c + 1 > b0 + 20 && c + 1 < L) load_window(c);
        const double tx = A[0] * bx + A[1] * by + A[2] * bz + tb[0];
        const double ty = A[3] * bx + A[4] * by + A[5] * bz + tb[1];
        const double tz = A[6] * bx + A[7] * by + A[8] * bz + tb[2];
        if (odd && lane >= 3 * (c - b0) && lane < 3 * (c - b0) + 3) {   // residue c's backbone is final
          double* q = atom(gatoms, c, lane - 3 * (c - b0));
          q[0] = tx; q[1] = ty; q[2] = tz;
        }
        if (k + 1 < n) prepare(k + 1, tx, ty, tz, true);
      }
      if (odd && wl == kTransWave) {
        const D3 xc = ldx(c);
        for (int ch = 0; ch < nchunk; ++ch) {
          const int x = 64 * ch + lane;
          const bool use = x < L && x != c;
          const int i = !use ? 0 : x < c ? x : c, j = !use ? 1 : x < c ? c : x;
          const float* row = P.ydev + (unsigned)(pair_row(i, j, L) * P.stride);
          const float d2 = use ? dist2_64(ldx(x), xc) : __builtin_inff();
          float f;
          const float4 q = ld_stencil(stencil_addr(row, P.zrow, d2, sp, P.d2far, f));
          const double e = fixed30_units(catmull_rom(q.x, q.y, q.z, q.w, f));
          tr += x < c ? -e : e;
        }
      }
      if (pairs && wl < TW) {
        int fill = 0;   // pairs in the wavefront's queue (uniform)
        const int Ip = (p - 1) >> 3, Jp = p >> 3, nJ = nb8 - Jp, ncand = (Ip + 1) * nJ;
        const int row_shift = nres8 - 8 * Jp;   // of the pivot block's rows
        // evaluate the queue's last nq pairs, one per lane
        auto flush = [&](int nq) {
          fill -= nq;
          wave_sync();
          if (lane < nq) {
            const uint2 e = qb[fill + lane];
            int bin;
            float f;
            spline_pos(__builtin_amdgcn_sqrtf(__uint_as_float(e.y)), sp, bin, f);
            int i = (int)(e.x & 2047u);
            i = i >= nres8 ? i - row_shift : i;
            // row i (2L - i - 1) / 2 + (j - i - 1): all factors below 2^24
            const unsigned row = (__umul24((unsigned)i, (unsigned)(2 * L - 1 - i)) >> 1) + (e.x >> 11) - (unsigned)i - 1u;
            const float* q = P.ydev + (__umul24(row, (unsigned)P.stride) + (unsigned)bin);
            acc += fixed30_units(catmull_rom(q[0], q[1], q[2], q[3], f));
          }
          wave_sync();
        };
        // four tiles, the list's entries from `at` on (absent ones: the far tile); pairs
        // inside the last knot go to the queue (ballot and lane rank give the slot), which
        // is evaluated 64 pairs at a time
        auto step = [&](unsigned int e) {
          e += lane_pair;
          const float4 xi = w32[e & 2047u];
          float4 xj[4];
          float d2[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) xj[u] = w32[(e >> 11) + u];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            d2[u] = norm2(xj[u].x - xi.x, xj[u].y - xi.y, xj[u].z - xi.z);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned long long bal = __ballot(d2[u] < P.d2far);
            const unsigned at = __builtin_amdgcn_mbcnt_hi((unsigned int)(bal >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned int)bal, (unsigned)fill));
            if (__builtin_amdgcn_inverse_ballot_w64(bal))
              qb[at] = make_uint2(e + ((unsigned int)u << 11), __float_as_uint(d2[u]));
            fill += (int)__popcll(bal);
          }
          while (fill >= 64) {
            wk_near += 64;
            flush(64);
          }
        };
        // The rectangle's tiles: row blocks I up to that of p - 1, column blocks J from
        // that of p.  Candidate tiles are tested one per lane and dealt to the wavefronts
        // round-robin; the survivors are listed and taken four at a time.
        const float inv_nJ = __builtin_amdgcn_rcpf((float)nJ);
        int ntile = 0;   // tiles listed (uniform)
        for (int cb = 0; cb < ncand; cb += 64 * TW) {
          const int cand = cb + lane * TW + wl;
          unsigned int code = code0;   // first row | first column << 11
          if (cb > 0 || Ip != I_code || Jp != J_code) {
            // quotient through the float reciprocal, exact for operands below 2^21
            const int I = (int)(((float)cand + 0.5f) * inv_nJ), J = Jp + (cand - I * nJ);
            code = cand < ncand ? (unsigned)(8 * (I == Jp ? nb8 : I)) | ((unsigned)(8 * J) << 11) : 0u;
            if (cb == 0) { code0 = code; I_code = Ip; J_code = Jp; }
          }
          const float4 a = sph[(code & 2047u) >> 3], b = sph[code >> 14];
          const float dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
          const float lim = rcut + a.w + b.w;
          const unsigned long long m = __ballot(cand < ncand && dx * dx + dy * dy + dz * dz <= lim * lim);
          if (__builtin_amdgcn_inverse_ballot_w64(m)) {
            const unsigned at = __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned int)m, (unsigned)ntile));
            list[at] = code;
            if (count) {   // pairs inside the rectangle
              const int j0 = (int)(code >> 11), i0 = (int)(code & 2047u);
              wk_tests += (unsigned)(i0 == nres8 ? p - 8 * Jp : 8) * (unsigned)((j0 + 8 < L ? j0 + 8 : L) - (j0 > p ? j0 : p));
            }
          }
          const int found = (int)__popcll(m);
          ntile += found;
          wk_tiles += (unsigned)found;
          wave_sync();
          while (ntile >= 4) {
            ntile -= 4;
            step(list[ntile + (lane >> 4)]);
          }
        }
        if (ntile > 0) step((lane >> 4) < ntile ? list[lane >> 4] : far_tile);
        if (fill > 0) {
          wk_near += (unsigned int)fill;
          flush(fill);
        }
      }
      {
        double v = fold_halves(acc, tr);
        v += dpp_d<kDppXor1>(v);
        v += dpp_d<kDppXor2>(v);
        v += dpp_d<kDppRor4>(v);
        v += dpp_d<kDppRor8>(v);
        if ((lane & 15) == 0) part[kHalf * (lane >> 5) + 2 * wl + ((lane >> 4) & 1)] = v;
      }
      lds_barrier();
      // [D] decision, commit, next rotation
      double pv = part[lane];
      const double log_u_next = slot->log_u, delta_next = slot->delta;
      pv += dpp_d<kDppXor1>(pv);
      if constexpr (NW > 1) pv += dpp_d<kDppXor2>(pv);
      if constexpr (NW > 2) {   // (a rotation by 4 brings lane 0 lane 12's sum: both are needed)
        pv += dpp_d<kDppRor4>(pv);
        pv += dpp_d<kDppRor8>(pv);
      }
      double snew = readlane_d(pv, 0), trn = readlane_d(pv, kHalf);
      if constexpr (NW == 16) { snew += readlane_d(pv, 16); trn += readlane_d(pv, 48); }
      rp += trn;
      const double dE = pairs ? (snew - rp) * (1.0 / 1073741824.0) : 0.0;
      const bool accepted = __builtin_amdgcn_readfirstlane((dE <= 0.0) || (log_u < -beta * dE) ? 1 : 0) != 0;
      dE_prev = dE;
      delta_prev = delta;
      acc_prev = accepted;
      log_u = log_u_next;
      delta = delta_next;
      if (accepted) {
        rp = pairs ? snew : 0.0;
        // commit: turn the C-betas the torsion moves (float64)
        const int c0 = p >> 6;
        for (int ch = c0 + ((wl - c0) & (NW - 1)); ch < nchunk; ch += NW) {
          const int r = 64 * ch + lane;
          if (r >= p && r < L) {
            const D3 x = apply_rot(R, ldx(r));
            xb[r] = x.x; xb[nres8 + r] = x.y; xb[2 * nres8 + r] = x.z;
          }
        }
        if (helper) {   // x -> R (x - a) + a after (A, b)
          double nA[9], nb[3];
#pragma unroll
          for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
              nA[3 * r + q] = R.r[3 * r] * A[q] + R.r[3 * r + 1] * A[3 + q] + R.r[3 * r + 2] * A[6 + q];
            nb[r] = R.r[3 * r] * (tb[0] - R.a[0]) + R.r[3 * r + 1] * (tb[1] - R.a[1]) +
                    R.r[3 * r + 2] * (tb[2] - R.a[2]) + R.a[r];
          }
#pragma unroll
          for (int q = 0; q < 9; ++q) A[q] = nA[q];
          tb[0] = nb[0]; tb[1] = nb[1]; tb[2] = nb[2];
        }
      }
      get(slot->rot[accepted ? 1 : 0]);   // (written again only after the next barrier)
    }
    if (helper) book(n - 1);
    // the helper reads back what it stored, and the slot
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    lds_barrier();
  }
  if (count) {
    if (lane == 0) {
      atomicAdd(P.work + 0, (unsigned long long)wk_tiles);
      atomicAdd(P.work + 2, (unsigned long long)wk_near);
    }
    atomicAdd(P.work + 1, (unsigned long long)wk_tests);
  }
  if (helper && lane == 0) P.counters[4 * chain + 1] += n_acc;
  // a wavefront stores the C-betas it has committed
  for (int r = 64 * wl + lane; r < L; r += 64 * NW) {
    double* q = atom(gatoms, r, 3);
    q[0] = xb[r]; q[1] = xb[nres8 + r]; q[2] = xb[2 * nres8 + r];
  }
}

template <int NW>
__global__ __launch_bounds__(NW == 16 ? 1024 : 512) void global_kernel(SweepParams P, int G) {
  global_body<NW>(P, blockIdx.x, G);
}

// Several proteins in one launch: workgroup b runs chain group map[b].y of the protein
// described by descs[map[b].x] (the grid is ordered by decreasing work).
template <int NW>
__global__ __launch_bounds__(NW == 16 ? 1024 : 512) void global_batch_kernel(const SweepParams* __restrict__ descs,
                                                                             const int2* __restrict__ map, int G) {
  const int2 wm = map[blockIdx.x];
  if (descs[wm.x].n_sweeps == 0) return;
  global_body<NW>(descs[wm.x], wm.y, G);
}

#define AMH_GLOBAL(NW)                                        \
  template __global__ void global_kernel<NW>(SweepParams, int); \
  template __global__ void global_batch_kernel<NW>(const SweepParams*, const int2*, int);
AMH_GLOBAL(1)
AMH_GLOBAL(2)
AMH_GLOBAL(4)
AMH_GLOBAL(8)
AMH_GLOBAL(16)

}  // namespace amh
