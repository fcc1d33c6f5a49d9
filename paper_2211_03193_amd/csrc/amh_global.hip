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
// one tile at a time and wrote the next rotation after the decision, with a third barrier
// (one sweep of chains near a minimum, called from the host): 1024 chains of 300 residues
// (2 chains and 4 wavefronts a workgroup) 9.1 -> 5.9 ms; 128 chains of 300 3.4 -> 1.8; 1500 of
// 250 11.9 -> 4.8; 64 of 800 10.1 -> 5.4; one of 64 residues 0.43 -> 0.28.  What bounds it is
// instructions: a wavefront alone issues one in 5 to 8 cycles (8 where it needs the one before),
// and with two a SIMD the vector units are busy for about half of the time (1024 chains of 300
// residues over a whole annealed run: 770 vector instructions a wavefront and proposal).  Four
// wavefronts a SIMD fit (the helper's state is in LDS and the randoms are drawn in a call, 128
// registers instead of 226): 1500 chains of 250 residues 3.3 -> 2.3 ms for the step that did it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amh_device.h"
#include "amh_geom.h"
#include "amh_kernels.h"
#include "amh_proposal.h"

namespace amh {

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

// The helper's state of a sweep, in LDS and not in registers: every wavefront is allocated
// the registers of the busiest point, and these would be live at all of them.
struct HelperState {
  double A[12];                    // the accepted moves composed: x -> A x + b (matrix, b)
  double window[64][3];            // backbone atoms from the window's first residue on
  Batch batch[64];                 // randoms of 64 consecutive proposals
};

// LDS of one chain: float64 C-betas (x, y, z arrays), float32 C-betas of the trial
// conformation (with two more blocks of 8: the fixed rows of the pivot's block, and one
// that is far from everything), spheres, the slots of the current and the next proposal,
// the helper's state, partial sums, near-pair queues and tile lists.
__host__ __device__ inline size_t global_chain_bytes(int L, int NW) {
  const size_t nb8 = (size_t)((L + 7) >> 3);
  return nb8 * (8 * 24 + 8 * 16 + 16) + (16 * 16 + 16) + 2 * sizeof(Slot) + sizeof(HelperState) + 8 * 64 +
         (8 * (size_t)kQueue + 4 * kList) * NW;
}

size_t global_lds_bytes(int G, int L, int NW) { return (size_t)G * global_chain_bytes(L, NW); }

// Workgroup barrier that orders LDS only: loads and stores of global memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Randoms of the 64 proposals from kn on, one per lane, to LDS.  A call and not inlined:
// the compiler keeps the constants of log, cos and sincos in registers throughout the
// loop that contains them (210 registers a lane against 128).
typedef __attribute__((address_space(3))) Batch LdsBatch;
__device__ __attribute__((noinline)) void draw_batch(CParams* P, int kn, uint32_t t, int chain, LdsBatch* out) {
  const int lane = threadIdx.x & 63;
  const Batch b = fill_batch(*P, kn, t, P->chain_offset + (uint32_t)chain, lane);
  out[lane].delta = b.delta;
  out[lane].log_u = b.log_u;
  out[lane].cd = b.cd;
  out[lane].sd = b.sd;
}

// The global sweeps [P.t0, P.t0 + P.n_sweeps) of chains group G .. group G + G - 1 of the
// protein that P describes, NW wavefronts a chain.
template <int NW>
__device__ __forceinline__ void global_body(CParams& P, const int group, const int G) {
  extern __shared__ __align__(16) unsigned char lds[];
  // From four wavefronts on the helper leaves the tiles to the others; with four it takes the
  // transitions (16 wavefronts a unit are busy, and taking them elsewhere cost 4 % at 1500
  // chains of 250 residues), below, the wavefronts share both.  With eight and more (kWide) the
  // helper's next rotation alone is as long as the others' tiles, so these take the
  // transitions too, gathered before the candidate tests, and the helper goes first on its
  // vector unit: 128 chains of 300 residues 1970 -> 1735 us a sweep, 64 of 800 8670 -> 7390.
  constexpr int TW = NW >= 4 ? NW - 1 : NW;
  constexpr bool kWide = NW >= 8;
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
  Slot* const slots = reinterpret_cast<Slot*>(sph + nb8 + 1);          // [2]
  HelperState* const hs = reinterpret_cast<HelperState*>(slots + 2);
  double* const part = reinterpret_cast<double*>(hs + 1);              // [64]
  uint2* const qb = reinterpret_cast<uint2*>(part + 64) + kQueue * wl;
  unsigned int* const list = reinterpret_cast<unsigned int*>(reinterpret_cast<uint2*>(part + 64) + kQueue * NW) +
                             kList * wl;
  auto ldx = [&](int r) { return D3{xb[r], xb[nres8 + r], xb[2 * nres8 + r]}; };

  const Spline32 sp{P.inv_w, P.off, P.tmax};
  const bool helper = wl == NW - 1;
  double* const gatoms = P.atoms + (size_t)chain * L * 12;
  double* const gs = P.s + (size_t)chain * n;
  const int slot_id = trace_slot(P, chain);
  const float d2far = P.d2far, rcut = __builtin_amdgcn_sqrtf(d2far) + 0.05f;
  const float* const ydev = P.ydev;
  const float* const zrow = P.zrow;
  const int stride = P.stride;
  // absent columns and the columns before the pivot stand at kFar, absent rows at -kFar
  constexpr float kFar = 1e18f;
  // a step's four tiles take 16 lanes each; a lane has one row and four columns
  const unsigned int lane_pair = (unsigned int)((lane >> 1) & 7) | ((unsigned int)(4 * (lane & 1)) << 11);
  const unsigned int far_tile = (unsigned int)(nres8 + 8);   // (the far block's rows, the first columns)
  const bool count = cold(P).work != nullptr;
  // sums of a wavefront's rows of 16 lanes: rows 0 and 1 the rectangle's, 2 and 3 the
  // transition's; part holds the former in its first half, the latter in its second
  constexpr int kHalf = NW == 16 ? 32 : 16;
  int n_acc = 0;   // accepted proposals (run_end keeps them below 2^31)
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
    const double beta = sweep_beta(&P, t);
    double rp = 0.0;   // D(p) in units of 2^-30
    int b0 = 0;        // first residue of the helper's window
    double sv = 0.0;   // helper: torsion (k & ~63) + lane
    auto load_window = [&](int r0) {
      b0 = r0;
      const int m = 3 * r0 + lane;
      if (lane < kWindowAtoms && m < 3 * L) {
        const double* q = atom(gatoms, m / 3, m % 3);
        const double x = q[0], y = q[1], z = q[2];
        hs->window[lane][0] = x; hs->window[lane][1] = y; hs->window[lane][2] = z;
      }
      wave_sync();
    };
    auto get = [&](const double* o) {
      Rot R;
#pragma unroll
      for (int q = 0; q < 9; ++q) R.r[q] = o[q];
      R.a[0] = o[9]; R.a[1] = o[10]; R.a[2] = o[11];
      return R;
    };
    // slot of proposal kn, from the conformation that proposal kn - 1 starts from; `prev`:
    // the rotation of proposal kn - 1, or null.  `done`: the residue whose backbone is
    // final and is written back, or -1.
    auto prepare = [&](int kn, const double* prev, int done) {
      if ((kn & 63) == 0 && kn < n) {
        draw_batch(&P, kn, (uint32_t)t, chain, (LdsBatch*)hs->batch);
        wave_sync();
      }
      // lanes 0 and 1: the axis atoms of kn, lanes 4 to 6 the backbone of `done`; all LDS
      // reads go out together
      const int m = 3 * ((kn >> 1) - b0) + (kn & 1), e = 3 * (done - b0);
      const double* w = hs->window[lane < 4 ? (kn < n ? m + (lane & 1) : 0) : done >= 0 ? e + (lane < 7 ? lane - 4 : 0) : 0];
      const double* A = hs->A;
      const double x = w[0], y = w[1], z = w[2];
      const Batch b = hs->batch[kn & 63];
      Rot R;
      if (prev) R = get(prev);
      // (the fused order of row3, written as products: its loads' order costs 1 % of a sweep)
      const D3 q{A[0] * x + A[1] * y + A[2] * z + A[9], A[3] * x + A[4] * y + A[5] * z + A[10],
                 A[6] * x + A[7] * y + A[8] * z + A[11]};
      if (done >= 0 && lane >= 4 && lane < 7) st3(atom(gatoms, done, lane - 4), q);
      if (kn >= n) return;
      D3 a{readlane_d(q.x, 0), readlane_d(q.y, 0), readlane_d(q.z, 0)};
      D3 u = unit(a, D3{readlane_d(q.x, 1), readlane_d(q.y, 1), readlane_d(q.z, 1)});
      if (prev) {
        // odd lanes: the outcome where proposal kn - 1 is accepted.  Its rotation turns the
        // next bond rigidly: psi_c moves both atoms of phi_{c+1}'s, phi_c the far atom of
        // psi_c's (whose near atom CA_c is on its axis)
        const D3 a1 = (kn & 1) ? a : apply_rot(R, a), u1 = rot_dir(R, u);
        if (lane & 1) { a = a1; u = u1; }
      }
      Rot o;
      make_rot_u(a, u, b.cd, b.sd, o);
      Slot& sl = slots[kn & 1];
      if (lane < 2) {
#pragma unroll
        for (int c = 0; c < 9; ++c) sl.rot[lane][c] = o.r[c];
        sl.rot[lane][9] = a.x; sl.rot[lane][10] = a.y; sl.rot[lane][11] = a.z;
      }
      if (lane == 0) { sl.log_u = b.log_u; sl.delta = b.delta; }
    };
    if (helper) {
      if (lane < 12) hs->A[lane] = lane == 0 || lane == 4 || lane == 8 ? 1.0 : 0.0;
      load_window(0);
      prepare(0, nullptr, -1);
      if (lane < n) sv = gs[lane];
    }
    lds_barrier();
    // origin of the float32 work array for this sweep: the middle C-beta
    const D3 org = ldx(L / 2);
    int sel = 0;     // the current proposal's rotation is slots[k & 1].rot[sel]
    int pprev = 0;   // pivot of the previous proposal (0: refresh every residue)
    // the previous proposal's outcome, for the helper's bookkeeping
    double dE_prev = 0.0, delta_prev = 0.0;
    auto book = [&](int k, bool acc) {   // of proposal k, by the helper
      if (acc && lane == (k & 63)) sv = wrap_angle(sv + delta_prev);
      if (lane == 0) {
        CParams& q = cold(P);
        if (!isfinite(dE_prev)) atomicOr(q.err, kErrEnergy);
        if (slot_id >= 0) trace_step(q, slot_id, t, k, dE_prev, delta_prev, acc);
      }
      n_acc += acc;
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
        const Rot R = get(slots[odd].rot[sel]);
        auto trial = [&](int ch) {   // this lane's residue of chunk ch
          const int r = 64 * ch + lane;
          float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          if (r < L) {
            D3 x = ldx(r);
            if (r >= p) x = apply_rot(R, x);
            v = make_float4((float)(x.x - org.x), (float)(x.y - org.y), (float)(x.z - org.z), 0.0f);
          }
          return v;
        };
        auto sphere = [&](int ch, float4 v) {
          // any centre will do (the radius is measured from it); the 0.05 A margin of the
          // tile test covers the 1-ulp hardware square root
          const bool real = 64 * ch + lane < L;
          const float cnt = sum8(real ? 1.0f : 0.0f), inv = __builtin_amdgcn_rcpf(cnt > 1.0f ? cnt : 1.0f);
          const float cx = sum8(v.x) * inv, cy = sum8(v.y) * inv, cz = sum8(v.z) * inv;
          const float rad = max8(real ? __builtin_amdgcn_sqrtf((v.x - cx) * (v.x - cx) + (v.y - cy) * (v.y - cy) +
                                                               (v.z - cz) * (v.z - cz))
                                      : 0.0f);
          return make_float4(cx, cy, cz, rad);
        };
        auto publish = [&](int ch, float4 v, float4 s) {
          const int r = 64 * ch + lane;
          const bool real = r < L;
          if (ch == p >> 6 && (r >> 3) == p >> 3) {
            // the pivot's block: its fixed rows have a block of their own
            w32[nres8 + (r & 7)] = r < p && real ? v : make_float4(-kFar, -kFar, -kFar, 0.0f);
            w32[r] = r >= p && real ? v : make_float4(kFar, kFar, kFar, 0.0f);
          } else if (real) {
            w32[r] = v;
          }
          if ((r & 7) == 0 && r < nres8) {
            sph[r >> 3] = s;
            if ((r >> 3) == p >> 3) sph[nb8] = s;
          }
        };
        const int c0 = pprev >> 6;
        for (int ch = c0 + ((wl - c0) & (NW - 1)); ch < nchunk; ch += NW) {
          const float4 v = trial(ch);
          publish(ch, v, sphere(ch, v));
        }
      }
      pprev = p;
      lds_barrier();
      // [C] the changed pairs of the trial conformation, and for odd k the row and column
      // that carry D from pivot p - 1 to p (current conformation): residue x against p - 1
      double acc = 0.0, tr = 0.0;
      const bool pairs = p > 0 && p < L;
      // the transition's pairs of chunk ch: their stencils, and their sum
      auto trans_load = [&](int ch, float4& q, float& f) {
        const int x = 64 * ch + lane;
        const bool use = x < L && x != c;
        const int i = !use ? 0 : x < c ? x : c, j = !use ? 1 : x < c ? c : x;
        const float* row = ydev + __umul24((unsigned)pair_row(i, j, L), (unsigned)stride);
        const float d2 = use ? dist2_64(ldx(x), ldx(c)) : __builtin_inff();
        q = ld_stencil(stencil_addr(row, zrow, d2, sp, d2far, f));
      };
      auto trans_add = [&](int ch, const float4& q, float f) {
        const double e = fixed30_units(catmull_rom(q.x, q.y, q.z, q.w, f));
        tr += 64 * ch + lane < c ? -e : e;
      };
      // chunks ch, ch + step, ...: two gathers in flight
      auto transitions = [&](int ch, int step) {
        for (; ch < nchunk; ch += 2 * step) {
          float4 q0, q1;
          float f0, f1;
          trans_load(ch, q0, f0);
          const bool two = ch + step < nchunk;
          if (two) trans_load(ch + step, q1, f1);
          trans_add(ch, q0, f0);
          if (two) trans_add(ch + step, q1, f1);
        }
      };
      if (helper) {
        if (kWide) __builtin_amdgcn_s_setprio(3);
        if (k > 0) book(k - 1, sel != 0);
        if (!odd && c + 1 > b0 + 20 && c + 1 < L) load_window(c);
        prepare(k + 1, slots[odd].rot[sel], odd ? c : -1);
      }
      const bool early = kWide && odd && wl < TW && wl < nchunk;
      float4 tq;
      float tf;
      if (early) trans_load(wl, tq, tf);
      if (kWide && helper) __builtin_amdgcn_s_setprio(0);
      if (!kWide && odd && (NW < 4 || helper)) transitions(NW < 4 ? wl : 0, NW < 4 ? NW : 1);
      if (pairs && wl < TW) {
        int fill = 0;   // pairs in the wavefront's queue (uniform)
        const int Ip = (p - 1) >> 3, Jp = p >> 3, nJ = nb8 - Jp, ncand = (Ip + 1) * nJ;
        const int row_shift = nres8 - 8 * Jp;   // of the pivot block's rows
        // evaluate the queue's last nq pairs, one per lane: their stencils are gathered
        // here and evaluated at the next call, so that the gather overlaps the steps between
        float4 fq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float ff = 0.0f;
        auto finish = [&]() { acc += fixed30_units(catmull_rom(fq.x, fq.y, fq.z, fq.w, ff)); };
        auto flush = [&](int nq) {
          finish();
          fill -= nq;
          wk_near += (unsigned int)nq;
          wave_sync();
          fq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);   // (evaluates to zero)
          if (lane < nq) {
            const uint2 e = qb[fill + lane];
            int bin;
            spline_pos(__builtin_amdgcn_sqrtf(__uint_as_float(e.y)), sp, bin, ff);
            int i = (int)(e.x & 2047u);
            i = i >= nres8 ? i - row_shift : i;
            // row i (2L - i - 1) / 2 + (j - i - 1): all factors below 2^24
            const unsigned row = (__umul24((unsigned)i, (unsigned)(2 * L - 1 - i)) >> 1) + (e.x >> 11) - (unsigned)i - 1u;
            fq = ld_stencil(ydev + (__umul24(row, (unsigned)stride) + (unsigned)bin));
          }
          wave_sync();
        };
        // a step of four tiles; pairs inside the last knot go to the queue (ballot and lane
        // rank give the slot), which is evaluated 64 pairs at a time
        auto step = [&](unsigned int e) {
          e += lane_pair;
          const float4 xi = w32[e & 2047u];
          float4 xj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) xj[u] = w32[(e >> 11) + u];
          // all 16 bytes are asked for: 12-byte LDS reads are slower (5 % of the sweep)
          asm volatile("" ::"v"(xi.w), "v"(xj[0].w), "v"(xj[1].w), "v"(xj[2].w), "v"(xj[3].w));
          float d2[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) d2[u] = norm2(xj[u].x - xi.x, xj[u].y - xi.y, xj[u].z - xi.z);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const unsigned long long bal = __ballot(d2[u] < d2far);
            const unsigned at = __builtin_amdgcn_mbcnt_hi((unsigned int)(bal >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((unsigned int)bal, (unsigned)fill));
            if (__builtin_amdgcn_inverse_ballot_w64(bal))
              qb[at] = make_uint2(e + ((unsigned int)u << 11), __float_as_uint(d2[u]));
            fill += (int)__popcll(bal);
          }
          while (fill >= 64) flush(64);
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
          unsigned int ahead = list[(ntile >= 4 ? ntile - 4 : 0) + (lane >> 4)];   // read a step ahead
          while (ntile >= 4) {
            ntile -= 4;
            const unsigned int e = ahead;
            ahead = list[(ntile >= 4 ? ntile - 4 : 0) + (lane >> 4)];
            step(e);
          }
        }
        if (ntile > 0) step((lane >> 4) < ntile ? list[lane >> 4] : far_tile);
        if (fill > 0) flush(fill);
        finish();
      }
      if (early) {
        trans_add(wl, tq, tf);
        if (wl + TW < nchunk) transitions(wl + TW, TW);
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
      const double log_u = slots[odd].log_u, delta = slots[odd].delta;
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
      if (accepted) {
        rp = pairs ? snew : 0.0;
        const Rot R = get(slots[odd].rot[sel]);
        // commit: turn the C-betas the torsion moves (float64)
        const int c0 = p >> 6;
        for (int ch = c0 + ((wl - c0) & (NW - 1)); ch < nchunk; ch += NW) {
          const int r = 64 * ch + lane;
          if (r >= p && r < L) {
            const D3 x = apply_rot(R, ldx(r));
            xb[r] = x.x; xb[nres8 + r] = x.y; xb[2 * nres8 + r] = x.z;
          }
        }
        if (helper) {   // x -> R (x - a) + a after (A, b): column q of (A | b) in lane q
          const int q = lane & 3;
          double* A = hs->A;
          double v0 = A[q < 3 ? q : 9], v1 = A[q < 3 ? 3 + q : 10], v2 = A[q < 3 ? 6 + q : 11];
          if (q == 3) { v0 -= R.a[0]; v1 -= R.a[1]; v2 -= R.a[2]; }
          double w[3];
#pragma unroll
          for (int r = 0; r < 3; ++r) w[r] = row3(R.r + 3 * r, v0, v1, v2);
          if (q == 3) { w[0] += R.a[0]; w[1] += R.a[1]; w[2] += R.a[2]; }
          wave_sync();
          if (lane < 4) { A[q < 3 ? q : 9] = w[0]; A[q < 3 ? 3 + q : 10] = w[1]; A[q < 3 ? 6 + q : 11] = w[2]; }
          wave_sync();
        }
      }
      sel = accepted ? 1 : 0;
    }
    if (helper) book(n - 1, sel != 0);
    // the helper reads back what it stored, and its slots
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    lds_barrier();
  }
  if (count) {
    if (lane == 0) {
      atomicAdd(cold(P).work + 0, (unsigned long long)wk_tiles);
      atomicAdd(cold(P).work + 2, (unsigned long long)wk_near);
    }
    atomicAdd(cold(P).work + 1, (unsigned long long)wk_tests);
  }
  if (helper && lane == 0) cold(P).counters[4 * chain + 1] += n_acc;
  // a wavefront stores the C-betas it has committed
  for (int r = 64 * wl + lane; r < L; r += 64 * NW) {
    double* q = atom(gatoms, r, 3);
    q[0] = xb[r]; q[1] = xb[nres8 + r]; q[2] = xb[2 * nres8 + r];
  }
}

template <int NW>
__global__ __launch_bounds__(NW == 16 ? 1024 : 512, 4) void global_kernel(SweepParams, int G) {
  // (the parameters stand at the start of the kernel's argument segment)
  global_body<NW>(*(CParams*)__builtin_amdgcn_kernarg_segment_ptr(), blockIdx.x, G);
}

// Several proteins in one launch: workgroup b runs chain group map[b].y of the protein
// described by descs[map[b].x] (the grid is ordered by decreasing work).
template <int NW>
__global__ __launch_bounds__(NW == 16 ? 1024 : 512, 4) void global_batch_kernel(const SweepParams* __restrict__ descs,
                                                                             const int2* __restrict__ map, int G) {
  const int2 wm = map[blockIdx.x];
  CParams& P = *(CParams*)(uintptr_t)(descs + wm.x);
  if (P.n_sweeps == 0) return;
  global_body<NW>(P, wm.y, G);
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
