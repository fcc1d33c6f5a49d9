// amh_local.hip -- localized sweeps of the Alternating Metropolis-Hastings sampler for
// MI355X (gfx950, wave64): every proposal is judged by the energy of the window of
// residues within d/2 of its own (localized MH, Sec. 2.3 and Algorithm 1 of
// arXiv 2211.03193).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amh_device.h"
#include "amh_geom.h"
#include "amh_kernels.h"
#include "amh_proposal.h"

namespace amh {

// ---------------------------------------------------------------------------
// LDS layout of a localized-sweep workgroup: per chain the float64 backbone atoms [3L][3], the
// C-betas (x, y and z arrays, which the lanes read without conflicts) and the torsions [2L]
// (112 L bytes, padded to 64 mod 256, so that the same residue of the G chains, read together,
// falls in different banks); then one progress counter per wavefront and the accept counts per
// wavefront and chain.
__host__ __device__ inline size_t chain_stride(int L) {
  const size_t b = 112 * (size_t)L;
  return b + ((64 + 256 - (b & 255)) & 255);
}

struct Lds {
  unsigned char* base;
  int L, G;
  __device__ size_t per() const { return chain_stride(L); }
  __device__ double* bb(int g) const { return reinterpret_cast<double*>(base + g * per()); }
  __device__ double* cb(int g) const { return bb(g) + 9 * L; }
  __device__ double* s(int g) const { return bb(g) + 12 * L; }
  __device__ int* prog() const { return reinterpret_cast<int*>(base + G * per()); }
  __device__ long long* nacc(int W) const { return reinterpret_cast<long long*>(prog() + ((W + 1) & ~1)); }
};

size_t local_lds_bytes(int G, int L, int W) {
  return (size_t)G * chain_stride(L) + 4 * (size_t)((W + 1) & ~1) + 8 * (size_t)W * G;
}

// Window half-width of localized sweep t: window_d, then the cascade radii in turn
// (Sec. 2.2 allows several localization ranges).
__device__ __forceinline__ int half_window_at(CParams& P, int64_t t) {
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
// Four chains a wavefront are bound by instruction issue (9 of the 12 wavefronts at work in a run of
// 9 sweeps, 2.25 a SIMD, 560 vector instructions a proposal), one chain by the chain of dependent
// ones.  So a proposal does as little as it can: commits write the window's C-betas only (the
// backbone follows when the sweep reaches it); where it pays (carry_pays) the energy as it is is
// carried along, one spline a changed pair and about 2h pairs that correct it, with one column of
// pairs a lane (its C-beta turned once) and pair deals kept from residue to residue.  9 sweeps of
// d = 12 against commits of all atoms, pair by pair throughout, us: L = 64 x 1 chain 489 -> 422;
// 300 x 128 1409 -> 1253; 300 x 1024 2612 -> 2247; 250 x 1500 4393 -> 3469; 800 x 64 3358 -> 2981;
// 100 x 4096 4401 -> 3980.
//
// Pipelining: the m-th sweep of a block of consecutive localized sweeps publishes
// m * 4096 + (proposals done) in `publish`; sweep m+1 waits on that counter so that
// it runs proposal k' (residue c') only once sweep m is past residue c'+2h, with carries past
// phi of the next one.  A localized proposal reads the geometry of its window and (phi) the
// residue before it, and turns residues downstream of its bond, so the two sweeps never touch
// the same residues and the results equal those of running them in turn.
struct Pipe {
  const int* wait_on;   // progress counter of the previous sweep, or null
  int* publish;         // this sweep's progress counter
  int m;                // index of the sweep in its block
};

// Waits until *ctr >= target and returns the value seen (bounded: on a stall the
// error word is flagged and the sweep goes on rather than hang).
__device__ __forceinline__ int wait_progress(CParams& P, const int* ctr, int target,
                                             bool& stalled) {
  if (stalled) return 0x7fffffff;
  for (int spin = 0; spin < P.spin_limit; ++spin) {
    const int v = __hip_atomic_load(ctr, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (v >= target) return v;
    __builtin_amdgcn_s_sleep(2);
  }
  stalled = true;
  atomicOr(cold(P).err, kErrStall);
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

// The sums of a and b over the LW lanes of each chain group.
template <int LW>
__device__ __forceinline__ void pair_sums(double a, double b, int lane, double& sa, double& sb) {
  if constexpr (LW == 64) {   // both at once, a in the lower half of the wavefront and b in the upper
    double v = fold_halves(a, b);
    v += dpp_d<kDppXor1>(v);
    v += dpp_d<kDppXor2>(v);
    v += dpp_d<kDppRor4>(v);
    v += dpp_d<kDppRor8>(v);
    sa = readlane_d(v, 0) + readlane_d(v, 16);
    sb = readlane_d(v, 32) + readlane_d(v, 48);
  } else {
    sa = group_sum<LW>(a, lane);
    sb = group_sum<LW>(b, lane);
  }
}

// Randoms of proposal k + ll of this lane's chain (a call, not inlined: the compiler would
// keep the constants of log, cos and sincos in registers throughout the proposal loop).
__device__ __attribute__((noinline)) Batch draw(CParams* P, int k, uint32_t t, uint32_t chain, int ll) {
  return fill_batch(*P, k, t, P->chain_offset + chain, ll);
}

// One localized sweep of the workgroup's chains (G of them, nact active) by one
// wavefront, with no workgroup barrier inside.  CARRY: the energy of the changed pairs is carried
// from proposal to proposal (carry_exact), else each energy change is summed pair by pair; both
// give the same bits where the carried sum is exact.
template <int G, bool CARRY>
__device__ __forceinline__ void local_sweep(CParams& P, const Lds& S, int nact, int c0, int64_t t, double beta, int h,
                                            int h_prev, int lane, int slot, int& n_acc, const Pipe& pipe,
                                            bool& stalled) {
  constexpr int LW = 64 / G;   // lanes per chain
  constexpr int R = G > 2 ? 3 : G;   // rows a lane scores at a time (42 pairs of d = 12: 3 rows at G = 4)
  const int L = P.L, n = 2 * L;
  const int q = lane / LW, ll = lane - q * LW;
  const bool act = q < nact;
  double* __restrict__ cb = S.cb(q);   // C-beta x, y, z arrays
  double* __restrict__ bb = S.bb(q);   // backbone atoms [3L][3]
  double* __restrict__ s = S.s(q);
  const uint32_t chain = (uint32_t)(c0 + q);
  const Spline32 sp{P.inv_w, P.off, P.tmax};
  const float d2far = P.d2far;
  const float* const ydev = P.ydev;
  const unsigned stride = (unsigned)P.stride, zero_row = (unsigned)(P.zrow - P.ydev);
  auto ldx = [&](int r) { return D3{cb[r], cb[L + r], cb[2 * L + r]}; };
  // accepted moves of the sweep composed, x -> A x + b (float64, uniform over the chain's
  // lanes): what the residues not yet in the window, and the backbone atoms the sweep has
  // not reached, still have to follow
  double A[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, tb[3] = {0, 0, 0};
  // The pairs of a proposal, dealt to the chain's lanes.  The changed pairs (i, j), lo <= i <
  // p <= j <= hi, are scored at their new distance: a lane has one column and consecutive
  // rows of it (j - c | (c - first row) << 10 | rows << 21; the lanes form groups of one lane
  // a column).  The carries take `sum` from the previous proposal's changed pairs to this
  // one's, at their current distance: for psi_c the pivot moves past residue c (its pairs with
  // the rows before it go, those with the columns after it come), for phi_c the window moves
  // on by a residue (the pairs of the first row go, those of the column that enters come);
  // one a lane (c - i | (j - c) << 11 | 1 to take off, 2 to add, 0 none << 22).  So dE needs a
  // spline a changed pair and 2h more, instead of two a pair.  The deal is the same relative
  // to c at every residue away from the chain's ends, and kept.  Near the ends it is made
  // anew, but for one chain a wavefront (`narrow`) kept too and clipped: 4 % less time at
  // L = 64, where the clipping at four chains took 1 % at every length.
  const bool narrow = G == 1 && 4 * h < L && 2 * h + 1 <= LW;
  auto deal_column = [&](int c, int odd, int lo, int hi, int b0, int& rows) {
    const int p = c + odd, nF = p - lo, nM = hi - p + 1, cols = nM - b0 < LW ? nM - b0 : LW;
    if (cols <= 0 || nF <= 0) { rows = 0; return 0; }
    // (hardware reciprocals: quotients of numbers below 2^11 stay exact)
    const float inv = __builtin_amdgcn_rcpf((float)cols);
    const int groups = (int)(((float)LW + 0.5f) * inv);
    rows = __builtin_amdgcn_readfirstlane(
        (int)(((float)(nF + groups - 1) + 0.5f) * __builtin_amdgcn_rcpf((float)groups)));
    const int g = (int)(((float)ll + 0.5f) * inv), j = p + b0 + (ll - g * cols), i0 = lo + g * rows;
    const int cnt = g < groups && i0 < p ? (i0 + rows < p ? rows : p - i0) : 0;
    return (j - c) | ((cnt > 0 ? c - i0 : 0) << 10) | (cnt << 21);
  };
  auto deal_carry = [&](int c, int odd, int lo, int hi, int y) {
    const int lo1 = narrow || c - 1 - h > 0 ? c - 1 - h : 0, hi1 = narrow || c - 1 + h < L - 1 ? c - 1 + h : L - 1;
    const int ngo = odd ? c - lo : lo > lo1 ? hi1 - c + 1 : 0, ncome = odd ? hi - c : hi > hi1 ? c - lo : 0;
    const bool go = y < ngo, use = y >= 0 && y < ngo + ncome;
    const int i = odd ? (go ? lo + y : c) : go ? lo1 : lo + y - ngo;
    const int j = odd ? (go ? c : c + 1 + y - ngo) : go ? c + y : hi;
    return use ? (c - i) | ((j - c) << 11) | ((go ? 1 : 2) << 22) : 0;
  };
  int column[2] = {0, 0}, carry[2] = {0, 0}, nrow[2] = {0, 0};
  bool one[2] = {false, false}, known[2] = {false, false};
  auto deal = [&](int c, int odd, int lo, int hi) {
    const int p = c + odd, nF = p - lo, nM = hi - p + 1, npair = nF > 0 && nM > 0 ? nF * nM : 0;
    column[odd] = deal_column(c, odd, lo, hi, 0, nrow[odd]);
    one[odd] = G == 1 && npair + 2 * h + 1 <= LW;   // all of them in a lane of their own
    carry[odd] = deal_carry(c, odd, lo, hi, one[odd] ? ll - npair : ll);
    if (one[odd] && column[odd] >> 21)   // (one row a lane here)
      carry[odd] = ((column[odd] >> 10) & 2047) | ((column[odd] & 1023) << 11) | (3 << 22);
  };
  double sum = 0.0;   // energy of the current proposal's changed pairs as they are, in units of 2^-30
  int seen = -1;      // progress of the previous sweep last read
  Batch bt{};
  for (int k = 0; k < n; ++k) {
    const int kl = k & (LW - 1);
    if (kl == 0) bt = draw(&P, k, (uint32_t)t, chain, ll);
    // this proposal's randoms from the lane of the chain that drew them
    const double cd = group_bcast<LW>(bt.cd, lane, kl), sd = group_bcast<LW>(bt.sd, lane, kl);
    const double log_u = group_bcast<LW>(bt.log_u, lane, kl), delta = group_bcast<LW>(bt.delta, lane, kl);
    const int c = k >> 1, odd = k & 1, p = c + odd;
    const int lo = c - h > 0 ? c - h : 0, hi = c + h < L - 1 ? c + h : L - 1;
    if (pipe.wait_on) {
      // the previous sweep (half-width h_prev) must be done with every proposal that reads
      // residue c + h: those of residues up to c' = c + h + h_prev, whose windows reach it,
      // and with carries phi of the next one, which takes the pairs of the row before its window
      // away
      const int ahead = 2 * (c + h + h_prev) + (CARRY ? 3 : 2);
      const int need = (pipe.m - 1) * 4096 + (ahead < n ? ahead : n);
      if (seen < need) seen = wait_progress(P, pipe.wait_on, need, stalled);
    }
    if (!odd && c > 0) {
      // the sweep reaches residue c: its backbone (lanes 0 to 2), and the C-beta of the
      // residue that enters the window (lane 3), follow the moves accepted so far
      const bool enters = hi > c - 1 + h;
      if (ll < 3 || (ll == 3 && enters)) {
        double* const x = ll < 3 ? bb + 3 * (3 * c + ll) : cb + hi;
        const int step = ll < 3 ? 1 : L;
        const double X = x[0], Y = x[step], Z = x[2 * step];
        x[0] = row3(A, X, Y, Z) + tb[0];
        x[step] = row3(A + 3, X, Y, Z) + tb[1];
        x[2 * step] = row3(A + 6, X, Y, Z) + tb[2];
      }
      wave_sync();
    }
    const bool live = k != 0 && k != n - 1, interior = c > h && c < L - h;
    double dE = 0.0, snew = 0.0;
    Rot Rk;
    if (live) {
      // stencil of a pair of the given row at a squared distance (+inf: none): an unused slot
      // and a pair beyond the last knot read the zero row, so that a slot has no branch and
      // all loads are in flight together
      auto gather = [&](unsigned row, float d2, float4& e, float& fr) {
        int bin;
        spline_pos(__builtin_amdgcn_sqrtf(fminf(d2, d2far)), sp, bin, fr);
        const unsigned off = (d2 < d2far ? __umul24(row, stride) : zero_row) + (unsigned)bin;
        e = ld_stencil(ydev + off);
      };
      const int nF = p - lo, nM = hi - p + 1;
      const double* ax = bb + 3 * (3 * c + odd);   // phi_c: N_c -> CA_c; psi_c: CA_c -> C_c
      double str = 0.0;
      if constexpr (!CARRY) {
        // the changed pairs (lo + a, p + b), pair x = a nM + b in slot x / LW of lane x mod LW, at
        // the distance they have and at the proposed one
        const int npair = nF > 0 && nM > 0 ? nF * nM : 0;
        // (hardware reciprocal, 1 ulp: floor((x + 1/2) / nM) stays exact for x < 2^22)
        const float inv_nM = __builtin_amdgcn_rcpf((float)(nM > 0 ? nM : 1));
        for (int x0 = 0; x0 == 0 || x0 < npair; x0 += LW * R) {
          int row[R], col[R];
          float4 e0[R], e1[R];
          float f0[R], f1[R];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int x = x0 + r * LW + ll, a = (int)(((float)x + 0.5f) * inv_nM);
            const bool use = x < npair;
            row[r] = use ? lo + a : -1;
            col[r] = use ? p + (x - a * nM) : c;
            const int i = use ? row[r] : c;
            gather((unsigned)pair_row(i, col[r], L),
                   use ? dist2_64(ldx(i), ldx(col[r])) : __builtin_inff(), e0[r], f0[r]);
          }
          if (x0 == 0) make_rot(ld3(ax), ld3(ax + 3), cd, sd, Rk);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const bool use = row[r] >= 0;
            const int i = use ? row[r] : c;
            gather((unsigned)pair_row(i, col[r], L),
                   use ? dist2_64(ldx(i), apply_rot(Rk, ldx(col[r]))) : __builtin_inff(), e1[r], f1[r]);
          }
#pragma unroll
          for (int r = 0; r < R; ++r)
            snew += fixed30_units(catmull_rom(e1[r].x, e1[r].y, e1[r].z, e1[r].w, f1[r])) -
                    fixed30_units(catmull_rom(e0[r].x, e0[r].y, e0[r].z, e0[r].w, f0[r]));
        }
      } else {
        if (!known[odd] || !(interior || narrow)) {
          deal(c, odd, narrow ? c - h : lo, narrow ? c + h : hi);
          known[odd] = interior || narrow;
        }
        int u = carry[odd], w = column[odd];
        if (!interior && narrow) {
          if (c < (u & 2047) || c + ((u >> 11) & 2047) > hi) u = 0;
          const int out = ((w >> 10) & 2047) - c;   // rows before the chain's first residue
          if (out > 0) w -= out << 21 | out << 10;
          if (w < 0 || c + (w & 1023) > hi) w = 0;
        }
        if (one[odd]) {
          // every pair in a lane of its own: 3 = changed, 1 and 2 = carries, taken off and added
          const int kind = u >> 22, i = c - (u & 2047), j = c + ((u >> 11) & 2047);
          const D3 xi = ldx(i), xj = ldx(j);
          make_rot(ld3(ax), ld3(ax + 3), cd, sd, Rk);
          const D3 xr = apply_rot(Rk, xj);
          const D3 y{kind == 3 ? xr.x : xj.x, kind == 3 ? xr.y : xj.y, kind == 3 ? xr.z : xj.z};
          float4 e;
          float fr;
          gather((unsigned)pair_row(i, j, L), kind != 0 ? dist2_64(xi, y) : __builtin_inff(), e, fr);
          const float v = rintf(catmull_rom(e.x, e.y, e.z, e.w, fr) * 1073741824.0f);
          snew = (double)(kind == 3 ? v : 0.0f);
          str = (double)(kind == 3 ? 0.0f : kind == 1 ? -v : v);
        } else {
          // the carries, at their current distance: their gathers overlap the rotation's set-up
          float4 te;
          float tf;
          auto carry_load = [&]() {
            const int i = c - (u & 2047), j = c + ((u >> 11) & 2047);
            gather((unsigned)pair_row(i, j, L), u >> 22 ? dist2_64(ldx(i), ldx(j)) : __builtin_inff(), te, tf);
          };
          auto carry_add = [&]() {
            const float v = rintf(catmull_rom(te.x, te.y, te.z, te.w, tf) * 1073741824.0f);
            str += (double)(u >> 22 == 1 ? -v : v);
          };
          carry_load();
          make_rot(ld3(ax), ld3(ax + 3), cd, sd, Rk);
          // the changed pairs: a lane has one column (turned once) and some rows of it
          int rows = nrow[odd];
          for (int b0 = 0;;) {
            const int j = c + (w & 1023), i0 = c - ((w >> 10) & 2047), i1 = i0 + (w >> 21);
            const D3 xj = apply_rot(Rk, ldx(j));
            for (int r0 = 0; r0 < rows; r0 += R) {
              float4 e[R];
              float fr[R];
  #pragma unroll
              for (int r = 0; r < R; ++r) {
                const int i = i0 + r0 + r;
                const bool use = i < i1;
                const int ii = use ? i : c;
                gather((unsigned)pair_row(ii, j, L), use ? dist2_64(ldx(ii), xj) : __builtin_inff(), e[r], fr[r]);
              }
              if (b0 + r0 == 0) carry_add();
  #pragma unroll
              for (int r = 0; r < R; ++r)
                snew += fixed30_units(catmull_rom(e[r].x, e[r].y, e[r].z, e[r].w, fr[r]));
            }
            b0 += LW;
            if (b0 >= nM) break;
            w = deal_column(c, odd, lo, hi, b0, rows);
          }
          for (int y = LW; y < (odd ? 2 * h : 2 * h + 1); y += LW) {
            u = deal_carry(c, odd, lo, hi, y + ll);
            carry_load();
            carry_add();
          }
        }
      }
      pair_sums<LW>(act ? snew : 0.0, act ? str : 0.0, lane, snew, str);
      sum += str;
      if (nF > 0 && nM > 0) dE = (snew - sum) * (1.0 / 1073741824.0);
    }
    const int acc = (dE <= 0.0) || (log_u < -beta * dE);
    if (act && ll == 0) {
      if (!isfinite(dE)) atomicOr(cold(P).err, kErrEnergy);
      if (slot >= 0) trace_step(cold(P), slot, t, k, dE, delta, acc);
    }
    if (act && acc) {
      if (ll == 0) s[k] = wrap_angle(s[k] + delta);
      ++n_acc;
      if (live) {
        if constexpr (CARRY) sum = snew;
        // rotate the C-betas of the window that the torsion moves, and for phi_c also C_c
        // (which leaves N_c and CA_c in place); further residues follow when they are reached
        const int nat = hi - p + 1 + (odd ? 0 : 1);
        for (int y = ll; y < nat; y += LW) {
          double* const x = p + y <= hi ? cb + p + y : bb + 3 * (3 * c + 2);
          const int step = p + y <= hi ? L : 1;
          const D3 v = apply_rot(Rk, D3{x[0], x[step], x[2 * step]});
          x[0] = v.x; x[step] = v.y; x[2 * step] = v.z;
        }
        // compose: x -> R (x - a) + a after (A, b)
        double nA[9], nb[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
          for (int qq = 0; qq < 3; ++qq)
            nA[3 * r + qq] = row3(Rk.r + 3 * r, A[qq], A[3 + qq], A[6 + qq]);
          const double* m = Rk.r + 3 * r;
          nb[r] = fma(m[2], tb[2] - Rk.a[2], fma(m[1], tb[1] - Rk.a[1], m[0] * (tb[0] - Rk.a[0]))) + Rk.a[r];
        }
#pragma unroll
        for (int qq = 0; qq < 9; ++qq) A[qq] = nA[qq];
        tb[0] = nb[0]; tb[1] = nb[1]; tb[2] = nb[2];
      }
    }
    wave_sync();
    if (pipe.publish && lane == 0)
      __hip_atomic_store(pipe.publish, pipe.m * 4096 + k + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// The localized sweeps [P.t0, P.t0 + P.n_sweeps) of one workgroup: the G chains from
// P.chain0 + group G on, of the protein that P describes.  Every wavefront runs all chains of
// the workgroup (64 / G lanes each); the W wavefronts run the consecutive sweeps in turn,
// pipelined.
template <int G, bool CARRY>
__device__ __forceinline__ void local_body(CParams& P, const int group) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, W = T >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = P.L, n = 2 * L;
  const int c0 = P.chain0 + group * G;
  const int nact = P.C - c0 < G ? P.C - c0 : G;
  const Lds S{lds, L, G};

  // load chain state; absent chains (a last workgroup with nact < G) hold zeros: their
  // lanes compute on them without any effect
  for (int e = tid; e < G * L * 12; e += T) {
    const int g = e / (12 * L), z = e - g * 12 * L, r = z / 12, w = z - 12 * r;
    double* o = w < 9 ? S.bb(g) + 9 * r + w : S.cb(g) + (w - 9) * L + r;
    *o = g < nact ? P.atoms[(size_t)c0 * L * 12 + e] : 0.0;
  }
  for (int e = tid; e < nact * n; e += T) S.s(e / n)[e % n] = P.s[(size_t)c0 * n + e];
  const int lslot = (lane / (64 / G)) < nact ? trace_slot(P, c0 + lane / (64 / G)) : -1;
  int acc_stage = 0;   // accepted proposals of this lane's chain (run_end keeps them below 2^31)
  bool stalled = false;
  // blocks of at most 4096 sweeps (the progress counters' range)
  for (int64_t t = P.t0, t_end = P.t0 + P.n_sweeps; t < t_end;) {
    const int nblk = t_end - t < 4096 ? (int)(t_end - t) : 4096;
    for (int e = tid; e < W; e += T) S.prog()[e] = 0;
    __syncthreads();
    for (int m = wave; m < nblk; m += W) {
      const int64_t tm = t + m;
      Pipe pipe;
      pipe.m = m;
      pipe.publish = S.prog() + wave;
      pipe.wait_on = m > 0 ? S.prog() + ((m - 1) % W) : nullptr;
      local_sweep<G, CARRY>(P, S, nact, c0, tm, sweep_beta(&P, tm), half_window_at(P, tm),
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
    const int g = e / (12 * L), z = e - g * 12 * L, r = z / 12, w = z - 12 * r;
    P.atoms[(size_t)c0 * L * 12 + e] = w < 9 ? S.bb(g)[9 * r + w] : S.cb(g)[(w - 9) * L + r];
  }
  for (int e = tid; e < nact * n; e += T) P.s[(size_t)c0 * n + e] = S.s(e / n)[e % n];
}

template <int G, bool CARRY>
__global__ __launch_bounds__(768) void local_kernel(SweepParams) {
  // (the parameters stand at the start of the kernel's argument segment)
  local_body<G, CARRY>(*(CParams*)__builtin_amdgcn_kernarg_segment_ptr(), blockIdx.x);
}

// Several proteins in one launch: workgroup b runs chain group map[b].y of the
// protein described by descs[map[b].x] (the grid is ordered by decreasing work).
template <int G, bool CARRY>
__global__ __launch_bounds__(768) void local_batch_kernel(const SweepParams* __restrict__ descs,
                                                          const int2* __restrict__ map) {
  const int2 wm = map[blockIdx.x];
  CParams& P = *(CParams*)(uintptr_t)(descs + wm.x);
  if (P.n_sweeps == 0) return;
  local_body<G, CARRY>(P, wm.y);
}

#define AMH_LOCAL(G, CARRY)                                       \
  template __global__ void local_kernel<G, CARRY>(SweepParams); \
  template __global__ void local_batch_kernel<G, CARRY>(const SweepParams*, const int2*);
AMH_LOCAL(1, true)
AMH_LOCAL(2, true)
AMH_LOCAL(4, true)
AMH_LOCAL(1, false)
AMH_LOCAL(2, false)
AMH_LOCAL(4, false)

}  // namespace amh
