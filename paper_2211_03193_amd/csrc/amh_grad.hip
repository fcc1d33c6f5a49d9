// amh_grad.hip -- gradient of the distogram energy with respect to the torsions,
// and a per-chain L-BFGS minimiser built on it, for MI355X (gfx950, wave64).
//
// The energy is V(s) = sum_{i<j} E_ij(|CB_i - CB_j|) over the conformation G(s)
// (the AlphaFold1 distogram term the paper samples, Sec. 2.3).  Turning torsion k
// by eps rotates every residue from the pivot p on about the bond axis u through
// the point a (N_c -> CA_c for phi_c, CA_c -> C_c for psi_c), so with the C-beta
// forces F_j = dV/dx_j
//     dV/ds_k = sum_{j >= p} F_j . (u x (x_j - a)) = u . (T_p - a x S_p),
// where S_p = sum_{j >= p} F_j and T_p = sum_{j >= p} x_j x F_j are suffix sums
// along the chain (pairs with both ends at or after p move rigidly and cancel).
// One O(L^2) force pass and an O(L) scan give the whole gradient.
//
// Everything here is float64 (coordinates, distances, spline and its derivative of
// the float32 table values, sums); this is not the sampling hot loop.
//
// The minimiser is L-BFGS (Liu and Nocedal 1989; two-loop recursion) with a
// backtracking Armijo line search against the largest of the last M accepted
// values (Grippo, Lampariello and Lucidi 1986), the minimiser the paper pairs with
// its sampler (Sec. 3, the L-BFGS columns of Fig. 3).  One workgroup runs one
// chain's whole minimisation; the vectors and the curvature history live in a
// global workspace (resident in L2 for a few hundred chains), the geometry in LDS.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amh_device.h"
#include "amh_geom.h"
#include "amh_grad.h"

namespace amh {

// Pair energy and its derivative dE/dd from a padded row [y1, y0 .. y_{nb-1}, y_{nb-2}]:
// uniform Catmull-Rom on the bin centres, flat (zero derivative) outside the knots.
// t is the position in bin widths from the first centre; the four taps row[b .. b+3]
// are gathered beforehand at b = stencil_base(t): b = 0 below the first knot (q1 =
// row[1] is the value there) and for a NaN position, b = nb - 3 at or beyond the last
// knot (q3 = row[nb]), else the interval of t.  The order of the fused operations is
// written out, here and where the forces are formed: a minimisation multiplies their last
// bits by 10^2 to 10^3 an iteration.
__device__ __forceinline__ int stencil_base(double t, int nb) {
  return !(t > 0.0) ? 0 : t >= (double)(nb - 1) ? nb - 3 : (int)floor(t);
}

__device__ __forceinline__ void spline64_ed(double q0, double q1, double q2, double q3, double t, int b,
                                            int nb, double inv_w, double& E, double& dE) {
  const double f = t - (double)b;
  const double a1 = q2 - q0;
  const double a2 = fma(4.0, q2, fma(2.0, q0, -5.0 * q1)) - q3;
  const double a3 = fma(-3.0, q2, fma(3.0, q1, -q0)) + q3;
  E = 0.5 * fma(f, f * (f * a3), fma(f, f * a2, fma(2.0, q1, f * a1)));
  dE = 0.5 * fma(f, f * (3.0 * a3), fma(f, a2 + a2, a1)) * inv_w;
  if (t <= 0.0) { E = q1; dE = 0.0; }
  if (t >= (double)(nb - 1)) { E = q3; dE = 0.0; }
  if (t != t) { E = t; dE = t; }   // a NaN distance: V turns NaN
}

typedef __attribute__((address_space(1))) const float gfloat;

// integer add to an LDS word through an LDS pointer (a generic-pointer atomic would be a
// flat operation, which the compiler then waits on together with the table gathers)
__device__ __forceinline__ void lds_add(long long* p, long long v) {
  __hip_atomic_fetch_add((__attribute__((address_space(3))) long long*)p, v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_WORKGROUP);
}

// x rounded to a multiple of 2^-44, as an integer count of 2^-44 (|x| < 2^19)
__device__ __forceinline__ long long fixed44(double x) { return (long long)rint(x * 0x1p44); }

// Sum over the 64 lanes by a fixed butterfly: every lane gets the same value.
__device__ __forceinline__ double wave_allsum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double wave_allmax(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Block-wide reductions; every thread returns the same value, summed in a fixed
// order (strided partials of the first kReduceThreads threads, the lane butterfly, their
// waves in order), which does not depend on the workgroup's size.
// `red` holds 3 kReduceThreads / 64 doubles.  Each call begins and ends with a barrier.
__device__ void block_sum3(double& a, double& b, double& c, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int W = kReduceThreads / 64;
  a = wave_allsum(a); b = wave_allsum(b); c = wave_allsum(c);
  __syncthreads();
  if (lane == 0 && wave < W) { red[3 * wave] = a; red[3 * wave + 1] = b; red[3 * wave + 2] = c; }
  __syncthreads();
  a = 0.0; b = 0.0; c = 0.0;
  for (int v = 0; v < W; ++v) { a += red[3 * v]; b += red[3 * v + 1]; c += red[3 * v + 2]; }
  __syncthreads();
}

__device__ double block_dot(const double* __restrict__ x, const double* __restrict__ y, int n,
                            double* red) {
  double a = 0.0, b = 0.0, c = 0.0;
  if (threadIdx.x < kReduceThreads)
    for (int e = threadIdx.x; e < n; e += kReduceThreads) a += x[e] * y[e];
  block_sum3(a, b, c, red);
  return a;
}

__device__ double block_maxabs(const double* __restrict__ x, int n, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int W = kReduceThreads / 64;
  double m = 0.0;
  if (threadIdx.x < kReduceThreads)
    for (int e = threadIdx.x; e < n; e += kReduceThreads) m = fmax(m, fabs(x[e]));
  m = wave_allmax(m);
  __syncthreads();
  if (lane == 0 && wave < W) red[wave] = m;
  __syncthreads();
  m = 0.0;
  for (int v = 0; v < W; ++v) m = fmax(m, red[v]);
  __syncthreads();
  return m;
}

// Adds x to s and what the addition rounds off to c (Knuth's two-sum).
__device__ __forceinline__ void two_sum(double& s, double& c, double x) {
  const double t = s + x, b = t - s;
  c += (s - (t - b)) + (x - b);
  s = t;
}

__device__ __forceinline__ double pair_dist2(double ex, double ey, double ez) {
  return fma(ez, ez, fma(ex, ex, ey * ey));
}

// V by one wavefront, pair by pair in a fixed order with Neumaier's compensation, of any finite
// energies: for tables whose pairs can be 2^16 nats or more from their no-contact value, which
// the integer sums of value_grad do not hold.
__device__ __attribute__((noinline)) double ordered_energy(int L, const gfloat* table, int stride, int nb,
                                                           double first, double inv_w, double d2far,
                                                           const double* x64) {
  const int lane = threadIdx.x & 63;
  double s = 0.0, c = 0.0;
  for (int i = 0; i < L; ++i) {
    const double* xi = atom(x64, i, 3);
    for (int j = i + 1 + lane; j < L; j += 64) {
      const double* xj = atom(x64, j, 3);
      const double d2 = pair_dist2(xj[0] - xi[0], xj[1] - xi[1], xj[2] - xi[2]);
      const gfloat* row = table + (size_t)pair_row(i, j, L) * stride;
      double E = (double)row[nb], dE;
      if (!(d2 >= d2far)) {   // (a NaN distance gives a NaN energy)
        const double t = fma(d2, d2 > 0.0 ? rsqrt64(d2) : 0.0, -first) * inv_w;
        const int b = stencil_base(t, nb);
        spline64_ed((double)row[b], (double)row[b + 1], (double)row[b + 2], (double)row[b + 3], t, b, nb, inv_w, E, dE);
      }
      neumaier_add(s, c, E);
    }
  }
  double a = 0.0, b = 0.0;
  for (int l = 0; l < 64; ++l) {
    neumaier_add(a, b, readlane_d(s, l));
    b += readlane_d(c, l);
  }
  return a + b;
}

// V(s) and, if g != null, dV/ds of one conformation, by the whole workgroup.
// x64 [12 L], ft [6 (L + 1)], sph [(L + 7) / 8] and pairs [wavefronts] (of grad_pair_bytes(cap)
// bytes each) are LDS scratch, vacc three LDS words.
// Returns V in every thread; g is complete after the closing barrier.
//
// Only pairs inside the last knot have a force and an energy other than their row's
// no-contact value (whose sum is vfar): a few in a hundred of a folded chain's.  They are
// taken by tiles of 64 rows by 64 columns, which the wavefronts draw in turn from the diagonal
// (where most of them are) outwards, a row and a column of the tile per lane:
//   * every lane marks its row's pairs inside the last knot (blocks of 8 columns that the
//     bounding spheres rule out for all lanes are passed over); the ballots are the columns'
//     marks;
//   * the pairs are listed row by row and evaluated 64 at a time, dE/dd / d going to LDS;
//   * every lane adds the forces of its row and then of its column, each in the order
//     u = (j - i) mod 64.  A list that its LDS does not hold is taken in ranges of u.
// A tile's forces on a residue, rounded to multiples of 2^-44, and a pair's energy, in multiples of
// 2^-26 and 2^-70, are added as integers: the totals do not depend on the order of the tiles or
// on the launch shape.  `ordered` (a table with deviations beyond these integers): the energies are
// left out, and the number returned says only whether V is NaN.
// At 512 conformations of 400 residues (two workgroups of 4 wavefronts a unit, one pair in six
// inside the last knot) the time goes to the sums (27 %), the marks (20 %), the coordinates
// (19 %) and the evaluations (17 %): vector instructions, at two wavefronts a SIMD.  (Inlined, with
// LDS reads instead of flat ones and 130 registers instead of 248, it takes 1 to 10 % longer, 128
// minimisations of 200 residues 7 %.)  Evaluating all pairs, absent and far ones too, one a lane
// and step: 290 us, now 250; 64 of 800 665, now 278; one of 300 152, now 56; 1024 of 300 368, now
// 283; 128 of 200 minimised for 20 iterations 4.4 ms, now 2.3.
//
// FEW (up to three tiles, no more than wavefronts): folded chains of up to 128 residues have most
// of their pairs inside the last knot and one dense tile, which one wavefront would take while the
// others wait (70 of 88 thousand cycles at 64 residues).  So the wavefronts share every tile's
// marks, evaluations and sums, with barriers between: conformations of 64 residues, with all pairs
// evaluated / a tile a wavefront / tiles shared, 1 of them 38 / 39 / 24 us, 512 43 / 54 / 34; 200 of
// 100 48 / 50 / 36, of 128 51 / 57 / 39.
template <bool FEW>
__device__ __attribute__((noinline)) double value_grad(const double* __restrict__ s, int L, const float* __restrict__ table,
                             int stride, int nb, double d_min, double w, double vfar, bool ordered, double* x64, double* ft,
                             float4* sph, unsigned char* pairs, int cap, long long* vacc,
                             double* __restrict__ g) {
  const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, wave = tid >> 6, W = T >> 6;
  const double dfar = d_min + w * ((double)nb - 0.5), d2far = dfar * dfar;   // the last knot
  const double inv_w = 1.0 / w, first = d_min + 0.5 * w;
  const float rcut = (float)dfar + 0.05f;   // (0.05 A: far above float32 rounding)
  // the table through a global-memory pointer: its gathers do not wait for LDS reads (but the LDS
  // arrays come as generic pointers, whose flat reads wait for the gathers in flight too)
  const gfloat* gtable = (const gfloat*)table;
  // the C-beta forces F_k accumulate as integers (multiples of 2^-44) in the first
  // three slots of ft[6k .. 6k+5]
  long long* facc = reinterpret_cast<long long*>(ft);
  nerf_wg(s, L, x64, ft);   // (ft holds the NeRF's scratch: nerf_scratch(L) <= 6 (L + 1))
  for (int k = tid; k < L; k += T) facc[6 * k] = facc[6 * k + 1] = facc[6 * k + 2] = 0;
  if (tid == 0) vacc[0] = vacc[1] = vacc[2] = 0;
  block_spheres(x64, L, sph);
  __syncthreads();
  bool wide = false;   // an item's sum beyond the integer range (or NaN): V is returned NaN
  const int nb64 = (L + 63) >> 6, ntile = nb64 * (nb64 + 1) / 2;
  // this wavefront's list of a tile's pairs: dE/dd / d, the marks and list positions of its
  // rows, and the pairs themselves (row | u << 6)
  unsigned char* const scratch = pairs + grad_pair_bytes(cap) * wave;
  double* const qs = reinterpret_cast<double*>(scratch);
  unsigned long long* const marks = reinterpret_cast<unsigned long long*>(qs + cap);
  unsigned short* const base = reinterpret_cast<unsigned short*>(marks + 64);
  unsigned short* const code = base + 64;
  // retire every memory operation before the tiles (the NeRF's spill stores among them)
  __builtin_amdgcn_s_waitcnt(0);
  double whole = 0.0, part = 0.0;   // energies of the pairs, multiples of 2^-26 and of 2^-70
  struct Tile { int off, i0, j0; };
  // 64 pairs: ends, distance, stencil base and taps, issued one step ahead of their
  // evaluation (the flat read of a pair's code waits for the gather before it, which
  // therefore overlaps that step's arithmetic only)
  struct Pair {
    double inv_d, t;
    int b;
    bool use;
    float q0, q1, q2, q3, qn;
  };
  auto prep = [&](const Tile& tl, const unsigned short* list, int count, int k) {
    Pair a;
    a.use = k < count;
    const int cd = a.use ? list[k] : 0;
    const int pi = tl.i0 + (cd & 63), pj = a.use ? tl.j0 + (((cd & 63) + (cd >> 6)) & 63) : 0;
    const double* xa = atom(x64, pi, 3);
    const double* xb = atom(x64, pj, 3);
    const double d2 = pair_dist2(xb[0] - xa[0], xb[1] - xa[1], xb[2] - xa[2]);
    // distance through the hardware reciprocal square root and two Newton steps
    a.inv_d = a.use && d2 > 0.0 ? rsqrt64(d2) : 0.0;
    a.t = fma(d2, a.inv_d, -first) * inv_w;
    a.b = stencil_base(a.t, nb);
    const gfloat* r = gtable + (size_t)(a.use ? pair_row(pi, pj, L) : 0) * stride;
    a.q0 = r[a.b]; a.q1 = r[a.b + 1]; a.q2 = r[a.b + 2]; a.q3 = r[a.b + 3];
    a.qn = r[nb];
    return a;
  };
  auto eval = [&](const Pair& a, double* q, int k) {
    if (!a.use) return;
    double E, dE;
    spline64_ed((double)a.q0, (double)a.q1, (double)a.q2, (double)a.q3, a.t, a.b, nb, inv_w, E, dE);
    // deviation e + low from the no-contact value, exactly (Knuth's two-sum), in multiples
    // of 2^-26 and of 2^-70: every digit of a pair's energy down to these
    double e = E, low = 0.0;
    two_sum(e, low, -(double)a.qn);
    const double n = rint(e * 0x1p26);   // (sums of integers below 2^53)
    whole += n;
    part += rint((fma(n, -0x1p-26, e) + low) * 0x1p70);
    q[k] = a.inv_d > 0.0 ? dE * a.inv_d : 0.0;
  };
  // dV/dx_j = +q (x_j - x_i), dV/dx_i = -q (x_j - x_i): the steps of `left` added to the force on
  // this lane's row (whose pairs lie in the list from k on) ...
  // (two a step, so that their reads overlap; an absent one adds zero)
  auto add_row = [&](const Tile& tl, const double* q, unsigned long long left, int k, double ix, double iy, double iz,
                     double& rx, double& ry, double& rz) {
    while (left != 0) {
      const int ua = __builtin_ctzll(left);
      left &= left - 1;
      const bool two = left != 0;
      const int ub = two ? __builtin_ctzll(left) : ua;
      left &= left - 1;
      const double* xa = atom(x64, tl.j0 + ((lane + ua) & 63), 3);
      const double* xb = atom(x64, tl.j0 + ((lane + ub) & 63), 3);
      const double qa = -q[k], qb = two ? -q[k + 1] : 0.0;
      rx = fma(xa[0] - ix, qa, rx); ry = fma(xa[1] - iy, qa, ry); rz = fma(xa[2] - iz, qa, rz);
      rx = fma(xb[0] - ix, qb, rx); ry = fma(xb[1] - iy, qb, ry); rz = fma(xb[2] - iz, qb, rz);
      k += 2;
    }
  };
  // ... and to that on its column
  auto add_col = [&](const Tile& tl, const double* q, const unsigned long long* mk, const unsigned short* bs,
                     unsigned long long left, double jx, double jy, double jz, double& cx, double& cy, double& cz) {
    while (left != 0) {
      const int ua = __builtin_ctzll(left), ra = (lane - ua) & 63;
      left &= left - 1;
      const bool two = left != 0;
      const int ub = two ? __builtin_ctzll(left) : ua, rb = (lane - ub) & 63;
      left &= left - 1;
      const double* xa = atom(x64, tl.i0 + ra, 3);
      const double* xb = atom(x64, tl.i0 + rb, 3);
      const double qa = q[bs[ra] + (int)__popcll(mk[ra] & ((1ull << ua) - 1))];
      const double qv = q[bs[rb] + (int)__popcll(mk[rb] & ((1ull << ub) - 1))], qb = two ? qv : 0.0;
      cx = fma(jx - xa[0], qa, cx); cy = fma(jy - xa[1], qa, cy); cz = fma(jz - xa[2], qa, cz);
      cx = fma(jx - xb[0], qb, cx); cy = fma(jy - xb[1], qb, cy); cz = fma(jz - xb[2], qb, cz);
    }
  };
  if constexpr (FEW) {   // fewer tiles than wavefronts: they share each tile
    auto tile_at = [&](int t) {
      int off = 0, I = t;   // J - I, I
      while (I >= nb64 - off) { I -= nb64 - off; ++off; }
      return Tile{off, 64 * I, 64 * (I + off)};
    };
    // marks of the 8 columns from jq on: `mine` of this lane's row, `rows` of column lane & 7
    auto mark8 = [&](const float4& si, double ix, double iy, double iz, bool present, int jq, unsigned int& mine,
                     unsigned long long& rows) {
      mine = 0;
      rows = 0;
      const float4 sq = sph[jq >> 3];
      const float dx = si.x - sq.x, dy = si.y - sq.y, dz = si.z - sq.z, lim = rcut + si.w + sq.w;
      if (__ballot(present && !(dx * dx + dy * dy + dz * dz > lim * lim)) == 0) return;
#pragma unroll
      for (int r = 0; r < 8; ++r) {   // (NaN distances are evaluated, so V turns NaN)
        const double* x = atom(x64, jq + r < L ? jq + r : 0, 3);
        const bool use = !(pair_dist2(x[0] - ix, x[1] - iy, x[2] - iz) >= d2far);
        const unsigned long long bal = __ballot(use);
        mine |= use ? 1u << r : 0u;
        if ((lane & 7) == r) rows = bal;
      }
    };
    // marks by column and by row -> by the step u
    auto by_step = [&](const Tile& tl, unsigned long long near, unsigned long long column, unsigned long long& row,
                       unsigned long long& col) {
      if (tl.j0 + 64 > L) near &= (1ull << (L - tl.j0)) - 1;
      if (tl.j0 + lane >= L) column = 0;
      if (tl.off == 0) {
        near &= ~1ull << lane;
        column &= (1ull << lane) - 1;
      }
      const unsigned long long rev = __brevll(column);
      const int by = (lane + 1) & 63;
      row = near >> lane | near << ((64 - lane) & 63);
      col = rev << by | rev >> ((64 - by) & 63);
    };
    // list position of the row's first pair of m, and the number of all rows' pairs
    auto place = [&](unsigned long long m, int& at, int& count) {
      const int n = (int)__popcll(m);
      at = count = 0;
#pragma unroll
      for (int b = 0; b < 7; ++b) {
        const unsigned long long bal = __ballot((n >> b) & 1);
        at += (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0)) << b;
        count += (int)__popcll(bal) << b;
      }
    };
    const double lim = 0x1p13;   // |tile sum| < 2^13: a residue's total stays below 2^19
    auto add_force = [&](int k, double x, double y, double z) {
      lds_add(facc + 6 * k, fixed44(x));
      lds_add(facc + 6 * k + 1, fixed44(y));
      lds_add(facc + 6 * k + 2, fixed44(z));
    };
    // the wavefronts' list memory: per tile its marks (of row i by column, then by step), its list
    // positions and its columns' marks, then one list of all tiles' pairs
    unsigned long long* const all_marks = reinterpret_cast<unsigned long long*>(pairs);
    unsigned long long* const columns = all_marks + 64 * ntile;
    unsigned short* const all_base = reinterpret_cast<unsigned short*>(columns + 64 * ntile);
    double* const all_qs = reinterpret_cast<double*>(all_base + 64 * ntile);
    const int room = grad_shared_pairs(W, cap, ntile);
    unsigned short* const all_code = reinterpret_cast<unsigned short*>(all_qs + room);
    int* const counts = reinterpret_cast<int*>(vacc + 3);
    // marks, 8 columns an item
    for (int e = wave; e < 8 * ntile; e += W) {
      const Tile tl = tile_at(e >> 3);
      const int q = 8 * (e & 7), i = tl.i0 + lane;
      const double* xp = atom(x64, i < L ? i : 0, 3);
      unsigned int mine = 0;
      unsigned long long rows = 0;
      if (tl.j0 + q < L)
        mark8(sph[i < L ? i >> 3 : 0], i < L ? xp[0] : 1e300, xp[1], xp[2], i < L, tl.j0 + q, mine, rows);
      const int k = 64 * (e >> 3) + lane;
      reinterpret_cast<unsigned char*>(all_marks + k)[e & 7] = (unsigned char)mine;
      if ((lane >> 3) == (e & 7)) columns[k] = rows;
    }
    __syncthreads();
    // the steps of the tile sides that this wavefront will add; list positions, a tile a wavefront
    unsigned long long mask[2] = {0, 0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = wave + h * W, k = 64 * (e >> 1) + lane;   // tile and side
      if (e >= 2 * ntile) continue;
      unsigned long long row, col;
      by_step(tile_at(e >> 1), all_marks[k], columns[k], row, col);
      mask[h] = e & 1 ? col : row;
    }
    unsigned long long row = 0;
    int at = 0;
    if (wave < ntile) {
      unsigned long long col;
      int count;
      by_step(tile_at(wave), all_marks[64 * wave + lane], columns[64 * wave + lane], row, col);
      place(row, at, count);
      if (lane == 0) counts[wave] = count;
    }
    __syncthreads();
    // as many tiles at a time as the list holds (one at least; the rule of FEW sees to that)
    for (int t0 = 0, t1; t0 < ntile; t0 = t1) {
      int total = 0;
      for (t1 = t0; t1 < ntile && (t1 == t0 || total + counts[t1] <= room); ++t1) {
        if (t1 == wave) at += total;
        total += counts[t1];
      }
      if (t0 > 0) __syncthreads();   // (the list has been read)
      if (t0 <= wave && wave < t1) {
        all_marks[64 * wave + lane] = row;
        all_base[64 * wave + lane] = (unsigned short)at;
        for (unsigned long long left = row; left != 0; left &= left - 1)
          all_code[at++] = (unsigned short)(lane | (__builtin_ctzll(left) << 6));
      }
      __syncthreads();
      // evaluations, 64 pairs of a tile an item
      for (int t = t0, from = 0, k = wave; t < t1; from += counts[t], ++t) {
        const int n = counts[t];
        for (; 64 * k < n; k += W) {
          const Pair A = prep(tile_at(t), all_code + from, n, 64 * k + lane);
          eval(A, all_qs + from, 64 * k + lane);
        }
        k -= (n + 63) >> 6;
      }
      __syncthreads();
      // sums, a side of a tile an item
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int e = wave + h * W, t = e >> 1;
        if (t < t0 || t >= t1 || __ballot(mask[h] != 0) == 0) continue;
        const Tile tl = tile_at(t);
        const int k = (e & 1 ? tl.j0 : tl.i0) + lane;
        const double* xp = atom(x64, k < L ? k : 0, 3);
        double fx = 0.0, fy = 0.0, fz = 0.0;
        if (e & 1) add_col(tl, all_qs, all_marks + 64 * t, all_base + 64 * t, mask[h], xp[0], xp[1], xp[2], fx, fy, fz);
        else add_row(tl, all_qs, mask[h], all_base[64 * t + lane], xp[0], xp[1], xp[2], fx, fy, fz);
        const bool fits = fabs(fx) < lim && fabs(fy) < lim && fabs(fz) < lim;
        wide = wide || !fits;
        if (fits && mask[h] != 0) add_force(k, fx, fy, fz);
      }
    }
    if (!ordered && whole == whole) {   // (a NaN pair's coordinates make a sum NaN, too)
      lds_add(vacc, (long long)whole);
      lds_add(vacc + 2, (long long)part);
    }
  }
  while (!FEW) {
    int tile = 0;
    if (lane == 0)
      tile = (int)__hip_atomic_fetch_add((__attribute__((address_space(3))) int*)(vacc + 1), 1, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    tile = __builtin_amdgcn_readfirstlane(tile);
    if (tile >= ntile) break;
    int off = 0, I = tile;   // J - I, I
    while (I >= nb64 - off) { I -= nb64 - off; ++off; }
    const Tile tl{off, 64 * I, 64 * (I + off)};
    const int i0 = tl.i0, j0 = tl.j0, i = i0 + lane, j = j0 + lane;
    const double* xp = atom(x64, i < L ? i : 0, 3);
    // (absent rows stand far off; absent columns and those up to the row drop out of the marks)
    const double ix = i < L ? xp[0] : 1e300, iy = xp[1], iz = xp[2];
    const float4 si = sph[i < L ? i >> 3 : 0];
    unsigned long long near = 0;       // of row i, by column
    unsigned long long column = 0;     // of column j, by row
    for (int q = 0; q < 64 && j0 + q < L; q += 8) {
      const float4 sq = sph[(j0 + q) >> 3];
      const float dx = si.x - sq.x, dy = si.y - sq.y, dz = si.z - sq.z, lim = rcut + si.w + sq.w;
      if (__ballot(i < L && !(dx * dx + dy * dy + dz * dz > lim * lim)) == 0) continue;
      unsigned int mine = 0;
      unsigned long long rows = 0;
#pragma unroll
      for (int r = 0; r < 8; ++r) {   // (NaN distances are evaluated, so V turns NaN)
        const double* x = atom(x64, j0 + q + r < L ? j0 + q + r : 0, 3);
        const bool use = !(pair_dist2(x[0] - ix, x[1] - iy, x[2] - iz) >= d2far);
        const unsigned long long bal = __ballot(use);
        mine |= use ? 1u << r : 0u;
        if ((lane & 7) == r) rows = bal;
      }
      near |= (unsigned long long)mine << q;
      if ((lane >> 3) == (q >> 3)) column = rows;
    }
    if (j0 + 64 > L) near &= (1ull << (L - j0)) - 1;
    if (j >= L) column = 0;
    if (off == 0) {
      near &= ~1ull << lane;
      column &= (1ull << lane) - 1;
    }
    if (__ballot(near != 0) == 0) continue;
    // the marks by the step u
    const unsigned long long rev = __brevll(column);
    const int by = (lane + 1) & 63;
    const unsigned long long row = near >> lane | near << ((64 - lane) & 63), col = rev << by | rev >> ((64 - by) & 63);
    xp = atom(x64, j < L ? j : 0, 3);
    const double jx = xp[0], jy = xp[1], jz = xp[2];
    double rx = 0.0, ry = 0.0, rz = 0.0, cx = 0.0, cy = 0.0, cz = 0.0;
    whole = part = 0.0;
    for (int u0 = 0, width = 64; u0 < 64; u0 += width, width = 64 - u0) {
      unsigned long long range, m;   // steps [u0, u0 + width), as many as the list holds
      int at, count;                 // the row's first pair in the list, all pairs
      for (;;) {
        range = (width == 64 ? ~0ull : (1ull << width) - 1) << u0;
        m = row & range;
        const int n = (int)__popcll(m);
        at = count = 0;
#pragma unroll
        for (int b = 0; b < 7; ++b) {
          const unsigned long long bal = __ballot((n >> b) & 1);
          at += (int)__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0)) << b;
          count += (int)__popcll(bal) << b;
        }
        if (count <= cap) break;
        const int fit = width * cap / count;   // (one step has 64 pairs at most)
        width = fit < 1 ? 1 : fit;
      }
      if (count == 0) continue;
      marks[lane] = m;
      base[lane] = (unsigned short)at;
      {
        int k = at;
        for (unsigned long long left = m; left != 0; left &= left - 1)
          code[k++] = (unsigned short)(lane | (__builtin_ctzll(left) << 6));
      }
      wave_sync();
      // two records in turn, so that no gathered value is copied
      Pair A = prep(tl, code, count, lane);
      for (int k = lane;; k += 128) {
        const Pair B = prep(tl, code, count, k + 64);
        eval(A, qs, k);
        if (k - lane + 64 >= count) break;
        A = prep(tl, code, count, k + 128);
        eval(B, qs, k + 64);
        if (k - lane + 128 >= count) break;
      }
      wave_sync();
      add_row(tl, qs, m, at, ix, iy, iz, rx, ry, rz);
      add_col(tl, qs, marks, base, col & range, jx, jy, jz, cx, cy, cz);
      wave_sync();
    }
    const double lim = 0x1p13;   // |tile sum| < 2^13: a residue's total stays below 2^19
    wide = wide || !(fabs(rx) < lim && fabs(ry) < lim && fabs(rz) < lim && fabs(cx) < lim &&
                     fabs(cy) < lim && fabs(cz) < lim);
    if (!wide) {
      if (row != 0) {
        lds_add(facc + 6 * i, fixed44(rx));
        lds_add(facc + 6 * i + 1, fixed44(ry));
        lds_add(facc + 6 * i + 2, fixed44(rz));
      }
      if (col != 0) {
        lds_add(facc + 6 * j, fixed44(cx));
        lds_add(facc + 6 * j + 1, fixed44(cy));
        lds_add(facc + 6 * j + 2, fixed44(cz));
      }
      if (!ordered) {
        lds_add(vacc, (long long)whole);
        lds_add(vacc + 2, (long long)part);
      }
    }
  }
  __syncthreads();
  // force and torque x_k x F_k of every residue, in place
  for (int k = tid; k < L; k += T) {
    const double fx = (double)facc[6 * k] * 0x1p-44, fy = (double)facc[6 * k + 1] * 0x1p-44,
                 fz = (double)facc[6 * k + 2] * 0x1p-44;
    const double* xk = atom(x64, k, 3);
    const double kx = xk[0], ky = xk[1], kz = xk[2];
    double* o = ft + 6 * k;
    o[0] = fx; o[1] = fy; o[2] = fz;
    o[3] = ky * fz - kz * fy;
    o[4] = kz * fx - kx * fz;
    o[5] = kx * fy - ky * fx;
  }
  wide = __syncthreads_or(wide);   // (also the barrier that publishes ft)
  // far constant and the two sums; the first is split so that both parts convert exactly
  double V = vfar, Vc = (double)vacc[2] * 0x1p-70;
  two_sum(V, Vc, (double)(vacc[0] >> 32) * 0x1p6);
  two_sum(V, Vc, (double)(vacc[0] & 0xffffffffLL) * 0x1p-26);
  V = wide ? __builtin_nan("") : V + Vc;
  // suffix sums S_p, T_p (six components, one lane each, in chain order; eight residues
  // are read ahead of the additions, which alone are a chain)
  if (wave == 0 && lane < 6) {
    double acc = 0.0;
    double* f = ft + lane;
    f[6 * L] = 0.0;
    int j = L;
    double v[8], next[8];
    auto read = [&](double* o, int k) {   // residues k + 7 down to k
      const double* p = f + 6 * (k > 0 ? k : 0);
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = p[42 - 6 * q];
    };
    if (j >= 8) read(next, j - 8);
    for (; j >= 8; j -= 8) {
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = next[q];
      read(next, j - 16);
      double* const p = f + 6 * (j - 8);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        acc += v[q];
        p[42 - 6 * q] = acc;
      }
    }
    for (; j > 0; --j) {
      acc += f[6 * (j - 1)];
      f[6 * (j - 1)] = acc;
    }
  }
  __syncthreads();
  if (g) {
    for (int k = tid; k < 2 * L; k += T) {
      double gk = 0.0;
      if (k != 0 && k != 2 * L - 1) {   // phi_0 and psi_{L-1} move no C-beta
        const int c = k >> 1, p = (k & 1) ? c + 1 : c;
        const double* A = atom(x64, c, (k & 1) ? 1 : 0);
        const double* B = atom(x64, c, (k & 1) ? 2 : 1);
        double ux = B[0] - A[0], uy = B[1] - A[1], uz = B[2] - A[2];
        const double iu = 1.0 / sqrt(ux * ux + uy * uy + uz * uz);
        ux *= iu; uy *= iu; uz *= iu;
        const double* S = ft + 6 * p;
        const double tx = S[3] - (A[1] * S[2] - A[2] * S[1]);
        const double ty = S[4] - (A[2] * S[0] - A[0] * S[2]);
        const double tz = S[5] - (A[0] * S[1] - A[1] * S[0]);
        gk = ux * tx + uy * ty + uz * tz;
      }
      g[k] = gk;
    }
  }
  __syncthreads();
  return V;
}

// value_grad for a kernel whose parameters are P; V by ordered_energy where the table asks for it
// (called from here and not from value_grad, which a call would cost 2 % of a minimisation).
template <bool FEW, class Params>
__device__ __forceinline__ double evaluate(const Params& P, const double* s, double* x64, double* ft, float4* sph,
                                           unsigned char* pairs, double* red, double* g) {
  long long* const vacc = reinterpret_cast<long long*>(red);
  double V = value_grad<FEW>(s, P.L, P.table, P.stride, P.nb, P.d_min, P.bin_w, P.vfar, P.ordered, x64, ft, sph, pairs, P.cap,
                             vacc, g);
  if (P.ordered && V == V) {
    if (threadIdx.x < 64) {
      const double dfar = P.d_min + P.bin_w * ((double)P.nb - 0.5);
      const double v = ordered_energy(P.L, (const gfloat*)P.table, P.stride, P.nb, P.d_min + 0.5 * P.bin_w,
                                      1.0 / P.bin_w, dfar * dfar, x64);
      if (threadIdx.x == 0) red[0] = v;
    }
    __syncthreads();
    V = red[0];
    __syncthreads();
  }
  return V;
}

// ---------------------------------------------------------------------------
// Both kernels are held to two wavefronts per SIMD (at most 256 registers a lane).
// Left free, the compiler gives the NeRF scan 271 registers and every kernel one wavefront
// per SIMD; under the cap it spills a little inside that scan, and two workgroups of four
// wavefronts share each CU (the most their LDS allows at 400 residues).
template <bool FEW>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) grad_kernel(GradParams P) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int L = P.L;
  double* x64 = reinterpret_cast<double*>(lds);
  double* ft = x64 + 12 * L;
  float4* sph = reinterpret_cast<float4*>(ft + 6 * (L + 1));
  unsigned char* pairs = reinterpret_cast<unsigned char*>(sph + ((L + 7) >> 3));
  double* red = reinterpret_cast<double*>(pairs + (blockDim.x >> 6) * grad_pair_bytes(P.cap));
  const int b = blockIdx.x;
  const double V = evaluate<FEW>(P, P.s + (size_t)b * 2 * L, x64, ft, sph, pairs, red, P.g ? P.g + (size_t)b * 2 * L : nullptr);
  if (threadIdx.x == 0) {
    if (!isfinite(V)) atomicOr(P.err, kErrGradEnergy);
    if (P.V) P.V[b] = V;
  }
}

// ---------------------------------------------------------------------------
// One chain's L-BFGS.  Workspace rows (n = 2L doubles each): x, g, d, xn, gn, then
// the curvature pairs S[m], Y[m] kept as a ring (oldest at `head`).
template <bool FEW>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) lbfgs_kernel(LbfgsParams P) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int L = P.L, n = 2 * L, tid = threadIdx.x, T = blockDim.x;
  const int m = P.m, M = P.nonmonotone;
  double* x64 = reinterpret_cast<double*>(lds);
  double* ft = x64 + 12 * L;
  float4* sph = reinterpret_cast<float4*>(ft + 6 * (L + 1));
  unsigned char* pairs = reinterpret_cast<unsigned char*>(sph + ((L + 7) >> 3));
  double* red = reinterpret_cast<double*>(pairs + (blockDim.x >> 6) * grad_pair_bytes(P.cap));
  double* rho = red + 3 * kReduceThreads / 64;   // [m]
  double* alp = rho + m;         // [m]
  double* fh = alp + m;          // [M]
  const int b = blockIdx.x;
  double* ws = P.work + (size_t)b * (5 + 2 * (size_t)m) * n;
  double* x = ws;
  double* g = ws + n;
  double* d = ws + 2 * (size_t)n;
  double* xn = ws + 3 * (size_t)n;
  double* gn = ws + 4 * (size_t)n;
  double* Sh = ws + 5 * (size_t)n;
  double* Yh = Sh + (size_t)m * n;
  double* sb = P.s + (size_t)b * n;
  double* trace = P.f_trace ? P.f_trace + (size_t)b * (P.n_iter + 1) : nullptr;
  double* xtr = P.x_trace ? P.x_trace + (size_t)b * (P.n_iter + 1) * n : nullptr;

  for (int e = tid; e < n; e += T) {
    x[e] = sb[e];
    if (xtr) xtr[e] = sb[e];
  }
  __syncthreads();
  double f = evaluate<FEW>(P, x, x64, ft, sph, pairs, red, g);
  if (trace && tid == 0) trace[0] = f;
  if (tid == 0) fh[0] = f;
  int k = 0, head = 0, nf = 1, it = 0, status = 1;
  for (it = 0; it < P.n_iter; ++it) {
    const double gmax = block_maxabs(g, n, red);
    if (gmax <= P.gtol) { status = 0; break; }
    // direction: two-loop recursion, newest pair first, then oldest first
    double gamma = P.step0 / gmax;
    if (k > 0) {
      const int r = (head + k - 1) % m;
      double sy = 0.0, yy = 0.0, z = 0.0;
      for (int e = tid; e < n && tid < kReduceThreads; e += kReduceThreads) {
        const double ye = Yh[(size_t)r * n + e];
        sy += Sh[(size_t)r * n + e] * ye;
        yy += ye * ye;
      }
      block_sum3(sy, yy, z, red);
      gamma = sy / yy;
    }
    for (int e = tid; e < n; e += T) d[e] = g[e];
    __syncthreads();
    for (int i = k - 1; i >= 0; --i) {
      const int r = (head + i) % m;
      const double* sr = Sh + (size_t)r * n;
      const double* yr = Yh + (size_t)r * n;
      const double a = rho[r] * block_dot(sr, d, n, red);
      if (tid == 0) alp[r] = a;
      for (int e = tid; e < n; e += T) d[e] -= a * yr[e];
      __syncthreads();
    }
    for (int e = tid; e < n; e += T) d[e] *= gamma;
    __syncthreads();
    for (int i = 0; i < k; ++i) {
      const int r = (head + i) % m;
      const double* sr = Sh + (size_t)r * n;
      const double* yr = Yh + (size_t)r * n;
      const double bb = rho[r] * block_dot(yr, d, n, red);
      const double a = alp[r];
      for (int e = tid; e < n; e += T) d[e] += (a - bb) * sr[e];
      __syncthreads();
    }
    for (int e = tid; e < n; e += T) d[e] = -d[e];
    __syncthreads();
    double gd = block_dot(g, d, n, red);
    if (!(gd < 0.0)) {   // not a descent direction: drop the history, scaled steepest descent
      k = 0;
      head = 0;
      const double g0 = P.step0 / gmax;
      for (int e = tid; e < n; e += T) d[e] = -g0 * g[e];
      __syncthreads();
      gd = block_dot(g, d, n, red);
    }
    double fref = fh[0];
    for (int i = 1; i < (nf < M ? nf : M); ++i) fref = fmax(fref, fh[i]);
    // Armijo backtracking
    double alpha = 1.0, fnew = 0.0;
    bool ok = false;
    for (int ls = 0; ls < P.max_ls; ++ls) {
      for (int e = tid; e < n; e += T) xn[e] = x[e] + alpha * d[e];
      __syncthreads();
      fnew = evaluate<FEW>(P, xn, x64, ft, sph, pairs, red, gn);
      if (fnew <= fref + P.c1 * alpha * gd) { ok = true; break; }
      alpha *= P.shrink;
    }
    if (!ok) { status = 2; break; }
    // curvature pair, kept only when s.y is clearly positive
    double sy = 0.0, ss = 0.0, yy = 0.0;
    for (int e = tid; e < n && tid < kReduceThreads; e += kReduceThreads) {
      const double se = xn[e] - x[e], ye = gn[e] - g[e];
      sy += se * ye; ss += se * se; yy += ye * ye;
    }
    block_sum3(sy, ss, yy, red);
    if (sy > 1e-8 * sqrt(ss * yy)) {
      if (k == m) { head = (head + 1) % m; --k; }
      const int r = (head + k) % m;
      for (int e = tid; e < n; e += T) {
        Sh[(size_t)r * n + e] = xn[e] - x[e];
        Yh[(size_t)r * n + e] = gn[e] - g[e];
      }
      if (tid == 0) rho[r] = 1.0 / sy;
      ++k;
    }
    __syncthreads();
    // accept: swap the roles of (x, g) and (xn, gn)
    double* t0 = x; x = xn; xn = t0;
    double* t1 = g; g = gn; gn = t1;
    f = fnew;
    if (tid == 0) fh[nf % M] = f;
    ++nf;
    if (trace && tid == 0) trace[it + 1] = f;
    if (xtr)
      for (int e = tid; e < n; e += T) xtr[(size_t)(it + 1) * n + e] = x[e];
    __syncthreads();
  }
  for (int e = tid; e < n; e += T) sb[e] = wrap_angle(x[e]);
  if (P.v_state) {
    const bool better = f < P.v_state[2 * b + 1];
    __syncthreads();
    if (better)
      for (int e = tid; e < n; e += T) P.s_best[(size_t)b * n + e] = wrap_angle(x[e]);
    __syncthreads();
    if (tid == 0) {
      P.v_state[2 * b] = f;
      if (better) P.v_state[2 * b + 1] = f;
    }
  }
  if (tid == 0) {
    if (!isfinite(f)) atomicOr(P.err, kErrGradEnergy);
    if (P.V) P.V[b] = f;
    if (P.iters) P.iters[b] = it;
    if (P.status) P.status[b] = status;
  }
}

template __global__ void grad_kernel<false>(GradParams);
template __global__ void grad_kernel<true>(GradParams);
template __global__ void lbfgs_kernel<false>(LbfgsParams);
template __global__ void lbfgs_kernel<true>(LbfgsParams);

}  // namespace amh
