// amh_kernels.h -- kernel parameter blocks and launch entry points shared by the
// kernels (amh_kernels.hip) and the C ABI (amh_api.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace amh {

// bits of the device error word
constexpr unsigned int kErrTable = 1u;   // non-finite distogram entry
constexpr unsigned int kErrEnergy = 2u;  // non-finite energy or energy change
constexpr unsigned int kErrStall = 4u;   // a pipelined localized sweep waited past its bound

struct SweepParams {
  // distogram table, padded rows
  const float* table;     // padded -ln p rows (anchors)
  const float* ydev;      // padded rows minus the no-contact value (sweeps)
  const float* zrow;      // a padded row of zeros (read by pairs beyond the last knot)
  int stride, nb;
  float inv_w, off, tmax, d2far;
  double d_min, bin_w;
  double vfar;            // sum of every row's no-contact value (far_sum_kernel)
  // run
  int L, C, half_window, global_every, n_global, anchor_every;   // n_global >= 1
  int n_cascade, cascade_hw[3];   // extra window half-widths taken in turn with half_window
  double sigma, sigma_end, T0, T1;  // sigma_end > 0: geometric decay of the proposal width
  int64_t S, t0, n_sweeps;
  int chain0;         // first chain of a localized launch (its chains end before C)
  uint32_t key0, key1, chain_offset;
  int spin_limit;     // polls of a pipelined localized sweep's wait before it gives up
  double target;
  // chain state
  double* s;          // [C][2L]
  double* s_best;     // [C][2L]
  double* atoms;      // [C][L][4][3] N, CA, C, CB (float64)
  double* v;          // [C][2]     V at last anchor, best V
  int64_t* counters;  // [C][4]
  unsigned int* err;
  // trace
  int n_trace;
  int trace_chain[4];
  double* tr_dE;
  double* tr_delta;
  uint8_t* tr_acc;
  int64_t trace_cap, trace_t0;
  double* tr_anchor;
  int64_t trace_anchor_cap, trace_anchor0;
  // executed-work counters of the global sweeps, or null: [0] rectangle tiles that
  // survive the bounding-sphere test, [1] pair tests inside the rectangle in those
  // tiles, [2] near pairs evaluated (one stencil each); added to at the end of a launch
  unsigned long long* work;
};

struct ConfParams {
  int L;
  const double* s_in;   // [B][2L] or null (extended chain)
  // energy (optional: table == null skips it)
  const float* table;
  int stride, nb;
  double d_min, bin_w;
  double vfar;          // sum of every row's no-contact value (far_sum_kernel)
  double* V_out;        // [B]
  double* s_out;        // [B][2L]
  float* cb_out;        // [B][L][3]
  float* atoms_out;     // [B][L][4][3]
  double* atoms64_out;  // [B][L][4][3]
  // context initialisation (optional)
  double* v_state;      // [B][2]
  int64_t* counters;    // [B][4]
  double* s_best;       // [B][2L]
  int keep_best;        // v_state: set V as current, lower the best (and s_best) only if V is lower
  unsigned int* err;
};

size_t sweep_lds_bytes(int G, int L, int W);
size_t local_lds_bytes(int G, int L, int W);
size_t global_lds_bytes(int G, int L, int NW);

// Sweep t is global iff it is one of the last n_global sweeps of its cycle of
// global_every sweeps (Algorithm 1's alternation, localized sweeps first).
__host__ __device__ inline bool is_global(const SweepParams& P, int64_t t) {
  return P.global_every > 0 && (int)((uint32_t)t % (uint32_t)P.global_every) >= P.global_every - P.n_global;
}

// End of the run of sweeps that starts at t and goes into one launch: sweeps of one kind
// (localized or global), up to an anchor (after a sweep count that anchor_every divides) or `end`,
// and at most 2^30 proposals a chain, which a launch counts the accepted of in 32 bits.
inline int64_t run_end(const SweepParams& P, int64_t t, int64_t end) {
  const bool glob = is_global(P, t);
  const int64_t most = t + (1 << 30) / (2 * P.L);
  int64_t e = t + 1;
  while (e < end && e < most && e % P.anchor_every != 0 && is_global(P, e) == glob) ++e;
  return e;
}

// Whether localized sweeps of half-width h (the widest, where several are taken in turn) can carry
// the energy of their changed pairs along as one float64 count of 2^-30: it has to be exact, below
// 2^53, through every proposal, whatever the chain does, with a table whose entries deviate from
// their row's no-contact value by dev_max at most (a Catmull-Rom value is at most 1.25 times the
// largest of its four).  A wall of 1e15 nats would leave a nat's error in all energy changes.
inline bool carry_exact(int h, int L, float dev_max) {
  const double window = (h + 1.0) * (h + 1.0), chain = 0.25 * L * L;
  const double pairs = (window < chain ? window : chain) + 2.0 * h + 1.0;
  return pairs * 1.3 * (double)dev_max < 8388608.0;
}

// Whether carrying is also the faster way, for workgroups of G chains (64 / G lanes each, R rows of
// pairs a lane at a time) and a chain of L residues.  Summed afresh, a proposal gathers each
// changed pair's stencil twice; carried, once, with about 2h pairs more in a gather of their own,
// deals of the pairs by columns that leave lanes idle, and one proposal more between the
// pipelined sweeps.  Nine localized sweeps afresh / carried, us:
//   * pairs that fit the lanes once are summed afresh (1 chain of 16 residues, d = 12 296 / 386; of
//     64, d = 12 442 / 468, d = 15 466 / 616; 512 chains of 64, d = 8 518 / 589; 1024, d = 12 750 / 800)
//     unless the chain is so long that the gathers outweigh the deals made anew near its ends:
//     from 100 residues for four chains a wavefront, which are bound by instruction issue (1024
//     chains, d = 8, 100 850 / 826, 300 2145 / 1984; d = 12, 100 1017 / 1040, 200 1679 / 1649,
//     300 2405 / 2318), from 400 for two with d = 12 on (512 chains of 400 2464 / 2434, but with d = 8
//     of 300 1716 / 1814) and one, as long as pairs and carries fit together (512 chains of 800, one a
//     workgroup, d = 12 6411 / 6328; with d = 15 one of 300 1320 / 1623);
//   * beyond, by the gathers of a phi and a psi: carrying has to save more than three of them (200
//     residues: 1 chain, d = 20 1389 / 1480, d = 30 2430 / 2233; 512 chains, d = 16 1883 / 1659;
//     1024 chains, d = 15 2379 / 1837, d = 18 2783 / 2826, d = 30 6656 / 4454), and not in chains hardly
//     longer than the window, where no deal is kept (32 residues, 1 chain, d = 30 971 / 1177).
inline bool carry_pays(int G, int h, int L) {
  const int LW = 64 / G, R = G > 2 ? 3 : G;
  if (h * (h + 1) <= LW * R)
    return G == 4 ? L >= 100 : L >= 400 && (G == 2 ? h >= 6 : h * (h + 1) + 2 * h + 1 <= LW);
  const auto up = [](int a, int b) { return (a + b - 1) / b; };
  const auto rows = [&](int nF, int nM) {   // of a lane, with the changed pairs dealt by columns
    return R * (nM > LW ? up(nM, LW) * up(nF, R) : up(up(nF, LW / nM), R));
  };
  const int afresh = 2 * (2 * R * up(h * (h + 1), LW * R));
  const int carried = rows(h, h + 1) + rows(h + 1, h) + up(2 * h, LW) + up(2 * h + 1, LW);
  return L >= 16 + 32 / G && carried + 3 < afresh;
}

// Half-width of a localization radius d >= 0 in a chain of L residues.  The window [max(0, c - h),
// min(L - 1, c + h)] is the whole chain from h = L - 1 on, so a wider one is cut to it: the
// kernels' loops and sums of half-widths (c + 2h, 4h) stay within a few L whatever the d.
inline int half_window(int d, int L) { return d / 2 < L - 1 ? d / 2 : L - 1; }

// Squared distance of the last knot as the sweeps test it.  The global kernel's absent rows and
// columns stand 1e18 A off, and the localized one's unused slots at +inf: both have to lie beyond
// it, or they would be taken for pairs and read past the table.  No two residues of a chain are
// 1e15 A apart, so a knot farther off than that is as good as there.
inline float last_knot2(double d_min, double bin_w, int n_bins) {
  const double d = d_min + bin_w * (n_bins - 0.5), d2 = d * d;
  return d2 < 1e30 ? (float)d2 : 1e30f;
}

// A wavefront's pairs inside the last knot, waiting for their energies.
struct EnergyQueue {
  double d2[128];           // (63 and a tile at most)
  unsigned int code[128];   // i << 10 | j
};

inline size_t conf_lds_bytes(int L, int threads, bool energy) {
  const size_t frames = 8 * 12 * ((3 * ((size_t)L - 1) + 63) / 64);
  const size_t queues = energy ? sizeof(EnergyQueue) * (threads / 64) : 0;
  return 8 * (14 * (size_t)L + 2) + 16 * (size_t)((L + 7) / 8) + (frames > queues ? frames : queues);
}

__global__ void ingest_kernel(const float* y, int64_t P, int nb, int stride, float* out,
                              float* dev, float* most, unsigned int* err);
__global__ void conf_energy_kernel(ConfParams P);
__global__ void far_sum_kernel(const float* table, int64_t P, int stride, int nb, const float* most, int n_most,
                               double* out, float* dev_max);
__global__ void philox_kernel(const uint32_t* ctr, int64_t n, uint32_t k0, uint32_t k1, uint32_t* out);
__global__ void perturb_kernel(double* s, int64_t n_total, int n, uint32_t chain_offset, uint32_t tag,
                               uint32_t k0, uint32_t k1, double amplitude);
__global__ void anchor_kernel(SweepParams P);
__global__ void anchor_batch_kernel(const SweepParams* descs, const int2* map, int G);
// localized sweeps: G chains per workgroup, any number of wavefronts (<= 12); CARRY: the energy
// of the changed pairs is carried from proposal to proposal (carry_exact)
template <int G, bool CARRY>
__global__ void local_kernel(SweepParams P);
template <int G, bool CARRY>
__global__ void local_batch_kernel(const SweepParams* descs, const int2* map);
// global sweeps: G chains per workgroup, NW wavefronts each (1, 2, 4, 8 or 16)
template <int NW>
__global__ void global_kernel(SweepParams P, int G);
template <int NW>
__global__ void global_batch_kernel(const SweepParams* descs, const int2* map, int G);

}  // namespace amh
