// amh_api.hip -- the C ABI of libamh.so (declared in include/amh.h): host-side
// validation, device buffers of a sampler context and stream-ordered launches.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "amh.h"
#include "amh_error.h"
#include "amh_grad.h"
#include "amh_kernels.h"

static_assert(sizeof(amh_config) == 120, "amh_config layout");
static_assert(sizeof(amh_lbfgs_opts) == 48, "amh_lbfgs_opts layout");

namespace {
thread_local std::string g_last_error;
}  // namespace

namespace amh {
amh_status sfail(amh_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}
}  // namespace amh

namespace {

using amh::sfail;

#define HIP_OK(expr)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess)                                                              \
      return sfail(AMH_E_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));       \
  } while (0)

constexpr size_t kMaxLds = 160 * 1024;  // LDS per workgroup on gfx950
constexpr int kLocalWaves = 12;          // wavefronts of a localized launch (the most its registers allow)

int row_stride(int nb) { return ((nb + 2) + 3) & ~3; }   // nb values + 2 ghosts, 16-byte rows

}  // namespace

struct amh_ctx {
  amh_config cfg{};
  hipStream_t stream = nullptr;
  unsigned char* slab = nullptr;   // the arrays below, in one allocation
  float* table = nullptr;
  float* ydev = nullptr;
  int stride = 0;
  double* s = nullptr;
  double* s_best = nullptr;
  double* atoms = nullptr;   // [C][L][4][3]
  double* v = nullptr;
  int64_t* counters = nullptr;
  unsigned int* err = nullptr;
  int64_t t = 0;
  double target = -INFINITY;
  // shape of the context (chains and wavefronts per workgroup)
  int G = 1, W = 4;
  // sum of every table row's no-contact value (far_sum_kernel), and the largest deviation of an
  // entry from it (ingest_kernel)
  double vfar = 0.0;
  float dev_max = 0.0f;
  // launches of the localized-sweep kernel: chains [first, first + chains), G per workgroup
  struct LocalPart { int first = 0, chains = 0, G = 1; };
  LocalPart local[2];
  int n_local = 0;
  // launch shape of the global-sweep kernel (chains and wavefronts per workgroup)
  int G_global = 1, W_global = 4;
  // trace
  int n_trace = 0;
  int trace_chain[4] = {-1, -1, -1, -1};
  double* tr_dE = nullptr;
  double* tr_delta = nullptr;
  uint8_t* tr_acc = nullptr;
  int64_t trace_cap = 0, trace_t0 = 0;
  double* tr_anchor = nullptr;
  int64_t trace_anchor_cap = 0, trace_anchor0 = 0;
  int spin_limit = 1 << 24;   // bound of the pipelined sweeps' waits (amh_set_wait_bound)
  // L-BFGS workspace, grown on demand
  double* work = nullptr;
  size_t work_n = 0;
  // this device's copy of the library's fixed scratch array (amh_minimize_noalloc)
  double* scratch = nullptr;
  // caller's executed-work counters of the global sweeps (amh_set_work_counters)
  unsigned long long* work_counters = nullptr;
};

// Fixed scratch of amh_minimize_noalloc: the L-BFGS workspace of callers that cannot
// allocate.  Each device holds its own copy for the life of the process; host code
// reaches it only through the address hipGetSymbolAddress returns for the current
// device (the array's name in host code is not a device address).
static __device__ __align__(256) double scratch[amh::kNoallocScratchDoubles];

namespace {

std::mutex g_scratch_mu;
double* g_scratch_ptr[amh::kMaxDevices] = {};

// Device address of `scratch` on device `dev` (which must be current), looked up
// once per device and kept.
amh_status scratch_address(int dev, double** out) {
  if (dev < 0 || dev >= amh::kMaxDevices) return sfail(AMH_E_DEVICE, "device %d outside [0, %d)", dev, amh::kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return sfail(AMH_E_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return AMH_OK;
}

}  // namespace

namespace {

// What the kernels of amh_init leave of a table: the context's error word and, read back once,
// the rest.
struct TableFacts {
  unsigned int err;
  float dev_max;
  double vfar;
};

// n_cu: compute units of the device (for the automatic launch shape).
amh_status validate(const amh_config* c, int n_cu, int* G, int* W) {
  if (!c) return sfail(AMH_E_INVAL, "config is NULL");
  if (c->L < 2 || c->L > 1024) return sfail(AMH_E_INVAL, "L=%d outside [2, 1024]", c->L);
  if (c->n_chains < 1) return sfail(AMH_E_INVAL, "n_chains=%d < 1", c->n_chains);
  if (c->n_bins < 4 || c->n_bins > 64) return sfail(AMH_E_INVAL, "n_bins=%d outside [4, 64]", c->n_bins);
  if (c->window_d < 0) return sfail(AMH_E_INVAL, "window_d=%d < 0", c->window_d);
  if (!std::isfinite(c->d_min)) return sfail(AMH_E_INVAL, "d_min not finite");
  if (!(c->bin_w > 0.0) || !std::isfinite(c->bin_w)) return sfail(AMH_E_INVAL, "bin_w must be > 0");
  if (c->global_every < 0) return sfail(AMH_E_INVAL, "global_every=%d < 0", c->global_every);
  if (c->n_global < 0 || (c->global_every > 0 && c->n_global > c->global_every))
    return sfail(AMH_E_INVAL, "n_global=%d outside [0, global_every]", c->n_global);
  if (c->anchor_every < 1) return sfail(AMH_E_INVAL, "anchor_every=%d < 1", c->anchor_every);
  if (!(c->sigma >= 0.0) || !std::isfinite(c->sigma)) return sfail(AMH_E_INVAL, "sigma must be finite and >= 0");
  if (!(c->sigma_end >= 0.0) || !std::isfinite(c->sigma_end))
    return sfail(AMH_E_INVAL, "sigma_end must be finite and >= 0");
  if (c->n_cascade < 0 || c->n_cascade > 3) return sfail(AMH_E_INVAL, "n_cascade=%d outside [0, 3]", c->n_cascade);
  for (int i = 0; i < c->n_cascade; ++i)
    if (c->cascade_d[i] < 0) return sfail(AMH_E_INVAL, "cascade_d[%d]=%d < 0", i, c->cascade_d[i]);
  if (!(c->T0 > 0.0) || !(c->T1 > 0.0) || !std::isfinite(c->T0) || !std::isfinite(c->T1))
    return sfail(AMH_E_INVAL, "T0 and T1 must be finite and > 0");
  if (c->total_sweeps < 1 || c->total_sweeps > 0xFFFFFFFFLL)
    return sfail(AMH_E_INVAL, "total_sweeps=%lld outside [1, 2^32-1]", (long long)c->total_sweeps);
  if ((uint64_t)c->chain_offset + (uint64_t)c->n_chains > 0x100000000ULL)
    return sfail(AMH_E_INVAL, "chain_offset + n_chains exceeds 2^32");
  int g = c->chains_per_group;
  if (g != 0 && g != 1 && g != 2 && g != 4)
    return sfail(AMH_E_INVAL, "chains_per_group=%d not in {0,1,2,4}", g);
  int w = c->waves_per_group;
  if (w < 0 || w > 8) return sfail(AMH_E_INVAL, "waves_per_group=%d outside [0, 8]", w);
  if (g == 0) {
    g = 4;
    while (g > 1 && ((size_t)c->n_chains < (size_t)g * 256 ||
                     amh::sweep_lds_bytes(g, c->L, w ? w : (2 * g > 4 ? 2 * g : 4)) > kMaxLds))
      g >>= 1;
  }
  if (w == 0) {
    // eight waves (two per SIMD, the most the register budget allows) when the grid
    // gives each workgroup a compute unit of its own, else 2G (at least 4) so that
    // two workgroups share a compute unit
    const int64_t grid = ((int64_t)c->n_chains + g - 1) / g;
    w = 2 * g > 4 ? 2 * g : 4;
    if (grid <= n_cu && amh::sweep_lds_bytes(g, c->L, 8) <= kMaxLds) w = 8;
  }
  if (w < g) return sfail(AMH_E_INVAL, "waves_per_group=%d < chains_per_group=%d", w, g);
  const size_t need = amh::sweep_lds_bytes(g, c->L, w);
  if (need > kMaxLds)
    return sfail(AMH_E_INVAL, "L=%d with %d chains per workgroup needs %zu bytes of LDS (> %zu)",
                c->L, g, need, kMaxLds);
  *G = g;
  *W = w;
  return AMH_OK;
}

void free_ctx(amh_ctx* x) {
  if (!x) return;
  (void)hipFree(x->slab);
  (void)hipFree(x->work);
  delete x;
}

template <typename T>
amh_status dev_alloc(T** p, size_t count) {
  hipError_t e = hipMalloc(reinterpret_cast<void**>(p), sizeof(T) * (count ? count : 1));
  if (e != hipSuccess) return sfail(AMH_E_NOMEM, "hipMalloc(%zu bytes): %s", sizeof(T) * count, hipGetErrorString(e));
  return AMH_OK;
}

amh::ConfParams conf_base(const amh_ctx* x) {
  amh::ConfParams P{};
  P.L = x->cfg.L;
  P.table = x->table;
  P.stride = x->stride;
  P.nb = x->cfg.n_bins;
  P.d_min = x->cfg.d_min;
  P.bin_w = x->cfg.bin_w;
  P.vfar = x->vfar;
  P.err = x->err;
  return P;
}

int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
    n = 256;
  return n;
}

// Threads of a conformation's workgroup (energy and anchor kernels): the 16 wavefronts that a unit
// holds are divided among its conformations (128 registers a lane), but a short chain has no work
// for them and waits for their start and barriers.  Energies with 4 wavefronts throughout and so,
// us: one conformation of 300 residues 42 and 25, 256 of them 120 and 68, 64 of 500 186 and 97;
// 1024 of 300 have 4 still.  With 16, 4 and 2: 256 of 16 residues 10.2, 8.4 and 8.2, of 32 11.4, 10.3
// and 10.9, of 64 13.6, 14.6 and 20.0.  Coordinates alone take 4: 16 are no faster
// (L = 300: 1 conformation 29 against 27 us, 256 34 against 40).
int conf_threads(int64_t B, int L) {
  const int64_t per_cu = (B + compute_units() - 1) / compute_units();
  return std::min(per_cu <= 1 ? 1024 : per_cu <= 2 ? 512 : 256, L <= 16 ? 128 : L <= 40 ? 256 : 1024);
}

// Shape of a conformation's workgroup in the gradient and L-BFGS kernels: threads, of which a
// unit holds 512 (256 registers a lane; 16 wavefronts of 128 are slower by a quarter), and
// pairs a wavefront's list holds, as the LDS of the workgroups a unit is to hold allows.  One
// conformation a unit takes all 512 threads (gradients with 256 and 512, us: one of 200 residues 77
// and 59, of 300 80 and 57, 256 of 300 164 and 102, 64 of 800 424 and 277; of 100 residues and
// less the two lie together); more take 256, and from three a unit on 128 where there are three
// tiles at most (1024 of 16 residues with 256 and 128 34 and 22, of 64 92 and 62, of 100 100 and 82).
// Where two workgroups with lists of 256 pairs each do not fit a unit (from 471 residues on), it has
// one of 512 threads: 512 conformations of 500 residues with one of 256 threads, two of them with
// short lists and one of 512 468, 423 and 336 us, of 540 489, 531 and 341, of 800 911 and 599 (256
// threads with long lists against 512 with short ones: one of 830 residues 416 and 272).
// `few`: the wavefronts share tiles, where there are three at most and as many wavefronts (64
// residues: 512 conformations 34 us against 54 with a tile a wavefront, 1024 43 against 61), from
// 9 residues on (2: 13.1 against 12.4, 8: 13.9 and 13.8, 12: 14.9 against 16.1), and where their
// list holds any one tile (it does with the LDS of today's shapes).  With six tiles,
// 130 to 192 residues, and 8 wavefronts it is slower (200 conformations of 180 77 against 69).
// `least`: threads the kernel needs, `extra`: its LDS beyond the gradient's.
struct GradShape { int threads, cap; size_t lds; bool few; };

GradShape grad_shape(int L, int64_t B, int least, size_t extra) {
  const int n_cu = compute_units();
  GradShape s{B <= n_cu ? 512 : B > 2 * (int64_t)n_cu && L <= 128 ? 128 : 256, 0, 0, false};
  if (s.threads < least) s.threads = least;
  // (the kernels' own 256 bytes are the barrier votes')
  const auto bytes = [&](int cap) { return amh::grad_lds_bytes(L, s.threads / 64, cap) + extra + 256; };
  size_t room = kMaxLds / (512 / s.threads);   // of a workgroup, as many on a unit as it holds
  if (bytes(256) > room) {
    room = kMaxLds;
    s.threads = 512;
    if (bytes(256) > room) s.threads = 256;
  }
  s.cap = 64;
  while (s.cap < 2048 && bytes(s.cap + 8) <= room) s.cap += 8;
  s.lds = bytes(s.cap) - 256;
  const int ntile = L <= 64 ? 1 : 3;
  s.few = L > 8 && L <= (s.threads >= 256 ? 128 : 64) &&
          amh::grad_shared_pairs(s.threads / 64, s.cap, ntile) >= (ntile == 1 ? 2016 : 4096);
  return s;
}

amh_status launch_conf(const amh::ConfParams& P, int B, hipStream_t st) {
  if (B <= 0) return AMH_OK;
  const int threads = P.table ? conf_threads(B, P.L) : 256;
  const size_t lds = amh::conf_lds_bytes(P.L, threads, P.table != nullptr);
  HIP_OK(hipFuncSetAttribute((const void*)amh::conf_energy_kernel,
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(amh::conf_energy_kernel, dim3(B), dim3(threads), lds, st, P);
  HIP_OK(hipGetLastError());
  return AMH_OK;
}

amh::SweepParams sweep_params(const amh_ctx* x, int64_t n_sweeps) {
  const amh_config& c = x->cfg;
  amh::SweepParams P{};
  P.table = x->table;
  P.ydev = x->ydev;
  P.zrow = x->ydev + (size_t)c.L * (c.L - 1) / 2 * x->stride;
  P.stride = x->stride;
  P.nb = c.n_bins;
  P.inv_w = (float)(1.0 / c.bin_w);
  P.off = (float)((c.d_min + 0.5 * c.bin_w) / c.bin_w);
  P.tmax = (float)(c.n_bins - 1);
  P.d2far = amh::last_knot2(c.d_min, c.bin_w, c.n_bins);
  P.d_min = c.d_min;
  P.bin_w = c.bin_w;
  P.vfar = x->vfar;
  P.L = c.L;
  P.C = c.n_chains;
  P.half_window = amh::half_window(c.window_d, c.L);
  P.n_cascade = c.n_cascade;
  for (int i = 0; i < 3; ++i) P.cascade_hw[i] = i < c.n_cascade ? amh::half_window(c.cascade_d[i], c.L) : 0;
  P.sigma_end = c.sigma_end;
  P.global_every = c.global_every;
  P.n_global = c.n_global < 1 ? 1 : c.n_global;
  P.anchor_every = c.anchor_every;
  P.sigma = c.sigma;
  P.T0 = c.T0;
  P.T1 = c.T1;
  P.S = c.total_sweeps;
  P.t0 = x->t;
  P.n_sweeps = n_sweeps;
  P.key0 = (uint32_t)c.seed;
  P.key1 = (uint32_t)(c.seed >> 32);
  P.chain_offset = c.chain_offset;
  P.spin_limit = x->spin_limit;
  P.target = x->target;
  P.s = x->s;
  P.s_best = x->s_best;
  P.atoms = x->atoms;
  P.v = x->v;
  P.counters = x->counters;
  P.err = x->err;
  P.n_trace = x->n_trace;
  for (int m = 0; m < 4; ++m) P.trace_chain[m] = x->trace_chain[m];
  P.tr_dE = x->tr_dE;
  P.tr_delta = x->tr_delta;
  P.tr_acc = x->tr_acc;
  P.trace_cap = x->trace_cap;
  P.trace_t0 = x->trace_t0;
  P.tr_anchor = x->tr_anchor;
  P.trace_anchor_cap = x->trace_anchor_cap;
  P.trace_anchor0 = x->trace_anchor0;
  P.work = x->work_counters;
  return P;
}

amh_status read_err(amh_ctx* x, unsigned int* out) {
  HIP_OK(hipStreamSynchronize(x->stream));
  HIP_OK(hipMemcpy(out, x->err, sizeof(unsigned int), hipMemcpyDeviceToHost));
  return AMH_OK;
}

}  // namespace

namespace {

template <typename... Args>
amh_status launch(const void* fn, dim3 grid, int threads, size_t lds, hipStream_t st, Args&&... args) {
  HIP_OK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  void* a[] = {(void*)&args...};
  HIP_OK(hipLaunchKernel(fn, grid, dim3(threads), a, lds, st));
  return AMH_OK;
}

// What a launch takes against what a workgroup can have.
amh_status check_lds(size_t bytes, const char* what) {
  return bytes <= kMaxLds ? AMH_OK
                          : sfail(AMH_E_INVAL, "a %s launch needs %zu bytes of LDS (> %zu)", what, bytes, kMaxLds);
}

// Wavefronts a chain gets in a global-sweep workgroup of G chains and W wavefronts (a
// power of two; wavefronts left over idle).
int global_waves(int G, int W) {
  int nw = 1;
  while (2 * nw * G <= W && nw < 16) nw *= 2;
  return nw;
}

// Launch shape of an automatically shaped context's global sweeps, by the chains each
// compute unit gets (a unit holds 16 of the kernel's wavefronts, four per SIMD): one chain a
// workgroup, with as many wavefronts as the unit's chains leave room for.  A proposal of one
// chain shortens with its wavefronts, the work all chains share grows with them.  One global
// sweep with 2 / 4 / 8 / 16 wavefronts a chain, us:
//   L = 100: 128 chains  -   / 551  / 458  / -;    512  -   / 629  / 589  / -;
//            1024        887 / 748  / 1088 / -;   2048 1131 / 1389 / 2070 / -
//   L = 300: 256 chains  -   / 2964 / 1887 / 1747;  512  -   / 3571 / 2521 / -;
//            1024       5127 / 3654 / 4049 / -;   2048 7232 / 6192 / 7536 / -
//   L = 800: 64 chains   -   / 12313 / 7321 / 5801
// 16 where a unit has one chain and that is longer than 256 residues: it has the tiles to share.
// Below, 16 and 8 lie together (two sweeps with 8 / 16, us: 256 chains of 64 562 / 604, of 100 942 / 951,
// of 130 1502 / 1402, of 200 2234 / 2106, of 256 2755 / 2631; one chain of 130 1244 / 1206, of 160
// 1429 / 1450, of 256 2320 / 2342).  2 where every unit is full, up to 160 residues: eight such workgroups
// fill a unit, but from 225 residues on its LDS no longer holds them (two sweeps with 2 / 4, ms: 2048
// chains of 160 4.1 / 4.9, of 200 6.5 / 7.3, of 250 11.5 / 9.6, of 300 14.1 / 11.5; 1280 of 300, five a
// unit, 8.8 / 9.7).
int waves_per_chain(int64_t chains, int L, int n_cu) {
  const int64_t per_cu = (chains + n_cu - 1) / n_cu;
  return per_cu <= 1 ? (L > 256 ? 16 : 8) : per_cu <= 2 ? 8 : per_cu <= 4 || L > 160 ? 4 : 2;
}

// ... except that a context of four-chain groups, at most one a unit (1024 chains on 256 units),
// keeps the shape that amh_info_launches has reported for it, two chains and four wavefronts: two
// sweeps of 1024 chains of 300 residues take 9.2 ms so, 6.5 with four wavefronts a chain (1023 chains).
void global_shape(const amh_config* c, int n_cu, int G, int* G_global, int* W_global) {
  const bool reported = G == 4 && c->n_chains <= 4 * (int64_t)n_cu;
  *G_global = reported ? 2 : 1;
  *W_global = reported ? 4 : waves_per_chain(c->n_chains, c->L, n_cu);
}

const void* global_fn(int nw, bool batch) {
  switch (nw) {
    case 1: return batch ? (const void*)amh::global_batch_kernel<1> : (const void*)amh::global_kernel<1>;
    case 2: return batch ? (const void*)amh::global_batch_kernel<2> : (const void*)amh::global_kernel<2>;
    case 4: return batch ? (const void*)amh::global_batch_kernel<4> : (const void*)amh::global_kernel<4>;
    case 8: return batch ? (const void*)amh::global_batch_kernel<8> : (const void*)amh::global_kernel<8>;
    default: return batch ? (const void*)amh::global_batch_kernel<16> : (const void*)amh::global_kernel<16>;
  }
}

template <int G, bool CARRY>
const void* local_fn(bool batch) {
  return batch ? (const void*)amh::local_batch_kernel<G, CARRY> : (const void*)amh::local_kernel<G, CARRY>;
}

const void* local_fn(int G, bool carry, bool batch) {
  switch (G) {
    case 1: return carry ? local_fn<1, true>(batch) : local_fn<1, false>(batch);
    case 2: return carry ? local_fn<2, true>(batch) : local_fn<2, false>(batch);
    default: return carry ? local_fn<4, true>(batch) : local_fn<4, false>(batch);
  }
}

// The widest half-width of a context's localized sweeps.
int widest(const amh_ctx* x) {
  int h = amh::half_window(x->cfg.window_d, x->cfg.L);
  for (int i = 0; i < x->cfg.n_cascade; ++i) h = std::max(h, amh::half_window(x->cfg.cascade_d[i], x->cfg.L));
  return h;
}

// Whether localized launches of G chains a workgroup carry this context's energies along.
bool carries(const amh_ctx* x, int G) {
  return amh::carry_pays(G, widest(x), x->cfg.L) && amh::carry_exact(widest(x), x->cfg.L, x->dev_max);
}

// Localized launches of a context.  A unit holds one workgroup of the localized kernel (12 of
// its wavefronts), and takes 1 : 1.45 : 1.75 as long for one of 1 : 2 : 4 chains (L = 250, 9
// sweeps: 1.12, 1.60, 1.95 ms; L = 100: 0.59, 0.85, 1.03 ms).  So an automatically shaped
// context's chains go four to a workgroup (as LDS allows) while that fills every unit, and
// what is left to the fewest that give each workgroup a unit.  Before, with 1, 2 and 4 chains
// from 1, 512 and 1024 chains on throughout, L = 250: 476 chains 2.17 ms (two rounds), now
// 1.60; 768 chains 3.11, now 1.92; 1500 chains 3.82, now 3.57.
void local_parts(amh_ctx* x, int n_cu) {
  const amh_config& c = x->cfg;
  if (c.chains_per_group != 0 || c.waves_per_group != 0) {
    x->local[0] = {0, c.n_chains, x->G};
    x->n_local = 1;
    return;
  }
  const auto part = [&](int first, int chains, int G) { x->local[x->n_local++] = {first, chains, G}; };
  int most = 4;
  while (most > 1 && amh::local_lds_bytes(most, c.L, kLocalWaves) > kMaxLds) most >>= 1;
  const int64_t round = (int64_t)most * n_cu;
  const int whole = (int)(c.n_chains / round * round), rest = c.n_chains - whole;
  int G = 1;
  while (G < most && rest > (int64_t)G * n_cu) G *= 2;
  x->n_local = 0;
  if (whole > 0) part(0, whole, most);
  if (rest > 0) part(whole, rest, G);
}

size_t local_launch_lds(const amh_ctx* x) {
  return amh::local_lds_bytes(x->local[0].G, x->cfg.L, kLocalWaves);   // (the first of two has most chains)
}

size_t global_launch_lds(const amh_ctx* x) {
  return amh::global_lds_bytes(x->G_global, x->cfg.L, global_waves(x->G_global, x->W_global));
}

}  // namespace

namespace {

// amh_minimize (workspace owned by the context, grown with hipMalloc) and
// amh_minimize_noalloc (workspace = this device's fixed scratch array).
amh_status minimize_impl(amh_ctx* x, double* s_dev, int32_t B, const amh_lbfgs_opts* o,
                         double* V_out_dev, int32_t* iters_out_dev, int32_t* status_out_dev,
                         double* f_trace_dev, double* x_trace_dev, bool no_alloc) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (!o) return sfail(AMH_E_INVAL, "opts is NULL");
  if (B < 0) return sfail(AMH_E_INVAL, "B < 0");
  if (!s_dev && B != x->cfg.n_chains)
    return sfail(AMH_E_INVAL, "B=%d must equal n_chains=%d when s is NULL", B, x->cfg.n_chains);
  if (o->n_iter < 0) return sfail(AMH_E_INVAL, "n_iter=%d < 0", o->n_iter);
  if (o->m < 1 || o->m > amh::kLbfgsMaxHistory)
    return sfail(AMH_E_INVAL, "m=%d outside [1, %d]", o->m, amh::kLbfgsMaxHistory);
  if (o->nonmonotone < 1 || o->nonmonotone > amh::kLbfgsMaxNonmonotone)
    return sfail(AMH_E_INVAL, "nonmonotone=%d outside [1, %d]", o->nonmonotone, amh::kLbfgsMaxNonmonotone);
  if (o->max_ls < 1) return sfail(AMH_E_INVAL, "max_ls=%d < 1", o->max_ls);
  if (!(o->c1 > 0.0 && o->c1 < 1.0)) return sfail(AMH_E_INVAL, "c1 must lie in (0, 1)");
  if (!(o->shrink > 0.0 && o->shrink < 1.0)) return sfail(AMH_E_INVAL, "shrink must lie in (0, 1)");
  if (!(o->gtol >= 0.0) || !std::isfinite(o->gtol)) return sfail(AMH_E_INVAL, "gtol must be finite and >= 0");
  if (!(o->step0 > 0.0) || !std::isfinite(o->step0)) return sfail(AMH_E_INVAL, "step0 must be finite and > 0");
  if (B == 0) return AMH_OK;
  const int L = x->cfg.L;
  const size_t need = amh::lbfgs_work_doubles(L, o->m) * (size_t)B;
  double* work = x->work;
  if (no_alloc) {
    if (need > (size_t)amh::kNoallocScratchDoubles)
      return sfail(AMH_E_INVAL,
                   "B=%d conformations of L=%d with m=%d need %zu workspace doubles; the fixed "
                   "scratch holds %lld (B (5 + 2m) 2L <= %lld)", B, L, o->m, need,
                   (long long)amh::kNoallocScratchDoubles, (long long)amh::kNoallocScratchDoubles);
    if (!x->scratch) return sfail(AMH_E_DEVICE, "the scratch array has no device address");
    work = x->scratch;
  } else if (need > x->work_n) {
    HIP_OK(hipStreamSynchronize(x->stream));
    (void)hipFree(x->work);
    x->work = nullptr;
    x->work_n = 0;
    amh_status st = dev_alloc(&x->work, need);
    if (st != AMH_OK) return st;
    x->work_n = need;
    work = x->work;
  }
  amh::LbfgsParams P{};
  P.L = L;
  P.s = s_dev ? s_dev : x->s;
  P.table = x->table;
  P.stride = x->stride;
  P.nb = x->cfg.n_bins;
  P.d_min = x->cfg.d_min;
  P.bin_w = x->cfg.bin_w;
  P.vfar = x->vfar;
  P.ordered = amh::ordered_energies(x->dev_max);
  P.n_iter = o->n_iter;
  P.m = o->m;
  P.nonmonotone = o->nonmonotone;
  P.max_ls = o->max_ls;
  P.c1 = o->c1;
  P.shrink = o->shrink;
  P.gtol = o->gtol;
  P.step0 = o->step0;
  P.work = work;
  P.V = V_out_dev;
  P.iters = iters_out_dev;
  P.status = status_out_dev;
  P.f_trace = f_trace_dev;
  P.x_trace = x_trace_dev;
  P.err = x->err;
  if (!s_dev) {   // the context's chains: keep V, the best state and the coordinates current
    P.v_state = x->v;
    P.s_best = x->s_best;
  }
  const size_t history = amh::lbfgs_lds_bytes(L, 0, 0, o->m, o->nonmonotone) - amh::grad_lds_bytes(L, 0, 0);
  const GradShape shape = grad_shape(L, B, amh::kReduceThreads, history);
  const size_t lds = shape.lds;
  P.cap = shape.cap;
  if (lds > kMaxLds) return sfail(AMH_E_INVAL, "L=%d needs %zu bytes of LDS for L-BFGS", L, lds);
  const auto kernel = shape.few ? amh::lbfgs_kernel<true> : amh::lbfgs_kernel<false>;
  HIP_OK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kernel, dim3(B), dim3(shape.threads), lds, x->stream, P);
  HIP_OK(hipGetLastError());
  if (!s_dev) {
    amh::ConfParams cp{};
    cp.L = L;
    cp.s_in = x->s;
    cp.atoms64_out = x->atoms;
    return launch_conf(cp, B, x->stream);
  }
  return AMH_OK;
}

}  // namespace

extern "C" {

const char* amh_last_error(void) { return g_last_error.c_str(); }

amh_status amh_init(const amh_config* cfg, const float* y_dev, const double* s0_dev, void* stream,
                    amh_ctx** out) {
  if (!out) return sfail(AMH_E_INVAL, "out is NULL");
  *out = nullptr;
  int G = 0, W = 0;
  int dev = 0;
  const bool have_dev = hipGetDevice(&dev) == hipSuccess;
  const int n_cu = compute_units();
  amh_status st = validate(cfg, n_cu, &G, &W);
  if (st != AMH_OK) return st;
  if (!y_dev) return sfail(AMH_E_INVAL, "distogram table is NULL");
  if (!have_dev) return sfail(AMH_E_DEVICE, "no current HIP device");
  double* scratch_dev = nullptr;
  if ((st = scratch_address(dev, &scratch_dev)) != AMH_OK) return st;
  amh_ctx* x = new amh_ctx;
  x->cfg = *cfg;
  x->scratch = scratch_dev;
  x->stream = reinterpret_cast<hipStream_t>(stream);
  x->G = G;
  x->W = W;
  local_parts(x, n_cu);
  // global sweeps of an automatically shaped context
  x->G_global = G;
  x->W_global = W;
  if (cfg->chains_per_group == 0 && cfg->waves_per_group == 0) global_shape(cfg, n_cu, G, &x->G_global, &x->W_global);
  if ((st = check_lds(local_launch_lds(x), "localized")) != AMH_OK ||
      (st = check_lds(global_launch_lds(x), "global")) != AMH_OK) {
    free_ctx(x);
    return st;
  }
  const int L = cfg->L, C = cfg->n_chains, n = 2 * L;
  const int64_t P = (int64_t)L * (L - 1) / 2;
  x->stride = row_stride(cfg->n_bins);
  // one allocation a context: an allocation and its release cost 17 us of host time together,
  // of eight arrays 0.8 ms for six served jobs
  const int ingest_blocks = (int)std::min<int64_t>((P * x->stride + 255) / 256, 4096);
  size_t used = 0;
  const auto take = [&](size_t bytes) {
    const size_t at = used;
    used += (bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t o_table = take(sizeof(float) * P * x->stride), o_ydev = take(sizeof(float) * (P + 1) * x->stride),
               o_s = take(sizeof(double) * C * n), o_best = take(sizeof(double) * C * n),
               o_atoms = take(sizeof(double) * C * L * 12), o_v = take(sizeof(double) * C * 2),
               o_cnt = take(sizeof(int64_t) * C * 4), o_err = take(sizeof(TableFacts)),
               o_most = take(sizeof(float) * ingest_blocks);
  if ((st = dev_alloc(&x->slab, used)) != AMH_OK) {
    free_ctx(x);
    return st;
  }
  x->table = reinterpret_cast<float*>(x->slab + o_table);
  x->ydev = reinterpret_cast<float*>(x->slab + o_ydev);
  x->s = reinterpret_cast<double*>(x->slab + o_s);
  x->s_best = reinterpret_cast<double*>(x->slab + o_best);
  x->atoms = reinterpret_cast<double*>(x->slab + o_atoms);
  x->v = reinterpret_cast<double*>(x->slab + o_v);
  x->counters = reinterpret_cast<int64_t*>(x->slab + o_cnt);
  x->err = reinterpret_cast<unsigned int*>(x->slab + o_err);
  float* const most = reinterpret_cast<float*>(x->slab + o_most);
  hipError_t e = hipMemsetAsync(x->err, 0, sizeof(TableFacts), x->stream);
  if (e == hipSuccess)   // row P of the deviation table is the zero row
    e = hipMemsetAsync(x->ydev + (size_t)P * x->stride, 0, sizeof(float) * x->stride, x->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(amh::ingest_kernel, dim3(ingest_blocks), dim3(256), 0, x->stream, y_dev, P,
                       cfg->n_bins, x->stride, x->table, x->ydev, most, x->err);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {   // the energy of the all-far conformation, read back once
    TableFacts* const facts = reinterpret_cast<TableFacts*>(x->err);
    TableFacts got{};
    hipLaunchKernelGGL(amh::far_sum_kernel, dim3(1), dim3(512), 0, x->stream, x->table, P, x->stride,
                       cfg->n_bins, most, ingest_blocks, &facts->vfar, &facts->dev_max);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&got, facts, sizeof(got), hipMemcpyDeviceToHost, x->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(x->stream);
    x->vfar = got.vfar;
    x->dev_max = got.dev_max;
  }
  if (e == hipSuccess && s0_dev)
    e = hipMemcpyAsync(x->s, s0_dev, sizeof(double) * C * n, hipMemcpyDeviceToDevice, x->stream);
  if (e != hipSuccess) {
    free_ctx(x);
    return sfail(AMH_E_DEVICE, "amh_init: %s", hipGetErrorString(e));
  }
  amh::ConfParams cp = conf_base(x);
  cp.s_in = s0_dev ? x->s : nullptr;
  cp.s_out = s0_dev ? nullptr : x->s;
  cp.atoms64_out = x->atoms;
  cp.v_state = x->v;
  cp.counters = x->counters;
  cp.s_best = x->s_best;
  if ((st = launch_conf(cp, C, x->stream)) != AMH_OK) { free_ctx(x); return st; }
  unsigned int err = 0;
  if ((st = read_err(x, &err)) != AMH_OK) { free_ctx(x); return st; }
  if (err) {
    free_ctx(x);
    return sfail(AMH_E_NUMERIC, (err & amh::kErrTable) ? "distogram table holds a non-finite entry"
                                                       : "initial energy is not finite");
  }
  *out = x;
  return AMH_OK;
}

amh_status amh_sweep(amh_ctx* x, int64_t n_sweeps) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (n_sweeps < 0) return sfail(AMH_E_INVAL, "n_sweeps < 0");
  if (x->t + n_sweeps > x->cfg.total_sweeps)
    return sfail(AMH_E_INVAL, "sweep %lld + %lld passes total_sweeps=%lld", (long long)x->t,
                (long long)n_sweeps, (long long)x->cfg.total_sweeps);
  if (n_sweeps == 0) return AMH_OK;
  amh::SweepParams P = sweep_params(x, n_sweeps);
  const amh_config& c = x->cfg;
  // one launch per run of sweeps of one kind (localized or global) and one per anchor, in
  // order on the stream; a launch boundary between two sweeps does not change any result
  const int64_t end = x->t + n_sweeps;
  for (int64_t t = x->t; t < end;) {
    const bool glob = amh::is_global(P, t);
    const int64_t e = amh::run_end(P, t, end);
    P.t0 = t;
    P.n_sweeps = e - t;
    amh_status st = AMH_OK;
    if (glob) {
      const int G = x->G_global, nw = global_waves(G, x->W_global);
      st = launch(global_fn(nw, false), dim3((c.n_chains + G - 1) / G), 64 * x->W_global,
                  amh::global_lds_bytes(G, c.L, nw), x->stream, P, G);
    }
    for (int i = 0; !glob && i < x->n_local && st == AMH_OK; ++i) {
      const auto& l = x->local[i];
      P.chain0 = l.first;
      P.C = l.first + l.chains;
      st = launch(local_fn(l.G, carries(x, l.G), false), dim3((l.chains + l.G - 1) / l.G),
                  64 * kLocalWaves, amh::local_lds_bytes(l.G, c.L, kLocalWaves), x->stream, P);
    }
    P.C = c.n_chains;
    if (st == AMH_OK && e % c.anchor_every == 0) {
      P.t0 = e;
      const int threads = conf_threads(c.n_chains, c.L);
      st = launch((const void*)amh::anchor_kernel, dim3(c.n_chains), threads,
                  amh::conf_lds_bytes(c.L, threads, true), x->stream, P);
    }
    if (st != AMH_OK) return st;
    t = e;
  }
  x->t += n_sweeps;
  return AMH_OK;
}

amh_status amh_energy(amh_ctx* x, const double* s_in_dev, int32_t B, int32_t which,
                      double* V_out_dev, double* s_out_dev, float* cb_out_dev) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (B < 0) return sfail(AMH_E_INVAL, "B < 0");
  amh::ConfParams P = conf_base(x);
  if (s_in_dev) {
    P.s_in = s_in_dev;
  } else {
    if (B != x->cfg.n_chains) return sfail(AMH_E_INVAL, "B=%d must equal n_chains=%d", B, x->cfg.n_chains);
    if (which != 0 && which != 1) return sfail(AMH_E_INVAL, "which=%d not in {0, 1}", which);
    P.s_in = which == 0 ? x->s : x->s_best;
  }
  P.V_out = V_out_dev;
  P.s_out = s_out_dev;
  P.cb_out = cb_out_dev;
  return launch_conf(P, B, x->stream);
}

amh_status amh_conformation(const double* s_dev, int32_t B, int32_t L, float* atoms_out_dev,
                            void* stream) {
  if (!s_dev || !atoms_out_dev) return sfail(AMH_E_INVAL, "NULL pointer");
  if (B < 0 || L < 2 || L > 1024) return sfail(AMH_E_INVAL, "B=%d, L=%d out of range", B, L);
  amh::ConfParams P{};
  P.L = L;
  P.s_in = s_dev;
  P.atoms_out = atoms_out_dev;
  return launch_conf(P, B, reinterpret_cast<hipStream_t>(stream));
}

amh_status amh_get_state(amh_ctx* x, double* s_dev, double* s_best_dev, double* v_dev,
                         int64_t* counters_dev, double* atoms_dev, int64_t* t_out) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  const size_t C = x->cfg.n_chains, n = 2 * (size_t)x->cfg.L;
  const auto D2D = hipMemcpyDeviceToDevice;
  if (s_dev) HIP_OK(hipMemcpyAsync(s_dev, x->s, sizeof(double) * C * n, D2D, x->stream));
  if (s_best_dev) HIP_OK(hipMemcpyAsync(s_best_dev, x->s_best, sizeof(double) * C * n, D2D, x->stream));
  if (v_dev) HIP_OK(hipMemcpyAsync(v_dev, x->v, sizeof(double) * C * 2, D2D, x->stream));
  if (counters_dev) HIP_OK(hipMemcpyAsync(counters_dev, x->counters, sizeof(int64_t) * C * 4, D2D, x->stream));
  if (atoms_dev) HIP_OK(hipMemcpyAsync(atoms_dev, x->atoms, sizeof(double) * C * x->cfg.L * 12, D2D, x->stream));
  if (t_out) *t_out = x->t;
  return AMH_OK;
}

amh_status amh_set_state(amh_ctx* x, const double* s_dev, const double* s_best_dev,
                         const double* v_dev, const int64_t* counters_dev, const double* atoms_dev,
                         int64_t t) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (t < 0 || t > x->cfg.total_sweeps) return sfail(AMH_E_INVAL, "t=%lld out of range", (long long)t);
  const size_t C = x->cfg.n_chains, n = 2 * (size_t)x->cfg.L;
  const auto D2D = hipMemcpyDeviceToDevice;
  if (s_dev) HIP_OK(hipMemcpyAsync(x->s, s_dev, sizeof(double) * C * n, D2D, x->stream));
  if (s_best_dev) HIP_OK(hipMemcpyAsync(x->s_best, s_best_dev, sizeof(double) * C * n, D2D, x->stream));
  if (v_dev) HIP_OK(hipMemcpyAsync(x->v, v_dev, sizeof(double) * C * 2, D2D, x->stream));
  if (counters_dev) HIP_OK(hipMemcpyAsync(x->counters, counters_dev, sizeof(int64_t) * C * 4, D2D, x->stream));
  if (atoms_dev) {
    HIP_OK(hipMemcpyAsync(x->atoms, atoms_dev, sizeof(double) * C * x->cfg.L * 12, D2D, x->stream));
  } else if (s_dev) {
    amh::ConfParams P{};
    P.L = x->cfg.L;
    P.s_in = x->s;
    P.atoms64_out = x->atoms;
    amh_status st = launch_conf(P, (int)C, x->stream);
    if (st != AMH_OK) return st;
  }
  x->t = t;
  return AMH_OK;
}

amh_status amh_perturb(amh_ctx* x, double amplitude, uint32_t tag) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (!(amplitude >= 0.0) || !std::isfinite(amplitude)) return sfail(AMH_E_INVAL, "amplitude must be finite and >= 0");
  const amh_config& c = x->cfg;
  const int64_t total = (int64_t)c.n_chains * 2 * c.L;
  int blocks = (int)((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(amh::perturb_kernel, dim3(blocks), dim3(256), 0, x->stream, x->s, total, 2 * c.L,
                     c.chain_offset, tag, (uint32_t)c.seed, (uint32_t)(c.seed >> 32), amplitude);
  HIP_OK(hipGetLastError());
  amh::ConfParams P = conf_base(x);   // rebuild coordinates, re-anchor V, keep the best
  P.s_in = x->s;
  P.atoms64_out = x->atoms;
  P.v_state = x->v;
  P.s_best = x->s_best;
  P.keep_best = 1;
  return launch_conf(P, c.n_chains, x->stream);
}

amh_status amh_set_wait_bound(amh_ctx* x, int32_t polls) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (polls < 1 || polls > (1 << 24)) return sfail(AMH_E_INVAL, "polls=%d outside [1, 2^24]", polls);
  x->spin_limit = polls;
  return AMH_OK;
}

amh_status amh_set_target(amh_ctx* x, double target) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (std::isnan(target)) return sfail(AMH_E_INVAL, "target is NaN");
  x->target = target;
  return AMH_OK;
}

amh_status amh_set_trace(amh_ctx* x, int32_t n, const int32_t* chain_ids, double* dE_dev,
                         double* delta_dev, uint8_t* acc_dev, int64_t capacity, double* anchor_dev,
                         int64_t anchor_capacity) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (n < 0 || n > 4) return sfail(AMH_E_INVAL, "n=%d outside [0, 4]", n);
  if (n > 0 && (!chain_ids || !dE_dev || !delta_dev || !acc_dev || capacity < 0 || anchor_capacity < 0 ||
                (anchor_capacity > 0 && !anchor_dev)))
    return sfail(AMH_E_INVAL, "trace buffers missing");
  for (int m = 0; m < 4; ++m) {
    x->trace_chain[m] = (m < n) ? chain_ids[m] : -1;
    if (m < n && (chain_ids[m] < -1 || chain_ids[m] >= x->cfg.n_chains))
      return sfail(AMH_E_INVAL, "trace chain %d out of range", chain_ids[m]);
  }
  x->n_trace = n;
  x->tr_dE = dE_dev;
  x->tr_delta = delta_dev;
  x->tr_acc = acc_dev;
  x->trace_cap = capacity;
  x->trace_t0 = x->t;
  x->tr_anchor = anchor_dev;
  x->trace_anchor_cap = anchor_capacity;
  x->trace_anchor0 = x->t / x->cfg.anchor_every + 1;
  return AMH_OK;
}

amh_status amh_set_work_counters(amh_ctx* x, int64_t* counters_dev) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  x->work_counters = reinterpret_cast<unsigned long long*>(counters_dev);
  return AMH_OK;
}

amh_status amh_poll(amh_ctx* x) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  unsigned int err = 0;
  amh_status st = read_err(x, &err);
  if (st != AMH_OK) return st;
  if (err & amh::kErrStall) return sfail(AMH_E_DEVICE, "a pipelined localized sweep exceeded its wait bound");
  if (err) return sfail(AMH_E_NUMERIC, "non-finite %s", (err & amh::kErrTable) ? "table entry" : "energy");
  return AMH_OK;
}

amh_status amh_info(amh_ctx* x, int32_t* G, int32_t* W, int32_t* lds, int64_t* t) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (G) *G = x->G;
  if (W) *W = x->W;
  if (lds) *lds = (int32_t)std::max(local_launch_lds(x), global_launch_lds(x));
  if (t) *t = x->t;
  return AMH_OK;
}

amh_status amh_info_launches(amh_ctx* x, int32_t* local_G, int32_t* local_W, int32_t* local_lds,
                             int32_t* global_G, int32_t* global_W, int32_t* global_lds) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (local_G) *local_G = x->local[0].G;
  if (local_W) *local_W = kLocalWaves;
  if (local_lds) *local_lds = (int32_t)local_launch_lds(x);
  if (global_G) *global_G = x->G_global;
  if (global_W) *global_W = x->W_global;
  if (global_lds) *global_lds = (int32_t)global_launch_lds(x);
  return AMH_OK;
}

amh_status amh_philox(const uint32_t* ctr_dev, int64_t n, uint64_t key, uint32_t* out_dev,
                      void* stream) {
  if (n < 0 || (n > 0 && (!ctr_dev || !out_dev))) return sfail(AMH_E_INVAL, "bad philox arguments");
  if (n == 0) return AMH_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(amh::philox_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), ctr_dev, n, (uint32_t)key,
                     (uint32_t)(key >> 32), out_dev);
  HIP_OK(hipGetLastError());
  return AMH_OK;
}

amh_status amh_grad(amh_ctx* x, const double* s_dev, int32_t B, double* V_out_dev, double* g_out_dev) {
  if (!x) return sfail(AMH_E_INVAL, "ctx is NULL");
  if (B < 0) return sfail(AMH_E_INVAL, "B < 0");
  if (!s_dev && B != x->cfg.n_chains)
    return sfail(AMH_E_INVAL, "B=%d must equal n_chains=%d when s is NULL", B, x->cfg.n_chains);
  if (!V_out_dev && !g_out_dev) return sfail(AMH_E_INVAL, "V_out and g_out are both NULL");
  if (B == 0) return AMH_OK;
  amh::GradParams P{};
  P.L = x->cfg.L;
  P.s = s_dev ? s_dev : x->s;
  P.table = x->table;
  P.stride = x->stride;
  P.nb = x->cfg.n_bins;
  P.d_min = x->cfg.d_min;
  P.bin_w = x->cfg.bin_w;
  P.vfar = x->vfar;
  P.ordered = amh::ordered_energies(x->dev_max);
  P.V = V_out_dev;
  P.g = g_out_dev;
  P.err = x->err;
  const GradShape shape = grad_shape(P.L, B, 64, 0);
  const size_t lds = shape.lds;
  P.cap = shape.cap;
  if (lds > kMaxLds) return sfail(AMH_E_INVAL, "L=%d needs %zu bytes of LDS for the gradient", P.L, lds);
  const auto kernel = shape.few ? amh::grad_kernel<true> : amh::grad_kernel<false>;
  HIP_OK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(kernel, dim3(B), dim3(shape.threads), lds, x->stream, P);
  HIP_OK(hipGetLastError());
  return AMH_OK;
}

amh_status amh_minimize(amh_ctx* x, double* s_dev, int32_t B, const amh_lbfgs_opts* o,
                        double* V_out_dev, int32_t* iters_out_dev, int32_t* status_out_dev,
                        double* f_trace_dev, double* x_trace_dev) {
  return minimize_impl(x, s_dev, B, o, V_out_dev, iters_out_dev, status_out_dev, f_trace_dev,
                       x_trace_dev, false);
}

amh_status amh_minimize_noalloc(amh_ctx* x, double* s_dev, int32_t B, const amh_lbfgs_opts* o,
                                double* V_out_dev, int32_t* iters_out_dev, int32_t* status_out_dev,
                                double* f_trace_dev, double* x_trace_dev) {
  return minimize_impl(x, s_dev, B, o, V_out_dev, iters_out_dev, status_out_dev, f_trace_dev,
                       x_trace_dev, true);
}

amh_status amh_destroy(amh_ctx* x) {
  if (!x) return AMH_OK;
  (void)hipStreamSynchronize(x->stream);
  free_ctx(x);
  return AMH_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batches: several contexts (proteins of different lengths) advanced by shared launches,
// one per launch shape and kind of sweep.

namespace {

constexpr int kRing = 8;   // pinned descriptor staging buffers in flight
constexpr int kMaxRuns = 8;   // descriptor sets (one a launch) uploaded together
constexpr int kLanes = 4;     // groups of members advanced side by side (hardware queues)
// launch plans: 0 = each context's own shape, then uniform (chains per group, waves)
constexpr int kPlans = 6;
constexpr int kPlanShape[kPlans][2] = {{0, 0}, {1, 4}, {2, 4}, {2, 8}, {4, 4}, {4, 8}};

// What a lane of a batch's sweeps is launched with: a stream, the parameter blocks of its steps
// (staged in a ring of pinned buffers) and its own list of workgroups.
struct Lane {
  hipStream_t stream = nullptr;
  amh::SweepParams* d_desc = nullptr;   // [kMaxRuns][members]
  amh::SweepParams* h_ring = nullptr;   // pinned, kRing of these
  hipEvent_t ev[kRing] = {};
  bool ev_used[kRing] = {};
  int ring = 0;
  // where a batch takes several: their workgroups (of all launches in turn; staged in kRing
  // buffers too) and the event that the batch's stream waits for
  int2* d_map = nullptr;
  int2* h_map = nullptr;   // pinned
  hipEvent_t done = nullptr;
};

}  // namespace

struct amh_batch {
  std::vector<amh_ctx*> m;
  hipStream_t stream = nullptr;
  int plan = 0;
  struct Launch {
    int G = 1, W = 4;
    int W_global = 4;                // wavefronts of a global launch
    bool carry = false;              // localized launches carry their energies along
    size_t lds_local = 0, lds_global = 0, lds_anchor = 0;   // of the longest member
    int anchor_threads = 256;
    std::vector<int2> map;           // workgroups: (member, chain group)
    int2* d_map = nullptr;
  };
  std::vector<Launch> launches;
  Lane lane[kLanes];
  hipEvent_t fork = nullptr;
};

namespace {

void free_launches(amh_batch* b) {
  for (auto& l : b->launches) (void)hipFree(l.d_map);
  b->launches.clear();
  for (Lane& l : b->lane) {
    (void)hipFree(l.d_map);
    if (l.h_map) (void)hipHostFree(l.h_map);
    l.d_map = l.h_map = nullptr;
  }
}

void free_batch(amh_batch* b) {
  if (!b) return;
  free_launches(b);
  for (Lane& l : b->lane) {
    (void)hipFree(l.d_desc);
    if (l.h_ring) (void)hipHostFree(l.h_ring);
    for (hipEvent_t e : l.ev)
      if (e) (void)hipEventDestroy(e);
    if (l.done) (void)hipEventDestroy(l.done);
    if (&l != b->lane && l.stream) (void)hipStreamDestroy(l.stream);
  }
  if (b->fork) (void)hipEventDestroy(b->fork);
  delete b;
}

int workgroups(const amh_batch* b) {
  int wg = 0;
  for (const auto& l : b->launches) wg += (int)l.map.size();
  return wg;
}

// The buffers and events of lane i, made on its first use, alone or as one of `several`.
amh_status ready_lane(amh_batch* b, int i, bool several) {
  Lane& l = b->lane[i];
  const size_t n = b->m.size();
  hipError_t e = hipSuccess;
  const auto event = [&](hipEvent_t* ev) {
    if (e == hipSuccess && !*ev) e = hipEventCreateWithFlags(ev, hipEventDisableTiming);
  };
  if (!l.d_desc) e = hipMalloc(reinterpret_cast<void**>(&l.d_desc), sizeof(amh::SweepParams) * kMaxRuns * n);
  // (one pinned allocation for the ring: 42 us of host time each, with its release)
  if (e == hipSuccess && !l.h_ring)
    e = hipHostMalloc(reinterpret_cast<void**>(&l.h_ring), sizeof(amh::SweepParams) * kMaxRuns * n * kRing);
  for (hipEvent_t& ev : l.ev) event(&ev);
  if (several) {
    event(&b->fork);
    event(&l.done);
    const size_t wg = workgroups(b);
    if (e == hipSuccess && !l.stream && i > 0) e = hipStreamCreateWithFlags(&l.stream, hipStreamNonBlocking);
    if (e == hipSuccess && !l.d_map) e = hipMalloc(reinterpret_cast<void**>(&l.d_map), sizeof(int2) * wg);
    if (e == hipSuccess && !l.h_map) e = hipHostMalloc(reinterpret_cast<void**>(&l.h_map), sizeof(int2) * wg * kRing);
  }
  return e == hipSuccess ? AMH_OK : sfail(AMH_E_NOMEM, "batch buffers: %s", hipGetErrorString(e));
}

void member_shape(const amh_ctx* x, int plan, int* G, int* W) {
  if (plan == 0) { *G = x->G; *W = x->W; return; }
  int g = kPlanShape[plan][0], w = kPlanShape[plan][1];
  while (g > 1 && amh::sweep_lds_bytes(g, x->cfg.L, w) > kMaxLds) g >>= 1;
  *G = g;
  *W = w;
}

// Work of one chain group per sweep, in pair evaluations (orders the grid only).
double member_cost(const amh_ctx* x) {
  const double L = x->cfg.L, h = x->cfg.window_d / 2;
  const int ge = x->cfg.global_every;
  const double fg = ge > 0 ? (double)(x->cfg.n_global < 1 ? 1 : x->cfg.n_global) / ge : 0.0;
  const double global = L * L * L / 3.0 * fg;
  const double local = 2.0 * L * h * (h + 1) * (1.0 - fg);
  return global + local;
}

amh_status build_launches(amh_batch* b, int plan) {
  HIP_OK(hipStreamSynchronize(b->stream));
  free_launches(b);
  std::vector<std::pair<int, int>> shapes;
  std::vector<int> shape_of(b->m.size());
  for (size_t i = 0; i < b->m.size(); ++i) {
    int G, W;
    member_shape(b->m[i], plan, &G, &W);
    auto it = std::find(shapes.begin(), shapes.end(), std::make_pair(G, W));
    shape_of[i] = (int)(it - shapes.begin());
    if (it == shapes.end()) shapes.emplace_back(G, W);
  }
  int64_t chains = 0;
  for (const amh_ctx* x : b->m) chains += x->cfg.n_chains;
  for (size_t s = 0; s < shapes.size(); ++s) {
    amh_batch::Launch l;
    l.G = shapes[s].first;
    l.W = shapes[s].second;
    int longest = 2;
    bool automatic = true;   // no member has a shape of its caller's choice
    bool exact = true;       // every member's energies can be carried along
    const amh_ctx* most = nullptr;   // the member that takes longest
    std::vector<std::pair<double, int2>> items;
    for (size_t i = 0; i < b->m.size(); ++i) {
      if (shape_of[i] != (int)s) continue;
      const amh_ctx* x = b->m[i];
      longest = std::max(longest, x->cfg.L);
      exact = exact && amh::carry_exact(widest(x), x->cfg.L, x->dev_max);
      if (!most || member_cost(x) > member_cost(most)) most = x;
      automatic = automatic && x->cfg.chains_per_group == 0 && x->cfg.waves_per_group == 0;
      const int groups = (x->cfg.n_chains + l.G - 1) / l.G;
      for (int g = 0; g < groups; ++g) items.push_back({member_cost(x), make_int2((int)i, g)});
    }
    std::stable_sort(items.begin(), items.end(),
                     [](const auto& a, const auto& c) { return a.first > c.first; });
    for (auto& it : items) l.map.push_back(it.second);
    l.carry = exact && amh::carry_pays(l.G, widest(most), most->cfg.L);
    l.lds_local = amh::local_lds_bytes(l.G, longest, kLocalWaves);
    // (single-chain groups of the contexts' own shapes share the units with all the batch)
    l.W_global = plan == 0 && l.G == 1 && automatic ? waves_per_chain(chains, longest, compute_units()) : l.W;
    l.lds_global = amh::global_lds_bytes(l.G, longest, global_waves(l.G, l.W_global));
    l.anchor_threads = conf_threads((int64_t)l.map.size() * l.G, longest);
    l.lds_anchor = amh::conf_lds_bytes(longest, l.anchor_threads, true);
    for (const auto& need : {std::make_pair(l.lds_local, "localized"), std::make_pair(l.lds_global, "global"),
                             std::make_pair(l.lds_anchor, "anchor")}) {
      const amh_status st = check_lds(need.first, need.second);
      if (st != AMH_OK) return st;
    }
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&l.d_map), sizeof(int2) * l.map.size());
    if (e != hipSuccess) return sfail(AMH_E_NOMEM, "hipMalloc: %s", hipGetErrorString(e));
    b->launches.push_back(l);
    HIP_OK(hipMemcpy(l.d_map, l.map.data(), sizeof(int2) * l.map.size(), hipMemcpyHostToDevice));
  }
  b->plan = plan;
  return AMH_OK;
}

enum class Step { local, global, anchor };

// The launches of one step (one per shape) over the members' descriptors, on a lane's stream and
// workgroups (n_wg of each launch; null: all, on the batch's own lists).
amh_status launch_step(const amh_batch* b, const Lane& lane, const std::vector<int>* n_wg, Step kind,
                       const amh::SweepParams* descs) {
  size_t at = 0;
  for (size_t q = 0; q < b->launches.size(); ++q) {
    const auto& l = b->launches[q];
    const int2* map = n_wg ? lane.d_map + at : l.d_map;
    const int wg = n_wg ? (*n_wg)[q] : (int)l.map.size();
    at += wg;
    if (wg == 0) continue;
    const int G = l.G, nw = global_waves(l.G, l.W_global);
    const amh_status st =
        kind == Step::local
            ? launch(local_fn(G, l.carry, true), dim3(wg), 64 * kLocalWaves, l.lds_local, lane.stream, descs, map)
        : kind == Step::global
            ? launch(global_fn(nw, true), dim3(wg), 64 * l.W_global, l.lds_global, lane.stream, descs, map, G)
            : launch((const void*)amh::anchor_batch_kernel, dim3(wg, G), l.anchor_threads, l.lds_anchor, lane.stream,
                     descs, map, G);
    if (st != AMH_OK) return st;
  }
  return AMH_OK;
}

// A member's way through its sweeps: runs of one kind (run_end) and anchors.
struct Walk {
  amh::SweepParams P;
  int64_t t, end, anchored;
  // the sweeps of its next run if that is of the given kind, else 0; the walk goes on behind it
  int64_t run(bool glob) {
    if (t >= end || amh::is_global(P, t) != glob) return 0;
    const int64_t from = t;
    t = amh::run_end(P, t, end);
    return t - from;
  }
  // (a walk that did not advance in a step stands at an anchor it has already made, or at its start)
  bool anchor() {
    if (t == anchored || t % P.anchor_every != 0) return false;
    anchored = t;
    return true;
  }
};

// Time of the first steps of walks that share every step, each as long as its longest run: one
// localized sweep of L residues counts L, 8 more pipelined behind it 1.3 L, a global one (1.8 + L / 400) L,
// an anchor 10 + L / 20 (measured at 64, 300 and 800 residues).
double shared_time(std::vector<Walk> w) {
  double sum = 0.0;
  bool left = true;
  for (int step = 0; left && step < 128; ++step) {
    double run = 0.0, anchor = 0.0;
    left = false;
    for (Walk& x : w) {
      const double L = x.P.L, n = (double)x.run(step & 1);
      if (n > 0.0) run = std::max(run, L * (step & 1 ? n * (1.8 + L / 400.0) : 0.84 + 0.16 * n));
      if (x.anchor()) anchor = std::max(anchor, 10.0 + L / 20.0);
      left = left || x.t < x.end;
    }
    sum += run + anchor;
  }
  return sum;
}

// The lane of every member.  Members whose runs of sweeps and anchors fall together share their
// launches.  Where they do not, a shared step takes as long as its longest run and the others wait,
// which side by side they need not (40 sweeps of two proteins, in one lane / in two, ms: 64 chains of
// 40 residues each, anchors every 2 and 10 sweeps 5.1 / 3.5, cycles of 10 and localized only
// 3.2 / 2.2; of 300 residues, anchors every 1 and 1000 sweeps 40.1 / 31.7; 256 chains of 100, anchors
// every 1 and 1000 15.1 / 14.8).  So a member joins the lane whose time it prolongs least, if that
// is by a twentieth at most, and else opens one, up to kLanes.
std::vector<int> assign_lanes(const std::vector<Walk>& w) {
  std::vector<int> lane(w.size(), 0), order;
  const auto same = [&](const Walk& a, const Walk& b) {
    return a.t == b.t && a.end == b.end && a.P.global_every == b.P.global_every && a.P.n_global == b.P.n_global &&
           a.P.anchor_every == b.P.anchor_every;
  };
  for (size_t i = 0; i < w.size(); ++i)
    if (w[i].t < w[i].end) order.push_back((int)i);
  bool all = true;
  for (const int i : order) all = all && same(w[i], w[order[0]]);
  if (all) return lane;
  std::vector<double> alone(w.size());
  for (const int i : order) alone[i] = shared_time({w[i]});
  std::stable_sort(order.begin(), order.end(), [&](int a, int c) { return alone[a] > alone[c]; });
  std::vector<Walk> in[kLanes];
  double time[kLanes];
  int n = 0;
  for (const int i : order) {
    int best = -1;
    double best_time = 0.0;
    for (int q = 0; q < n; ++q) {
      std::vector<Walk> with = in[q];
      with.push_back(w[i]);
      const double t = shared_time(std::move(with));
      if (best < 0 || t - time[q] < best_time - time[best]) { best = q; best_time = t; }
    }
    if (best < 0 || (n < kLanes && best_time > 1.05 * time[best])) {
      best = n++;
      best_time = alone[i];
    }
    in[best].push_back(w[i]);
    time[best] = best_time;
    lane[i] = best;
  }
  return lane;
}

}  // namespace

extern "C" {

amh_status amh_batch_create(amh_ctx* const* ctxs, int32_t n, amh_batch** out) {
  if (!out) return sfail(AMH_E_INVAL, "out is NULL");
  *out = nullptr;
  if (!ctxs || n < 1) return sfail(AMH_E_INVAL, "need at least one context");
  for (int i = 0; i < n; ++i) {
    if (!ctxs[i]) return sfail(AMH_E_INVAL, "context %d is NULL", i);
    if (ctxs[i]->stream != ctxs[0]->stream)
      return sfail(AMH_E_INVAL, "context %d is on another stream than context 0", i);
    for (int j = 0; j < i; ++j)
      if (ctxs[j] == ctxs[i]) return sfail(AMH_E_INVAL, "context %d appears twice", i);
  }
  amh_batch* b = new amh_batch;
  b->m.assign(ctxs, ctxs + n);
  b->stream = ctxs[0]->stream;
  b->lane[0].stream = b->stream;
  amh_status st = ready_lane(b, 0, false);
  if (st == AMH_OK) st = build_launches(b, 0);
  if (st != AMH_OK) { free_batch(b); return st; }
  *out = b;
  return AMH_OK;
}

amh_status amh_batch_sweep_each(amh_batch* b, const int64_t* n_sweeps) {
  if (!b) return sfail(AMH_E_INVAL, "batch is NULL");
  if (!n_sweeps) return sfail(AMH_E_INVAL, "n_sweeps is NULL");
  int64_t most = 0;
  for (size_t i = 0; i < b->m.size(); ++i) {
    const amh_ctx* x = b->m[i];
    if (n_sweeps[i] < 0) return sfail(AMH_E_INVAL, "member %zu: n_sweeps < 0", i);
    if (x->t + n_sweeps[i] > x->cfg.total_sweeps)
      return sfail(AMH_E_INVAL, "member %zu: sweep %lld + %lld passes total_sweeps=%lld", i,
                   (long long)x->t, (long long)n_sweeps[i], (long long)x->cfg.total_sweeps);
    most = std::max(most, n_sweeps[i]);
  }
  if (most == 0) return AMH_OK;
  const size_t nm = b->m.size();
  std::vector<Walk> walk(nm);
  for (size_t i = 0; i < nm; ++i) {
    const int64_t t = b->m[i]->t;
    walk[i] = Walk{sweep_params(b->m[i], n_sweeps[i]), t, t + n_sweeps[i], t};
  }
  const std::vector<int> lane_of = assign_lanes(walk);
  const int n_lanes = 1 + *std::max_element(lane_of.begin(), lane_of.end());
  // Steps of one kind in turn: every member of a lane whose next run of sweeps is of that kind
  // (localized or global, up to an anchor or its last sweep) takes part, the others pass
  // through (n_sweeps = 0); an anchor step follows for the members that reached one.
  // Members at the same point of their cycles share every step.  Descriptors go up
  // kMaxRuns steps at a time (stream order keeps an upload behind the launches that read
  // the last).
  struct Progress {
    std::vector<int> n_wg;      // workgroups of each launch (lanes beyond the first)
    std::vector<Step> steps;    // staged, not yet launched
    bool glob = false, left = true;
  };
  std::vector<Progress> progress(n_lanes);
  auto upload_and_launch = [&](int q) -> amh_status {
    Lane& l = b->lane[q];
    Progress& p = progress[q];
    if (p.steps.empty()) return AMH_OK;
    const int slot = l.ring;
    HIP_OK(hipMemcpyAsync(l.d_desc, l.h_ring + (size_t)slot * kMaxRuns * nm, sizeof(amh::SweepParams) * p.steps.size() * nm,
                          hipMemcpyHostToDevice, l.stream));
    HIP_OK(hipEventRecord(l.ev[slot], l.stream));
    l.ev_used[slot] = true;
    l.ring = (slot + 1) % kRing;
    for (size_t r = 0; r < p.steps.size(); ++r) {
      const amh_status st = launch_step(b, l, n_lanes > 1 ? &p.n_wg : nullptr, p.steps[r], l.d_desc + r * nm);
      if (st != AMH_OK) return st;
    }
    p.steps.clear();
    return AMH_OK;
  };
  // one more step of lane q; fill(x, P) completes a member's descriptor and says whether it takes part
  auto add_step = [&](int q, Step kind, auto fill) -> amh_status {
    Lane& l = b->lane[q];
    Progress& p = progress[q];
    if (p.steps.empty() && l.ev_used[l.ring]) HIP_OK(hipEventSynchronize(l.ev[l.ring]));
    amh::SweepParams* d = l.h_ring + ((size_t)l.ring * kMaxRuns + p.steps.size()) * nm;
    bool any = false;
    for (size_t i = 0; i < nm; ++i) {
      d[i] = walk[i].P;
      d[i].n_sweeps = 0;
      if (lane_of[i] == q) any = fill(walk[i], d[i]) || any;
    }
    if (!any) return AMH_OK;
    p.steps.push_back(kind);
    return p.steps.size() == (size_t)kMaxRuns ? upload_and_launch(q) : AMH_OK;
  };
  auto advance = [&](int q) -> amh_status {
    Progress& p = progress[q];
    amh_status st = add_step(q, p.glob ? Step::global : Step::local, [&](Walk& x, amh::SweepParams& P) {
      P.t0 = x.t;
      P.n_sweeps = x.run(p.glob);
      return P.n_sweeps > 0;
    });
    if (st == AMH_OK)
      st = add_step(q, Step::anchor, [&](Walk& x, amh::SweepParams& P) {
        if (!x.anchor()) return false;
        P.t0 = x.t;
        P.n_sweeps = 1;
        return true;
      });
    if (st != AMH_OK) return st;
    p.glob = !p.glob;
    p.left = false;
    for (size_t i = 0; i < nm; ++i) p.left = p.left || (lane_of[i] == q && walk[i].t < walk[i].end);
    return p.left ? AMH_OK : upload_and_launch(q);
  };
  // a lane's workgroups: those of its members
  const auto open_lane = [&](int q) -> amh_status {
    Lane& l = b->lane[q];
    if (l.ev_used[l.ring]) HIP_OK(hipEventSynchronize(l.ev[l.ring]));   // (the ring's slots hold them too)
    int2* const h = l.h_map + (size_t)l.ring * workgroups(b);
    int n = 0;
    for (const auto& launch : b->launches) {
      const int first = n;
      for (const int2& wg : launch.map)
        if (lane_of[wg.x] == q) h[n++] = wg;
      progress[q].n_wg.push_back(n - first);
    }
    HIP_OK(hipMemcpyAsync(l.d_map, h, sizeof(int2) * n, hipMemcpyHostToDevice, l.stream));
    return AMH_OK;
  };
  amh_status st = AMH_OK;
  int forked = 0;
  if (n_lanes > 1) {   // the lanes' work starts behind what the batch's stream holds
    for (int q = 0; q < n_lanes && st == AMH_OK; ++q) st = ready_lane(b, q, true);
    if (st == AMH_OK) HIP_OK(hipEventRecord(b->fork, b->stream));
    for (int q = 0; q < n_lanes && st == AMH_OK; ++q) {
      if (q > 0) HIP_OK(hipStreamWaitEvent(b->lane[q].stream, b->fork, 0));
      forked = q;
      st = open_lane(q);
    }
  }
  for (bool left = true; left && st == AMH_OK;) {
    left = false;
    for (int q = 0; q < n_lanes && st == AMH_OK; ++q) {
      if (progress[q].left) st = advance(q);
      left = left || progress[q].left;
    }
  }
  // and what follows on it waits for them, whatever became of them
  for (int q = 1; q <= forked; ++q) {
    const hipError_t e = hipEventRecord(b->lane[q].done, b->lane[q].stream);
    if (e != hipSuccess || hipStreamWaitEvent(b->stream, b->lane[q].done, 0) != hipSuccess) {
      (void)hipStreamSynchronize(b->lane[q].stream);
      if (st == AMH_OK) st = sfail(AMH_E_DEVICE, "joining a batch's streams: %s", hipGetErrorString(e));
    }
  }
  if (st != AMH_OK) return st;
  for (size_t i = 0; i < nm; ++i) b->m[i]->t += n_sweeps[i];
  return AMH_OK;
}

amh_status amh_batch_sweep(amh_batch* b, int64_t n_sweeps) {
  if (!b) return sfail(AMH_E_INVAL, "batch is NULL");
  if (n_sweeps < 0) return sfail(AMH_E_INVAL, "n_sweeps < 0");
  std::vector<int64_t> n(b->m.size(), n_sweeps);
  return amh_batch_sweep_each(b, n.data());
}

amh_status amh_batch_tune(amh_batch* b, int64_t sweeps_per_trial, float* ms_out, int32_t* plan_out) {
  if (!b) return sfail(AMH_E_INVAL, "batch is NULL");
  if (sweeps_per_trial < 1) return sfail(AMH_E_INVAL, "sweeps_per_trial < 1");
  for (size_t i = 0; i < b->m.size(); ++i) {
    const amh_ctx* x = b->m[i];
    if (x->t + kPlans * sweeps_per_trial > x->cfg.total_sweeps)
      return sfail(AMH_E_INVAL, "member %zu has fewer than %lld sweeps left for tuning", i,
                  (long long)(kPlans * sweeps_per_trial));
  }
  hipEvent_t e0, e1;
  HIP_OK(hipEventCreate(&e0));
  HIP_OK(hipEventCreate(&e1));
  int best = 0;
  float best_ms = 0.0f;
  amh_status st = AMH_OK;
  for (int p = 0; p < kPlans && st == AMH_OK; ++p) {
    if ((st = build_launches(b, p)) != AMH_OK) break;
    if (hipEventRecord(e0, b->stream) != hipSuccess) { st = sfail(AMH_E_DEVICE, "hipEventRecord"); break; }
    if ((st = amh_batch_sweep(b, sweeps_per_trial)) != AMH_OK) break;
    float ms = 0.0f;
    if (hipEventRecord(e1, b->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
      st = sfail(AMH_E_DEVICE, "timing a tuning trial failed");
      break;
    }
    if (ms_out) ms_out[p] = ms;
    if (p == 0 || ms < best_ms) { best = p; best_ms = ms; }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st != AMH_OK) return st;
  if ((st = build_launches(b, best)) != AMH_OK) return st;
  if (plan_out) *plan_out = best;
  return AMH_OK;
}

amh_status amh_batch_set_plan(amh_batch* b, int32_t plan) {
  if (!b) return sfail(AMH_E_INVAL, "batch is NULL");
  if (plan < 0 || plan >= kPlans) return sfail(AMH_E_INVAL, "plan=%d outside [0, %d)", plan, kPlans);
  return build_launches(b, plan);
}

amh_status amh_batch_info(const amh_batch* b, int32_t* plan, int32_t* n_launches, int32_t* workgroups) {
  if (!b) return sfail(AMH_E_INVAL, "batch is NULL");
  if (plan) *plan = b->plan;
  if (n_launches) *n_launches = (int)b->launches.size();
  if (workgroups) *workgroups = ::workgroups(b);
  return AMH_OK;
}

amh_status amh_batch_destroy(amh_batch* b) {
  if (!b) return AMH_OK;
  (void)hipStreamSynchronize(b->stream);
  free_batch(b);
  return AMH_OK;
}

}  // extern "C"
