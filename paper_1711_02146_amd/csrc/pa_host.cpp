// pa_host.cpp -- the C ABI of libpa (include/pa.h): instance state, workspace
// layout, the FP64 resampling table, the constant-culling bisection, and the
// stream-ordered sequence of kernel launches of one annealing step.
//
// Method: Amey & Machta, arXiv:1711.02146.
//   Sec. II     resampling factor tau (Eq. 1), normaliser Q (Eq. 2),
//               nearest-integer copy counts, family labels.
//   Sec. II.A   free-energy estimator (Eq. 9) and population averages.
//   Sec. III.A  rho_t;  Sec. III.C  culling fraction and step size.
//
// The FP64 work of a step (at most 3N + 1 energy levels) runs here, on the
// host, with the C library's exp and log and without contraction
// (-ffp-contract=off), every line rounded left to right.  That keeps the
// integer copy-count thresholds, which decide bits, reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <atomic>
#include <condition_variable>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include <unistd.h>

#include "../../include/pa.h"
#include "pa_host_state.hpp"
#include "pa_internal.hpp"

using pa::DevPop;
using pa::DevScalars;
using pa::SiteEntry;

using namespace pa_host;

// Scratch of pa_link_overlap_hist_noalloc, one copy in each GPU's memory:
// the kLinkCopies partial link-overlap histograms (u32, nbins apart), then the
// final counts (u64).  In host code `scratch` is only a stand-in for the
// symbol; its device address comes from hipGetSymbolAddress, once per device.
static_assert(pa::kLinkCopies == 32, "PA_NOALLOC_SCRATCH_BYTES counts 32 partial histograms");
constexpr size_t kScratchPartWords = (size_t)pa::kLinkCopies * PA_NOALLOC_MAX_BINS;
static __device__ __align__(256) uint32_t scratch[PA_NOALLOC_SCRATCH_BYTES / 4];

namespace {

constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

uint32_t isqrt32(uint32_t v) {
  uint32_t r = (uint32_t)std::sqrt((double)v);
  while ((uint64_t)r * r > v) --r;
  while ((uint64_t)(r + 1) * (r + 1) <= v) ++r;
  return r;
}

bool make_layout(const pa_params* p, Layout* out) {
  if (!p) return false;
  if (p->L < 4 || p->L > (uint32_t)pa::kMaxL || (p->L & 1u)) return false;
  if (p->R < 1) return false;
  if ((p->flags & ~(uint32_t)(PA_FLAG_CHECK_ENERGY | PA_FLAG_FAULT_HOOK | PA_FLAG_TIME_SWEEPS)) !=
          0 ||
      (p->model != PA_MODEL_PM && p->model != PA_MODEL_GAUSS16 && p->model != PA_MODEL_GAUSS))
    return false;
  // PA_LAYOUT_AUTO: the autotuner's layout for this shape (size class of the
  // target population), else the built-in one
  uint32_t layout = p->layout == PA_LAYOUT_AUTO
                        ? pa::layout_for(p->model, p->L, ((uint64_t)p->R + 63) / 64)
                        : p->layout;
  if (layout != PA_LAYOUT_INT8 && layout != PA_LAYOUT_BITPACK64) return false;
  uint64_t cap = p->capacity ? (uint64_t)p->capacity
                             : (uint64_t)p->R + 16ull * isqrt32(p->R) + 256ull;
  if (cap < p->R || cap > (1ull << 31)) return false;
  Layout l{};
  l.L = p->L;
  l.N = p->L * p->L * p->L;
  l.R = p->R;
  l.cap_limit = (uint32_t)cap;
  l.capacity = (uint32_t)((cap + pa::kBlockCounts - 1) / pa::kBlockCounts * pa::kBlockCounts);
  l.layout = layout;
  l.model = p->model;
  // energy levels: U = 0..3N, or every E16 window (|E16| <= 3N * 127); real
  // couplings have none (one placeholder level)
  const bool real = p->model == PA_MODEL_GAUSS;
  l.n_levels = p->model == PA_MODEL_GAUSS16 ? 6 * l.N * (uint32_t)pa::kGaussKMax + 1
               : real                       ? 1
                                            : 3 * l.N + 1;
  l.rowk_stride = (6 * (l.L / 2) + 3) / 4 * 4;
  l.n_blocks = l.capacity / pa::kBlockCounts;
  const size_t tiles = l.capacity / 64;
  l.spins_bytes = layout == PA_LAYOUT_BITPACK64 ? tiles * l.N * 8 : tiles * l.N * 64;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = align_up(o + bytes);
    return at;
  };
  for (int b = 0; b < 2; ++b) l.off_spins[b] = take(l.spins_bytes);
  // energy words: u32 (PA_MODEL_PM, PA_MODEL_GAUSS16) or int64 (PA_MODEL_GAUSS)
  for (int b = 0; b < 2; ++b) l.off_U[b] = take((size_t)l.capacity * (real ? 8 : 4));
  for (int b = 0; b < 2; ++b) l.off_fam[b] = take((size_t)l.capacity * 4);
  l.off_counts = take((size_t)l.capacity * 4);
  l.off_offsets = take((size_t)l.capacity * 4);
  l.off_src = take((size_t)l.capacity * 4);
  l.off_bsum = take((size_t)l.n_blocks * 4);
  l.off_bcull = take((size_t)l.n_blocks * 4);
  // the histogram and the device scalars side by side: one copy brings both
  // to the host after a step (PA_MODEL_PM, whose histogram covers every level)
  l.hist_bytes = ((size_t)l.n_levels * 4 + 63) / 64 * 64;
  l.off_hist = take(l.hist_bytes + sizeof(DevScalars) + sizeof(pa::RealScalars));
  l.off_sc = l.off_hist + l.hist_bytes;
  l.off_rs = l.off_sc + sizeof(DevScalars);
  l.off_table = take((size_t)l.n_levels * sizeof(pa::TableEntry));
  l.off_sites = take((size_t)l.N * sizeof(SiteEntry));
  l.off_psites = take((size_t)l.N * sizeof(pa::PlaneSite));
  l.off_cm = take((size_t)l.N * 2);
  l.off_rowj = take((size_t)2 * l.L * l.L * 8);
  l.off_rowk = take((size_t)2 * l.L * l.L * l.rowk_stride);
  l.off_gthr = take((size_t)(pa::kGaussDEMax + 1) * 8);
  l.off_ovl = take(65 * 8);
  l.off_lovl = take((size_t)(3 * l.N + 1) * 8);
  l.off_lpart = take((size_t)pa::kLinkCopies * (3 * l.N + 1) * 4);
  l.off_pops = take(sizeof(DevPop));
  l.off_meta = take(sizeof(MetaU32));
  // PA_MODEL_GAUSS: the he and threshold tables of every (site, pattern), and
  // one reduction partial per workgroup of the slot kernels
  const size_t rows = (size_t)l.N + pa::kPatternPadRows;
  l.off_rhe = take(real ? rows * pa::kRealPatterns * 8 : 0);
  l.off_rthr = take(real ? rows * pa::kRealPatterns * 8 : 0);
  l.off_rthr32 = take(real ? rows * pa::kRealPatterns * 4 : 0);
  // (one per slot block for the copy counts, kCullLanes per reduction workgroup
  // for the constant-culling search)
  const size_t n_part =
      std::max<size_t>(l.n_blocks, (size_t)pa::kCullLanes * (size_t)pa::kRealSumBlocks);
  l.off_rpart = take(real ? n_part * sizeof(pa::RealPartial) : 0);
  l.off_rsearch = take(real ? sizeof(pa::RealSearch) : 0);
  // PA_MODEL_GAUSS16: the threshold offsets of every (site, pattern)
  l.off_gaddr = take(p->model == PA_MODEL_GAUSS16 ? rows * pa::kRealPatterns * 2 : 0);
  l.total = o;
  *out = l;
  return true;
}

// Lattice tables of the colour-major order for even L: the per-site table,
// lexicographic -> colour-major, and the per-row coupling words (colour c,
// row (y, z): bit 6q + k for the bond from the row's q-th site of colour c,
// x = 2q + ((c + y + z) & 1), to its neighbour k in the order +x,-x,+y,-y,+z,-z).
void build_sites(uint32_t L, const int8_t* J, std::vector<SiteEntry>* sites,
                 std::vector<uint16_t>* cm_of_site, std::vector<uint64_t>* rowj) {
  const uint32_t N = L * L * L, half = N / 2;
  sites->assign(N, SiteEntry{});
  cm_of_site->assign(N, 0);
  auto cm_of = [&](uint32_t x, uint32_t y, uint32_t z) {
    uint32_t s = x + L * (y + L * z);
    return ((x + y + z) & 1u) * half + (s >> 1);
  };
  for (uint32_t z = 0; z < L; ++z)
    for (uint32_t y = 0; y < L; ++y)
      for (uint32_t x = 0; x < L; ++x) {
        const uint32_t s = x + L * (y + L * z);
        const uint32_t cm = cm_of(x, y, z);
        (*cm_of_site)[s] = (uint16_t)cm;
        SiteEntry e{};
        const uint32_t xp = (x + 1) % L, xm = (x + L - 1) % L;
        const uint32_t yp = (y + 1) % L, ym = (y + L - 1) % L;
        const uint32_t zp = (z + 1) % L, zm = (z + L - 1) % L;
        e.nb[0] = (uint16_t)cm_of(xp, y, z);
        e.nb[1] = (uint16_t)cm_of(xm, y, z);
        e.nb[2] = (uint16_t)cm_of(x, yp, z);
        e.nb[3] = (uint16_t)cm_of(x, ym, z);
        e.nb[4] = (uint16_t)cm_of(x, y, zp);
        e.nb[5] = (uint16_t)cm_of(x, y, zm);
        // bond d*N + site joins site and site + e_d
        const int8_t jb[6] = {J[0 * N + s], J[0 * N + (xm + L * (y + L * z))],
                              J[1 * N + s], J[1 * N + (x + L * (ym + L * z))],
                              J[2 * N + s], J[2 * N + (x + L * (y + L * zm))]};
        uint16_t neg = 0;
        for (int k = 0; k < 6; ++k)
          if (jb[k] < 0) neg |= (uint16_t)(1u << k);
        e.jneg = neg;
        e.site = (uint16_t)s;
        (*sites)[cm] = e;
      }
  rowj->assign((size_t)2 * L * L, 0);
  for (uint32_t c = 0; c < 2; ++c)
    for (uint32_t z = 0; z < L; ++z)
      for (uint32_t y = 0; y < L; ++y) {
        const uint32_t p = (c + y + z) & 1u;
        uint64_t word = 0;
        for (uint32_t q = 0; q < L / 2; ++q) {
          const uint32_t x = 2 * q + p;
          const uint32_t cm = c * half + ((x + L * (y + L * z)) >> 1);
          word |= (uint64_t)(*sites)[cm].jneg << (6 * q);
        }
        (*rowj)[(size_t)c * L * L + y + L * z] = word;
      }
}

// PA_MODEL_GAUSS16 row couplings: colour c, row (y, z), byte 6q + k of the row
// (rows `stride` bytes apart) is the coupling of the row's q-th site of colour
// c, x = 2q + ((c + y + z) & 1), to its neighbour k (+x,-x,+y,-y,+z,-z).
void build_rowk(uint32_t L, const int8_t* K, uint32_t stride, std::vector<int8_t>* rowk) {
  const uint32_t N = L * L * L;
  rowk->assign((size_t)2 * L * L * stride, 0);
  for (uint32_t c = 0; c < 2; ++c)
    for (uint32_t z = 0; z < L; ++z)
      for (uint32_t y = 0; y < L; ++y) {
        const uint32_t p = (c + y + z) & 1u;
        int8_t* row = rowk->data() + ((size_t)c * L * L + y + L * z) * stride;
        for (uint32_t q = 0; q < L / 2; ++q) {
          const uint32_t x = 2 * q + p, s = x + L * (y + L * z);
          const uint32_t xm = (x + L - 1) % L, ym = (y + L - 1) % L, zm = (z + L - 1) % L;
          const int8_t kb[6] = {K[0 * N + s], K[0 * N + (xm + L * (y + L * z))],
                                K[1 * N + s], K[1 * N + (x + L * (ym + L * z))],
                                K[2 * N + s], K[2 * N + (x + L * (y + L * zm))]};
          for (int k = 0; k < 6; ++k) row[6 * q + k] = kb[k];
        }
      }
}

// ---------------------------------------------------------------------------
// FP64 resampling table of one step (Sec. II, Eqs. 1-2).  With the lowest
// occupied level j_min as reference energy:
//   w_j = exp(-dbeta * 2 (j - j_min)),  S = sum_{j ascending, h_j > 0} h_j w_j,
//   tau_j = R w_j / S,  fl_j = floor(tau_j),  T_j = ceil(frac(tau_j) 2^53),
//   ln Q = ln S - ln R~ - dbeta E_min,  E_min = 2 j_min - 3N.
// ---------------------------------------------------------------------------
struct Table {
  int jmin = -1, jmax = -1;  // lowest and highest occupied level
  double S = 0.0, lnQ = 0.0;
  double eps = 0.0;          // culling fraction (Sec. III.C) of this step
};

// Levels j have energy unit * (E_lo + j): unit 2, E_lo = -3N/2 for +-J (E = 2U - 3N),
// unit 1/16, E_lo = lowest E16 of the population for quantised Gaussian couplings.
// Entries are written for the occupied levels only: the copy counts read the
// table at each replica's own level, which is occupied.  The culling fraction
// eps R = sum over occupied levels with tau_j < 1 of h_j (1 - tau_j) (Sec.
// III.C) is summed in the same pass, as pa_choose_beta evaluates it.
Table resample_table(const uint32_t* h, uint32_t n_levels, double unit, int64_t E_lo, uint32_t R,
                     uint32_t R_tilde, double dbeta, pa::TableEntry* tab) {
  Table t;
  for (uint32_t j = 0; j < n_levels; ++j)
    if (h[j] > 0) {
      if (t.jmin < 0) t.jmin = (int)j;
      t.jmax = (int)j;
    }
  if (t.jmin < 0) return t;
  const int jmin = t.jmin;
  // w_j once per occupied level (both loops use the same value)
  static thread_local std::vector<double> w;
  w.resize(n_levels);
  double S = 0.0;
  for (uint32_t j = (uint32_t)jmin; j <= (uint32_t)t.jmax; ++j) {
    if (h[j] == 0) continue;
    w[j] = std::exp(-dbeta * (unit * (double)((int)j - jmin)));
    S = S + (double)h[j] * w[j];
  }
  double acc = 0.0;
  for (uint32_t j = (uint32_t)jmin; j <= (uint32_t)t.jmax; ++j) {
    if (h[j] == 0) continue;
    const double tau = ((double)R * w[j]) / S;
    const uint64_t f = (uint64_t)std::floor(tau);
    const double fr = tau - (double)f;
    tab[j].fl = (uint32_t)f;
    tab[j].T = (uint64_t)std::ceil(std::ldexp(fr, 53));
    if (tau < 1.0) acc = acc + (double)h[j] * (1.0 - tau);
  }
  t.S = S;
  t.lnQ = std::log(S) - std::log((double)R_tilde) - dbeta * (unit * (double)(E_lo + jmin));
  t.eps = acc / (double)R;
  return t;
}

}  // namespace

namespace {

pa::BatchDev one_set(const pa_instance* in, const pa::PopStep& ps) {
  pa::BatchDev B{};
  B.pops = in->d_pops;
  B.n_pops = 1;
  B.single = ps;
  return B;
}

pa::Group group_of(const pa_instance* in, const uint32_t* d_start, uint32_t blocks) {
  pa::Group g{};
  g.pop = in->d_meta->pop0;
  g.start = d_start;
  g.n = 1;
  g.blocks = blocks;
  return g;
}

pa::PopStep plain_step(uint32_t cur) {
  pa::PopStep ps{};
  ps.thr[0] = ps.thr[1] = ps.thr[2] = 1ull << 32;
  ps.cur = cur;
  return ps;
}

// The workgroups of a sweep launch of one instance in the form `split` (the
// start table is made for one tile per workgroup; with one member it only says
// that every block is the member's).
pa::Group sweep_group(const pa_instance* in, uint32_t split) {
  return group_of(in, in->d_meta->tiles,
                  pa::sweep_blocks(in->dev.model, in->dev.L, split, in->dev.capacity));
}

// Sweep launch of one instance (its size after any pending copy sets the
// waves per tile).
hipError_t launch_sweep_of(pa_instance* in, const pa::PopStep& ps) {
  const uint32_t split = pa::sweep_split_for(in->dev.model, in->dev.layout, in->dev.L,
                                             ((uint64_t)in->R_tilde + 63) / 64);
  const bool timed = in->sweep_ev[0] != nullptr;
  hipError_t e = timed ? hipEventRecord(in->sweep_ev[0], in->stream) : hipSuccess;
  if (e != hipSuccess) return e;
  e = pa::launch_sweep(one_set(in, ps), sweep_group(in, split), in->dev.layout, in->dev.L, split,
                       in->dev.model, in->stream);
  if (e != hipSuccess || !timed) return e;
  in->sweep_timed = true;
  return hipEventRecord(in->sweep_ev[1], in->stream);
}

// PA_FLAG_TIME_SWEEPS: the duration of the last timed sweep launch, once the
// stream has passed it (call after a synchronisation).
hipError_t read_sweep_time(pa_instance* in) {
  if (!in->sweep_timed) return hipSuccess;
  float ms = 0.0f;
  const hipError_t e = hipEventElapsedTime(&ms, in->sweep_ev[0], in->sweep_ev[1]);
  if (e != hipSuccess) return e;
  in->last_sweep_ms = ms;
  in->sweep_timed = false;
  return hipSuccess;
}

// Energy levels of the histogram in in->h_hist: count, width and offset
// (level j has energy unit * (E_lo + j)).
struct Levels {
  uint32_t n;
  double unit;
  int64_t E_lo;
};

Levels levels_of(const pa_instance* in) {
  if (in->dev.model == pa::kModelGauss16) return {in->n_win, 1.0 / 16.0, (int64_t)in->E_lo};
  return {in->dev.n_levels, 2.0, -(int64_t)(3 * in->dev.N / 2)};
}

// Device address of `scratch` per device, resolved at the first instance
// created on that device (with the device current), kept for the process.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};

void resolve_scratch(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev]) return;
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess && p)
    g_scratch_ptr[dev] = static_cast<uint32_t*>(p);
}

// The kernels' code onto the device of the stream, at the first instance created
// there: once loaded it stays for the process.  A failure shows at the launch that
// needs the code.
std::atomic<uint64_t> g_code_loaded{0};  // bit d: device d

void load_code_beside(hipStream_t stream) {
  int dev = -1;
  if (hipStreamGetDevice(stream, &dev) == hipSuccess && dev >= 0 && dev < kMaxDevices &&
      ((g_code_loaded.load(std::memory_order_relaxed) >> dev) & 1u))
    return;
  const pa_host::DeviceOf current(stream);
  if (!current.ok() || pa::load_code() != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  if (dev >= 0 && dev < kMaxDevices)
    g_code_loaded.fetch_or(1ull << dev, std::memory_order_relaxed);
}

uint32_t* scratch_of(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[dev];
}

int dev_fail(pa_instance* in) {
  in->failed = true;
  return PA_EDEVICE;
}

#define PA_HIP(in, call)                      \
  do {                                        \
    if ((call) != hipSuccess) return dev_fail(in); \
  } while (0)

// Apply a pending order-preserving copy without sweeping (buffer swap).
int materialize(pa_instance* in) {
  if (!in->pending_gather) return PA_OK;
  pa::PopStep ps = plain_step(in->cur);
  ps.t0 = (uint32_t)in->sweeps;
  ps.n_sweeps = 0;
  ps.gather = 1;
  PA_HIP(in, launch_sweep_of(in, ps));
  in->cur ^= 1u;
  in->pending_gather = false;
  in->hist_valid = false;
  return PA_OK;
}

// Histogram of the current population into in->h_hist, plus the device
// scalars into in->h_sc.  Synchronises.  For PA_MODEL_GAUSS16 the histogram
// covers the occupied window [E_lo, E_hi] of E16, found on the device first.
int fetch_hist(pa_instance* in, bool with_family) {
  int rc = materialize(in);
  if (rc) return rc;
  const DevPop& P = in->dev;
  const pa::BatchDev B = one_set(in, plain_step(in->cur));
  PA_HIP(in, pa::launch_zero_acc(B, group_of(in, in->d_meta->perpop, 1), in->stream));
  if (P.model == pa::kModelReal) {
    // no levels: the lowest energy, the replicas at it and the energy sum
    PA_HIP(in, pa::launch_real_stats(B, group_of(in, in->d_meta->rsum, in->meta.rsum[1]),
                                     in->stream));
    if (with_family)
      PA_HIP(in, pa::launch_family(B, group_of(in, in->d_meta->slots, in->meta.slots[1]), in->stream));
    PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars) + sizeof(pa::RealScalars),
                              hipMemcpyDeviceToHost, in->stream));
    PA_HIP(in, hipStreamSynchronize(in->stream));
    PA_HIP(in, read_sweep_time(in));
    if (in->h_sc->err == 2) return dev_fail(in);
    in->R_tilde = in->h_sc->R_tilde;
    in->hist_valid = true;
    return PA_OK;
  }
  uint32_t n = P.n_levels;
  if (P.model == pa::kModelGauss16) {
    PA_HIP(in, pa::launch_minmax(B, group_of(in, in->d_meta->hist, in->meta.hist[1]), in->stream));
    PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars), hipMemcpyDeviceToHost, in->stream));
    PA_HIP(in, hipStreamSynchronize(in->stream));
    const int64_t w = (int64_t)in->h_sc->E_hi - (int64_t)in->h_sc->E_lo + 1;
    if (w < 1 || w > (int64_t)P.n_levels) return dev_fail(in);  // the population is empty or corrupt
    n = (uint32_t)w;
    in->E_lo = in->h_sc->E_lo;
    in->n_win = n;
    PA_HIP(in, pa::launch_fill_u32(P.hist, 0u, n, in->stream));
    PA_HIP(in, pa::launch_hist_window(B, group_of(in, in->d_meta->hist, in->meta.hist[1]), n,
                                      in->stream));
  } else {
    PA_HIP(in, pa::launch_hist(B, group_of(in, in->d_meta->hist, in->meta.hist[1]), P.n_levels,
                               in->stream));
  }
  if (with_family)
    PA_HIP(in, pa::launch_family(B, group_of(in, in->d_meta->slots, in->meta.slots[1]), in->stream));
  if (P.model == pa::kModelGauss16) {
    PA_HIP(in, hipMemcpyAsync(in->h_hist, P.hist, (size_t)n * 4, hipMemcpyDeviceToHost,
                              in->stream));
    PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars), hipMemcpyDeviceToHost,
                              in->stream));
  } else {  // the scalars follow the histogram in the workspace and in the staging
    PA_HIP(in, hipMemcpyAsync(in->h_hist, P.hist, in->lay.hist_bytes + sizeof(DevScalars),
                              hipMemcpyDeviceToHost, in->stream));
  }
  PA_HIP(in, hipStreamSynchronize(in->stream));
  PA_HIP(in, read_sweep_time(in));
  if (in->h_sc->err == 2) return dev_fail(in);
  in->R_tilde = in->h_sc->R_tilde;
  in->hist_valid = true;
  return PA_OK;
}

// Metropolis thresholds of a sweep at beta into the step parameters; for
// PA_MODEL_GAUSS16 the dE16 table goes to the instance's device buffer,
// stream-ordered, through a pinned buffer that is refilled only after the
// previous copy out of it has completed.
hipError_t set_thresholds(pa_instance* in, double beta, pa::PopStep* ps) {
  if (in->dev.model == pa::kModelReal)  // the (site, pattern) table, on the device
    return pa::launch_real_thresholds(in->dev, beta, in->stream);
  if (in->dev.model != pa::kModelGauss16) {
    thresholds(beta, ps->thr);
    return hipSuccess;
  }
  hipError_t e = hipEventSynchronize(in->gthr_copied);
  if (e != hipSuccess) return e;
  unsigned long long* tab = in->h_gthr;
  for (int d = 0; d <= pa::kGaussDEMax; ++d)
    tab[d] = (unsigned long long)std::floor(std::ldexp(std::exp(-beta * ((double)d / 16.0)), 32));
  // the largest and the smallest threshold of a positive move (dE16 is even):
  // a draw is needed unless every entry is 0 or every entry is 2^32
  ps->thr[0] = tab[2];
  ps->thr[1] = tab[pa::kGaussDEMax];
  ps->thr[2] = 0;
  e = hipMemcpyAsync(const_cast<unsigned long long*>(in->dev.gthr), tab,
                     (size_t)(pa::kGaussDEMax + 1) * 8, hipMemcpyHostToDevice, in->stream);
  if (e != hipSuccess) return e;
  return hipEventRecord(in->gthr_copied, in->stream);
}

bool usable(pa_instance* in) { return in && !in->failed && !in->in_batch; }

// Entry of every call on an instance: PA_ESTATE for an unusable one, then one
// call counted for fault injection.
int enter(pa_instance* in) {
  if (!usable(in)) return PA_ESTATE;
  return pa_host::count_call(in);
}

// PA_FLAG_CHECK_ENERGY: every replica's stored energy word of the current
// buffer against the energy recomputed from its spins.  Synchronises.
int check_energy(pa_instance* in) {
  if (!(in->flags & PA_FLAG_CHECK_ENERGY)) return PA_OK;
  const DevPop& P = in->dev;
  PA_HIP(in, pa::launch_fill_u32(&P.sc->check_bad, 0u, 1, in->stream));
  PA_HIP(in, pa::launch_energy(one_set(in, plain_step(in->cur)),
                               group_of(in, in->d_meta->etiles, in->meta.etiles[1]), P.layout, P.L,
                               P.model, true, in->stream));
  PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars), hipMemcpyDeviceToHost, in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  if (in->h_sc->check_bad != 0) {
    in->failed = true;
    return PA_ECHECK;
  }
  return PA_OK;
}

// Philox4x32-10 on the host (Salmon et al., SC'11): counter (c0, c1, c2, c3),
// key (k0, k1); each round multiplies c0 and c2 by the round constants,
// swaps in the high halves XORed with the other counter words and the key,
// and bumps the key by the Weyl constants.
void philox_host(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                 uint32_t out[4]) {
  for (int r = 0; r < 10; ++r) {
    const uint64_t pa = (uint64_t)0xD2511F53u * c0;
    const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(pb >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(pa >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)pb;
    c3 = (uint32_t)pa;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// The culling fraction of Sec. III.C at a candidate step dbeta over the
// occupied levels (exp argument, count) in level order: w_j, S and tau_j
// formed exactly as resample_table() does, eps R = the sum over levels with
// tau_j < 1 of h_j (1 - tau_j).  w is the caller's buffer of n entries.
struct EpsLevels {
  const double* arg;
  const double* cnt;
  size_t n;
  uint32_t R;
};

double culled_fraction(const EpsLevels& lv, double dbeta, double* w) {
  if (lv.n == 0) return 0.0;
  double S = 0.0;
  for (size_t i = 0; i < lv.n; ++i) {
    w[i] = std::exp(-dbeta * lv.arg[i]);
    S = S + lv.cnt[i] * w[i];
  }
  double acc = 0.0;
  for (size_t i = 0; i < lv.n; ++i) {
    const double tau = ((double)lv.R * w[i]) / S;
    if (tau < 1.0) acc = acc + lv.cnt[i] * (1.0 - tau);
  }
  return acc / (double)lv.R;
}

// culled_fraction at a step of 0, bit for bit: every weight is 1.
double culled_fraction_0(const EpsLevels& lv) {
  double S = 0.0;
  for (size_t i = 0; i < lv.n; ++i) S = S + lv.cnt[i];
  const double tau = (double)lv.R / S;
  double acc = 0.0;
  if (tau < 1.0)
    for (size_t i = 0; i < lv.n; ++i) acc = acc + lv.cnt[i] * (1.0 - tau);
  return acc / (double)lv.R;
}

// Host threads that evaluate culling fractions beside the calling thread, for
// the rounds of the search below: kEvalHelpers workers, started on first use
// and kept for the life of the process (never destroyed, so that process exit
// does not wait on them).  A round hands out one candidate per worker, the
// caller evaluates its own, and waits until every worker has finished.
// Workers spin for a short while after a round (the rounds of one search come
// microseconds apart), then sleep until the next.  One search uses the pool
// at a time; a search that finds it busy, or runs in a process forked after
// the workers started, evaluates its candidates itself.
constexpr int kEvalHelpers = pa::kCullLanes - 1;
constexpr long kEvalSpin = 1l << 13;  // pause loops before a worker sleeps (tens of microseconds)

class EvalPool {
 public:
  // nullptr (the caller evaluates by itself) when the workers could not all be
  // started, or in a process forked after they were
  static EvalPool* get() {
    static EvalPool* pool = make();
    return pool && pool->started_ == kEvalHelpers && pool->pid_ == getpid() ? pool : nullptr;
  }
  std::mutex& busy() { return busy_; }
  // out[k] = culled_fraction(lv, x[k]) for k < n (n <= kCullLanes); the
  // caller takes x[0] itself.  Call with busy() held.
  void run(const EpsLevels& lv, const double* x, double* out, int n) {
    lv_ = &lv;
    x_ = x;
    out_ = out;
    n_ = n;
    done_.store(0, std::memory_order_relaxed);
    {
      std::lock_guard<std::mutex> lk(m_);
      gen_.fetch_add(1, std::memory_order_release);
    }
    cv_.notify_all();
    own_.resize(lv.n);
    out[0] = culled_fraction(lv, x[0], own_.data());
    while (done_.load(std::memory_order_acquire) != kEvalHelpers) __builtin_ia32_pause();
  }

 private:
  static EvalPool* make() noexcept {
    try {
      return new EvalPool();
    } catch (...) {
      return nullptr;
    }
  }
  EvalPool() : pid_(getpid()) {
    for (int k = 0; k < kEvalHelpers; ++k) {
      try {
        std::thread([this, k] { work(k + 1); }).detach();
      } catch (...) {
        break;  // a pool without all its workers is never used
      }
      ++started_;
    }
  }
  void work(int lane) {
    std::vector<double> w;
    uint64_t seen = 0;
    for (;;) {
      uint64_t g = gen_.load(std::memory_order_acquire);
      for (long spin = 0; g == seen; g = gen_.load(std::memory_order_acquire)) {
        __builtin_ia32_pause();
        if (++spin > kEvalSpin) {
          std::unique_lock<std::mutex> lk(m_);
          cv_.wait(lk, [&] { return gen_.load(std::memory_order_acquire) != seen; });
          spin = 0;
        }
      }
      seen = g;
      if (lane < n_) {
        w.resize(lv_->n);
        out_[lane] = culled_fraction(*lv_, x_[lane], w.data());
      }
      done_.fetch_add(1, std::memory_order_acq_rel);
    }
  }
  const pid_t pid_;
  int started_ = 0;
  std::mutex busy_, m_;
  std::condition_variable cv_;
  std::atomic<uint64_t> gen_{0};
  std::atomic<int> done_{0};
  const EpsLevels* lv_ = nullptr;
  const double* x_ = nullptr;
  double* out_ = nullptr;
  int n_ = 0;
  std::vector<double> own_;
};

// Occupied levels from which the search uses the worker threads (about nine
// rounds of an evaluation each, 7 ns a level, and a hand-out of some 5 us);
// below it the 26 or so evaluations of the serial search cost less.
constexpr size_t kEvalPoolLevels = 512;

// The constant-culling step of Sec. III.C on the histogram in in->h_hist:
// the beta_next in (beta, beta_max] whose culling fraction is eps_target, by
// 64 bisection halvings keeping the lower end (pa_choose_beta).
int choose_from_hist(pa_instance* in, double eps_target, double beta_max, double* beta_next) {
  if (in->dev.model == pa::kModelReal) {
    // the search on the device (weights of every replica): rounds of two
    // launches until it has ended, kCullRounds queued before the first look
    // (eight end most searches; a round that finds it ended costs two
    // launches that leave at once)
    pa::CullArgs a{};
    a.E = reinterpret_cast<const long long*>(in->dev.U[in->cur]);
    a.sc = in->dev.sc;
    a.rs = in->dev.rs;
    a.search = in->dev.rsearch;
    a.rpart = in->dev.rpart;
    a.R = in->dev.R;
    a.capacity = in->dev.capacity;
    constexpr int kCullRounds = 8, kCullMore = 2;
    PA_HIP(in, pa::launch_real_cull_start(a, beta_max - in->beta, eps_target, in->stream));
    // (a round decides at least one halving once the interpolation has ended)
    for (int done = 0; done < pa::kCullInterp + pa::kCullHalvings + kCullRounds;) {
      const int n = done ? kCullMore : kCullRounds;
      for (int r = 0; r < n; ++r)
        PA_HIP(in, pa::launch_real_cull_round(a, in->meta.rsum[1], in->stream));
      done += n;
      PA_HIP(in, hipMemcpyAsync(in->h_rs, in->dev.rs, sizeof(pa::RealScalars),
                                hipMemcpyDeviceToHost, in->stream));
      PA_HIP(in, hipStreamSynchronize(in->stream));
      if (in->h_rs->result != 0) break;
    }
    const int32_t res = in->h_rs->result;
    if (res == -1) return PA_ESCHEDULE;
    if (res == 1) {
      *beta_next = beta_max;
      return PA_OK;
    }
    if (res != 2) return dev_fail(in);
    *beta_next = in->beta + in->h_rs->lo;
    return PA_OK;
  }
  const Levels lv = levels_of(in);
  const uint32_t nl = lv.n, R = in->dev.R;
  const uint32_t* h = in->h_hist;
  // The occupied levels once, as (exp argument, count) pairs in level order;
  // each evaluation of the culling fraction below, eps R = sum over them
  // with tau_j < 1 of h_j (1 - tau_j) (Sec. III.C), forms w_j, S and tau_j
  // exactly as resample_table() does, without scanning empty levels.
  static thread_local std::vector<double> arg, cnt;
  arg.clear();
  cnt.clear();
  int jmin = -1;
  for (uint32_t j = 0; j < nl; ++j) {
    if (h[j] == 0) continue;
    if (jmin < 0) jmin = (int)j;
    arg.push_back(lv.unit * (double)((int)j - jmin));
    cnt.push_back((double)h[j]);
  }
  const EpsLevels lvs{arg.data(), cnt.data(), arg.size(), R};
  static thread_local std::vector<double> w;
  w.resize(lvs.n);
  // The end point of the 64 halvings of [0, beta_max - beta] (pa_search.hpp)
  // in about 26 evaluations, or, with many occupied levels, nine rounds of
  // seven on the worker threads: a step took 66 evaluations, or 23 rounds.
  // The first guess is the crossing of a Gaussian of the levels' mean: a step
  // dbeta culls sigma dbeta / sqrt(2 pi), the mean lies sigma sqrt(2 ln R~)
  // above the lowest of R~ energies.
  EvalPool* pool = lvs.n >= kEvalPoolLevels ? EvalPool::get() : nullptr;
  std::unique_lock<std::mutex> held;
  if (pool) {
    held = std::unique_lock<std::mutex>(pool->busy(), std::try_to_lock);
    if (!held.owns_lock()) pool = nullptr;
  }
  double total = 0.0, mean_d = 0.0;
  for (size_t i = 0; i < lvs.n; ++i) {
    total += lvs.cnt[i];
    mean_d += lvs.cnt[i] * lvs.arg[i];
  }
  if (lvs.n > 0) mean_d /= total;
  pa::CullSearch s;
  pa::cull_eta(s, mean_d * 1.001, (double)lvs.n, total / (double)R);
  pa::cull_start(s, beta_max - in->beta, eps_target, lvs.n > 0 ? culled_fraction_0(lvs) : 0.0,
                 mean_d > 0.0 ? eps_target * 2.5 * std::sqrt(2.0 * std::log(total + 2.0)) / mean_d
                              : beta_max - in->beta,
                 pool ? pa::kCullLanes : pa::kCullSerial);
  while (s.result == 0) {
    if (pool) pool->run(lvs, s.x, s.e, s.n);
    else
      for (int k = 0; k < s.n; ++k) s.e[k] = culled_fraction(lvs, s.x[k], w.data());
    pa::cull_advance(s);
  }
  if (s.result == -1) return PA_ESCHEDULE;
  *beta_next = s.result == 1 ? beta_max : in->beta + s.lo;
  return PA_OK;
}

// The resampling step beta -> beta_next from the histogram in in->h_hist
// (Sec. II, Eqs. 1-2): the FP64 table on the host, its occupied range
// uploaded, then copy counts, scan (with the capacity check) and the copy map
// queued.  Nothing is synchronised.
int queue_resample(pa_instance* in, double beta_next, Table* t, uint32_t step_flags = 0) {
  const DevPop& P = in->dev;
  const double dbeta = beta_next - in->beta;
  if (P.model == pa::kModelReal) {
    // weights on the device: S at dbeta, then the counts (and the culled
    // fraction) from it; ln Q and eps are taken when the scalars come back
    if (in->R_tilde == 0) return PA_ESTATE;
    *t = Table{};
    t->jmin = 0;
    in->r_Emin_pre = in->h_rs->E_min;
    pa::PopStep ps = plain_step(in->cur);
    ps.step = in->step + 1;
    ps.flags = step_flags;
    ps.dbeta = dbeta;
    const pa::BatchDev B = one_set(in, ps);
    const pa::Group g = group_of(in, in->d_meta->slots, in->meta.slots[1]);
    PA_HIP(in, pa::launch_real_sum(B, group_of(in, in->d_meta->rsum, in->meta.rsum[1]),
                                   in->stream));
    PA_HIP(in, pa::launch_real_counts(B, group_of(in, in->d_meta->rsum, in->meta.rsum[1]),
                                      in->stream));
    PA_HIP(in, pa::launch_scan_scatter(B, g, in->stream));
    return PA_OK;
  }
  const Levels lv = levels_of(in);
  *t = resample_table(in->h_hist, lv.n, lv.unit, lv.E_lo, P.R, in->R_tilde, dbeta, in->h_table);
  if (t->jmin < 0) return PA_ESTATE;  // empty population
  // only the occupied range is read by the copy counts: passed with the
  // launch when it fits, else uploaded to the workspace's table first
  const size_t j0 = (size_t)t->jmin, nj = (size_t)(t->jmax - t->jmin + 1);
  pa::PopStep ps = plain_step(in->cur);
  ps.step = in->step + 1;
  ps.flags = step_flags;
  const pa::BatchDev B = one_set(in, ps);
  const pa::Group g = group_of(in, in->d_meta->slots, in->meta.slots[1]);
  if (nj <= pa::kInlineLevels) {
    static thread_local pa::InlineTable it;
    it.j0 = (uint32_t)j0;
    it.n = (uint32_t)nj;
    std::memcpy(it.e, in->h_table + j0, nj * sizeof(pa::TableEntry));
    PA_HIP(in, pa::launch_counts_inline(B, g, it, in->stream));
  } else {
    PA_HIP(in, hipMemcpyAsync(P.table + j0, in->h_table + j0, nj * sizeof(pa::TableEntry),
                              hipMemcpyHostToDevice, in->stream));
    PA_HIP(in, pa::launch_counts(B, g, in->stream));
  }
  // the scan and the copy map; over capacity, the flag stops the sweep
  PA_HIP(in, pa::launch_scan_scatter(B, g, in->stream));
  return PA_OK;
}

// PA_MODEL_GAUSS: ln Q (Eq. 2) and eps of a queued step from the scalars the
// device computed (in->h_rs after a synchronisation): ln Q = ln S - ln R~ -
// dbeta E_min with E_min the lowest energy of the population it weighed.
void finish_real_table(pa_instance* in, Table* t, double dbeta, uint32_t R_old) {
  if (in->dev.model != pa::kModelReal) return;
  t->S = in->h_rs->S;
  t->lnQ = std::log(t->S) - std::log((double)R_old) -
           dbeta * std::ldexp((double)in->r_Emin_pre, -32);
  t->eps = in->h_rs->eps;
}

// The host mirror after a resampling step that fitted (in->h_sc holds the
// scan's results; R_old: the population size before the step).
void commit_resample(pa_instance* in, const Table& t, double beta_next, uint32_t R_old) {
  in->last_R_old = R_old;
  in->R_tilde = in->h_sc->R_next;
  in->last_n_culled = in->h_sc->n_culled;
  in->last_dbeta = beta_next - in->beta;
  in->last_lnQ = t.lnQ;
  in->last_eps = t.eps;
  in->sum_lnQ = in->sum_lnQ + t.lnQ;
  in->beta = beta_next;
  in->step += 1;
  in->pending_gather = true;
  in->hist_valid = false;
}

// Scalars of the current population from in->h_hist and in->h_sc (filled by
// fetch_hist with the family sums).
// A 128-bit two's-complement integer rounded to FP64 (nearest, ties to even).
double i128_to_double(unsigned long long lo, long long hi) {
  const bool neg = hi < 0;
  unsigned __int128 x = ((unsigned __int128)(unsigned long long)hi << 64) | lo;
  if (neg) x = ~x + 1;
  if (x == 0) return 0.0;
  int p = 127;
  while (!((x >> p) & 1)) --p;
  double v;
  if (p <= 52) {
    v = (double)(unsigned long long)x;
  } else {
    const int sh = p - 52;
    unsigned __int128 mant = x >> sh;
    const unsigned __int128 rem = x - (mant << sh), half = (unsigned __int128)1 << (sh - 1);
    int e = sh;
    if (rem > half || (rem == half && (mant & 1))) {
      mant += 1;
      if (mant >> 53) {
        mant >>= 1;
        e += 1;
      }
    }
    v = std::ldexp((double)(unsigned long long)mant, e);
  }
  return neg ? -v : v;
}

void fill_observables(pa_instance* in, pa_obs* out) {
  const DevPop& P = in->dev;
  if (P.model == pa::kModelReal) {
    const pa::RealScalars& rs = *in->h_rs;
    std::memset(out, 0, sizeof(*out));
    out->beta = in->beta;
    out->dbeta = in->last_dbeta;
    out->lnQ = in->last_lnQ;
    out->beta_F = -((double)P.N * std::log(2.0) + in->sum_lnQ);
    out->mean_E = in->R_tilde ? i128_to_double(rs.sumE_lo, rs.sumE_hi) / (double)in->R_tilde *
                                    std::ldexp(1.0, -32)
                              : 0.0;
    out->sum_eta2 = in->h_sc->sum_eta2;
    out->rho_t = (double)out->sum_eta2 / (double)P.R;
    out->eps_expected = in->last_eps;
    out->R_tilde = in->R_tilde;
    out->n_culled = in->last_n_culled;
    out->E_min = 0;
    out->E_lowest = std::ldexp((double)rs.E_min, -32);
    out->n_at_E_min = rs.n_at_min;
    out->step = in->step;
    out->sweeps_done = in->sweeps;
    out->sum_lnQ = in->sum_lnQ;
    out->sweep_ms = in->last_sweep_ms;
    return;
  }
  const uint32_t* h = in->h_hist;
  const bool gauss = P.model == pa::kModelGauss16;
  const Levels lv = levels_of(in);
  // sum of E in integer units: 2U - 3N, or E16 = E_lo + j
  int64_t sumE = 0;
  int jmin = -1;
  for (uint32_t j = 0; j < lv.n; ++j) {
    if (h[j] && jmin < 0) jmin = (int)j;
    const int64_t e = gauss ? lv.E_lo + (int64_t)j : 2 * (int64_t)j - 3 * (int64_t)P.N;
    sumE += (int64_t)h[j] * e;
  }
  std::memset(out, 0, sizeof(*out));
  out->beta = in->beta;
  out->dbeta = in->last_dbeta;
  out->lnQ = in->last_lnQ;
  out->beta_F = -((double)P.N * std::log(2.0) + in->sum_lnQ);
  out->mean_E = in->R_tilde ? (double)sumE / (double)in->R_tilde : 0.0;
  if (gauss) out->mean_E = out->mean_E * (1.0 / 16.0);  // E16 -> E
  out->sum_eta2 = in->h_sc->sum_eta2;
  out->rho_t = (double)out->sum_eta2 / (double)P.R;
  out->eps_expected = in->last_eps;
  out->R_tilde = in->R_tilde;
  out->n_culled = in->last_n_culled;
  out->E_min = jmin < 0 ? 0 : gauss ? (int32_t)(lv.E_lo + jmin) : 2 * jmin - 3 * (int)P.N;
  out->n_at_E_min = jmin >= 0 ? h[jmin] : 0u;
  out->E_lowest = gauss ? (double)out->E_min / 16.0 : (double)out->E_min;
  out->step = in->step;
  out->sweeps_done = in->sweeps;
  out->sum_lnQ = in->sum_lnQ;
  out->sweep_ms = in->last_sweep_ms;
}

// One step of the anneal queued for a +-J population: the resampling step to
// `beta` (the scan clears the histogram and the family sum), the sweeps, the
// new population's histogram, one copy of the histogram and the scalars
// (event ev_step), the family sums and a copy of their total into staging slot
// `slot` (event ev_fam[slot]).
struct QueuedStep {
  double beta;
  Table t;
  uint32_t R_old, n_sweeps, slot;
};

int queue_step_pm(pa_instance* in, double beta, uint32_t n_sweeps, uint32_t slot, QueuedStep* q) {
  const DevPop& P = in->dev;
  q->beta = beta;
  q->R_old = in->R_tilde;
  q->n_sweeps = n_sweeps;
  q->slot = slot;
  int rc = queue_resample(in, beta, &q->t, pa::kStepHist);
  if (rc) return rc;
  pa::PopStep ps = plain_step(in->cur);
  PA_HIP(in, set_thresholds(in, beta, &ps));
  ps.t0 = (uint32_t)in->sweeps;
  ps.n_sweeps = n_sweeps;
  ps.gather = 1;
  // leaves at once when the scan flagged an overflow
  PA_HIP(in, launch_sweep_of(in, ps));
  const pa::BatchDev B = one_set(in, plain_step(in->cur ^ 1u));
  PA_HIP(in, pa::launch_hist(B, group_of(in, in->d_meta->hist, in->meta.hist[1]), P.n_levels,
                             in->stream));
  PA_HIP(in, hipMemcpyAsync(in->h_hist, P.hist, in->lay.hist_bytes + sizeof(DevScalars),
                            hipMemcpyDeviceToHost, in->stream));
  PA_HIP(in, hipEventRecord(in->ev_step, in->stream));
  PA_HIP(in, pa::launch_family(B, group_of(in, in->d_meta->slots, in->meta.slots[1]), in->stream));
  PA_HIP(in, hipMemcpyAsync(in->h_eta2 + slot, &P.sc->sum_eta2, 8, hipMemcpyDeviceToHost,
                            in->stream));
  PA_HIP(in, hipEventRecord(in->ev_fam[slot], in->stream));
  return PA_OK;
}

// Wait for the histogram and scalars of a queued step and take it over into
// the host mirror (obs without the family sum, which finish_family adds).
// PA_ECAPACITY: nothing after the scan ran; the population is as it was.
int finish_step_pm(pa_instance* in, const QueuedStep& q, pa_obs* out) {
  PA_HIP(in, hipEventSynchronize(in->ev_step));
  PA_HIP(in, read_sweep_time(in));
  if (in->h_sc->err == 2) return dev_fail(in);
  if (in->h_sc->err) {
    in->hist_valid = false;  // the scan cleared it for a sweep that did not run
    return PA_ECAPACITY;
  }
  commit_resample(in, q.t, q.beta, q.R_old);
  in->cur ^= 1u;
  in->R_tilde = in->h_sc->R_tilde;
  in->pending_gather = false;
  in->hist_valid = true;
  in->sweeps += q.n_sweeps;
  if (out) fill_observables(in, out);
  return PA_OK;
}

int finish_family(pa_instance* in, const QueuedStep& q, pa_obs* out) {
  PA_HIP(in, hipEventSynchronize(in->ev_fam[q.slot]));
  if (out) {
    out->sum_eta2 = in->h_eta2[q.slot];
    out->rho_t = (double)out->sum_eta2 / (double)in->dev.R;
  }
  return PA_OK;
}

// Up to max_steps steps of the anneal (Sec. II loop): with eps_target >= 0
// the constant-culling step (Sec. III.C) to at most beta_max, stopping there;
// otherwise one step to beta_fixed.  obs (nullable) receives each step's
// scalars.  Every bit equals pa_choose_beta + pa_resample + pa_sweep +
// pa_observables per step.  For +-J populations the work is queued so that
// one synchronisation per step brings back the histogram, and the family sums
// of a step run on the device while the host chooses the next step.
int anneal_steps(pa_instance* in, double eps_target, double beta_max, double beta_fixed,
                 uint32_t n_sweeps, uint32_t max_steps, pa_obs* obs, uint32_t* done) {
  const bool adaptive = eps_target >= 0.0;
  if (n_sweeps == 0 || in->sweeps + (uint64_t)n_sweeps * max_steps > 0xFFFFFFFFull)
    return PA_EINVAL;
  if (adaptive && (!std::isfinite(eps_target) || !std::isfinite(beta_max) ||
                   !(beta_max > in->beta)))
    return PA_EINVAL;
  if (!adaptive && (!std::isfinite(beta_fixed) || !(beta_fixed >= 0.0))) return PA_EINVAL;
  const bool fused = in->dev.model == pa::kModelPm && !(in->flags & PA_FLAG_CHECK_ENERGY);
  if (!fused) {
    // the separate calls, step by step
    for (uint32_t k = 0; k < max_steps; ++k) {
      if (adaptive && !(in->beta < beta_max)) break;
      double b = beta_fixed;
      int rc = check_energy(in);
      if (rc) return rc;
      if (!in->hist_valid || in->pending_gather) {
        rc = fetch_hist(in, false);
        if (rc) return rc;
      }
      if (adaptive) {
        rc = choose_from_hist(in, eps_target, beta_max, &b);
        if (rc) return rc;
      }
      Table t;
      rc = queue_resample(in, b, &t);
      if (rc) return rc;
      pa::PopStep ps = plain_step(in->cur);
      PA_HIP(in, set_thresholds(in, b, &ps));
      ps.t0 = (uint32_t)in->sweeps;
      ps.n_sweeps = n_sweeps;
      ps.gather = 1;
      PA_HIP(in, launch_sweep_of(in, ps));
      const uint32_t old_cur = in->cur, R_old = in->R_tilde;
      if (in->dev.model == pa::kModelGauss16) {
        // the energy window of the new population is found on the device
        // and read first; an unwritten buffer has none, so the overflow
        // check comes first
        PA_HIP(in, hipMemcpyAsync(in->h_sc, in->dev.sc, sizeof(DevScalars),
                                  hipMemcpyDeviceToHost, in->stream));
        PA_HIP(in, hipStreamSynchronize(in->stream));
        if (in->h_sc->err == 2) return dev_fail(in);
        if (in->h_sc->err) {
          in->sweep_timed = false;
          return PA_ECAPACITY;  // nothing after the scan ran: the population is as it was
        }
      }
      in->cur ^= 1u;
      rc = fetch_hist(in, true);  // histogram and family sums: the synchronisation
      if (rc) return rc;
      if (in->h_sc->err) {
        in->cur = old_cur;
        in->R_tilde = R_old;
        in->hist_valid = false;
        return PA_ECAPACITY;
      }
      finish_real_table(in, &t, b - in->beta, R_old);
      commit_resample(in, t, b, R_old);
      in->R_tilde = in->h_sc->R_tilde;
      in->pending_gather = false;
      in->hist_valid = true;
      in->sweeps += n_sweeps;
      rc = check_energy(in);
      if (rc) return rc;
      if (obs) fill_observables(in, obs + k);
      *done = k + 1;
    }
    return PA_OK;
  }
  if (!in->hist_valid || in->pending_gather) {
    const int rc = fetch_hist(in, false);
    if (rc) return rc;
  }
  double b = beta_fixed;
  if (adaptive) {
    const int rc = choose_from_hist(in, eps_target, beta_max, &b);
    if (rc) return rc;
  }
  QueuedStep q[2];
  int rc = queue_step_pm(in, b, n_sweeps, 0, &q[0]);
  if (rc) return rc;
  for (uint32_t k = 0;; ++k) {
    const QueuedStep& cur = q[k & 1];
    pa_obs* o = obs ? obs + k : nullptr;
    rc = finish_step_pm(in, cur, o);
    if (rc) {
      (void)hipStreamSynchronize(in->stream);  // let the queued family sums finish
      return rc;
    }
    *done = k + 1;
    // the next step is chosen and queued while this one's family sums run
    const bool more = k + 1 < max_steps && adaptive && in->beta < beta_max;
    if (more) {
      rc = choose_from_hist(in, eps_target, beta_max, &b);
      if (rc == PA_OK) rc = queue_step_pm(in, b, n_sweeps, (k + 1) & 1, &q[(k + 1) & 1]);
    }
    const int rc_fam = finish_family(in, cur, o);
    if (rc) return rc;
    if (rc_fam) return rc_fam;
    if (!more) return PA_OK;
  }
}

}  // namespace

extern "C" {

size_t pa_workspace_bytes(const pa_params* p) {
  Layout l;
  if (!make_layout(p, &l)) return 0;
  return l.total;
}

int pa_make_couplings_pm(uint64_t coupling_seed, uint32_t L, int8_t* J_out) {
  if (!J_out || L < 2 || L > 64) return PA_EINVAL;
  const uint64_t nb = 3ull * L * L * L;
  const uint32_t k0 = (uint32_t)coupling_seed, k1 = (uint32_t)(coupling_seed >> 32);
  for (uint64_t g = 0; 4 * g < nb; ++g) {
    uint32_t w[4];
    philox_host((uint32_t)g, 0u, 0u, pa::kTagJ, k0, k1, w);
    for (uint32_t i = 0; i < 4 && 4 * g + i < nb; ++i)
      J_out[4 * g + i] = (w[i] >> 31) ? (int8_t)-1 : (int8_t)1;
  }
  return PA_OK;
}

const char* pa_strerror(int status) {
  switch (status) {
    case PA_OK: return "ok";
    case PA_EINVAL: return "invalid argument";
    case PA_ENOMEM: return "workspace too small";
    case PA_ECAPACITY: return "resampled population exceeds capacity";
    case PA_EDEVICE: return "HIP error (instance unusable)";
    case PA_ESTATE: return "call out of order or instance unusable";
    case PA_ESCHEDULE: return "constant-culling step impossible (eps(0) > target)";
    case PA_ECHECK: return "energy check failed (instance unusable)";
    default: return "unknown status";
  }
}

}  // extern "C"

namespace {

std::vector<long long> real_he_table(uint32_t L, const std::vector<long long>& k);

// The body of pa_init_instance and pa_init_instance_real.  rhe: the he table
// of PA_MODEL_GAUSS (N x 64, colour-major), else null; J_host then only
// shapes the lattice tables.
int init_instance(const pa_params* p, const int8_t* J_host, const std::vector<long long>* rhe,
                  void* d_workspace, size_t ws_bytes, void* hip_stream, pa_instance** out) {
  if (!out) return PA_EINVAL;
  *out = nullptr;
  Layout l;
  if (!make_layout(p, &l) || !J_host || !d_workspace) return PA_EINVAL;
  if ((l.model == PA_MODEL_GAUSS) != (rhe != nullptr)) return PA_EINVAL;
  if (ws_bytes < l.total) return PA_ENOMEM;
  if (reinterpret_cast<uintptr_t>(d_workspace) % kAlign) return PA_EINVAL;

  pa_instance* in = new (std::nothrow) pa_instance();
  if (!in) return PA_EINVAL;
  in->lay = l;
  in->flags = p->flags;
  if (hipGetDevice(&in->device) != hipSuccess) {
    delete in;
    return PA_EDEVICE;
  }
  resolve_scratch(in->device);
  in->stream = static_cast<hipStream_t>(hip_stream);
  load_code_beside(in->stream);
  in->ws = static_cast<uint8_t*>(d_workspace);
  build_sites(l.L, J_host, &in->sites, &in->cm_of_site, &in->rowj);
  // PA_MODEL_GAUSS16: per (site, pattern) the LDS byte offset 8 max(dE16, 0)
  // = 16 max(he16, 0) of the move's threshold in the sweep's dE16 table
  std::vector<uint16_t> gaddr;
  if (l.model == PA_MODEL_GAUSS16) {
    build_rowk(l.L, J_host, l.rowk_stride, &in->rowk);
    const std::vector<long long> k16(J_host, J_host + 3 * (size_t)l.N);
    const std::vector<long long> he16 = real_he_table(l.L, k16);
    gaddr.resize(he16.size());
    for (size_t i = 0; i < he16.size(); ++i)
      gaddr[i] = (uint16_t)(16 * (he16[i] > 0 ? he16[i] : 0));  // <= 16 x 6 x 127
  }

  DevPop& P = in->dev;
  P.L = l.L;
  P.N = l.N;
  P.R = l.R;
  P.capacity = l.capacity;
  P.layout = l.layout;
  P.n_levels = l.n_levels;
  P.n_blocks = l.n_blocks;
  P.cap_limit = l.cap_limit;
  P.seed = p->seed;
  uint8_t* w = in->ws;
  for (int b = 0; b < 2; ++b) {
    P.spins[b] = w + l.off_spins[b];
    P.U[b] = reinterpret_cast<uint32_t*>(w + l.off_U[b]);
    P.fam[b] = reinterpret_cast<uint32_t*>(w + l.off_fam[b]);
  }
  P.counts = reinterpret_cast<uint32_t*>(w + l.off_counts);
  P.offsets = reinterpret_cast<uint32_t*>(w + l.off_offsets);
  P.src = reinterpret_cast<uint32_t*>(w + l.off_src);
  P.block_sums = reinterpret_cast<uint32_t*>(w + l.off_bsum);
  P.block_culled = reinterpret_cast<uint32_t*>(w + l.off_bcull);
  P.hist = reinterpret_cast<uint32_t*>(w + l.off_hist);
  P.table = reinterpret_cast<pa::TableEntry*>(w + l.off_table);
  P.sites = reinterpret_cast<const SiteEntry*>(w + l.off_sites);
  P.psites = reinterpret_cast<const pa::PlaneSite*>(w + l.off_psites);
  P.pmsites = reinterpret_cast<const pa::PmSite*>(w + l.off_psites);
  P.cm_of_site = reinterpret_cast<const uint16_t*>(w + l.off_cm);
  P.rowj = reinterpret_cast<const unsigned long long*>(w + l.off_rowj);
  P.ovl_hist = reinterpret_cast<unsigned long long*>(w + l.off_ovl);
  P.lovl_hist = reinterpret_cast<unsigned long long*>(w + l.off_lovl);
  P.lovl_part = reinterpret_cast<uint32_t*>(w + l.off_lpart);
  P.sc = reinterpret_cast<DevScalars*>(w + l.off_sc);
  P.model = l.model;
  P.rowk_stride = l.rowk_stride;
  P.rowk = reinterpret_cast<const int8_t*>(w + l.off_rowk);
  P.gthr = reinterpret_cast<const unsigned long long*>(w + l.off_gthr);
  const bool real = l.model == PA_MODEL_GAUSS;
  P.gaddr = gaddr.empty() ? nullptr : reinterpret_cast<const uint16_t*>(w + l.off_gaddr);
  P.rhe = real ? reinterpret_cast<const long long*>(w + l.off_rhe) : nullptr;
  P.rthr = real ? reinterpret_cast<unsigned long long*>(w + l.off_rthr) : nullptr;
  P.rthr32 = real ? reinterpret_cast<uint32_t*>(w + l.off_rthr32) : nullptr;
  P.rs = reinterpret_cast<pa::RealScalars*>(w + l.off_rs);
  P.rpart = real ? reinterpret_cast<pa::RealPartial*>(w + l.off_rpart) : nullptr;
  P.rsearch = real ? reinterpret_cast<pa::RealSearch*>(w + l.off_rsearch) : nullptr;
  in->d_pops = reinterpret_cast<DevPop*>(w + l.off_pops);
  in->d_meta = reinterpret_cast<MetaU32*>(w + l.off_meta);
  MetaU32& mt = in->meta;
  mt.pop0[0] = 0; mt.pop0[1] = 0;
  mt.perpop[0] = 0; mt.perpop[1] = 1;
  mt.slots[0] = 0; mt.slots[1] = pa::blocks_slots(l.capacity);
  mt.hist[0] = 0; mt.hist[1] = pa::blocks_hist(l.capacity);
  mt.tiles[0] = 0; mt.tiles[1] = pa::blocks_sweep(l.capacity, 1);
  mt.etiles[0] = 0; mt.etiles[1] = l.capacity / 64;
  mt.rsum[0] = 0; mt.rsum[1] = std::min(pa::blocks_slots(l.capacity), pa::kRealSumBlocks);

  auto fail = [&](int rc) {
    pa_free(in);
    return rc;
  };
  // histogram and scalars in one pinned block, laid out as in the workspace
  if (hipHostMalloc(reinterpret_cast<void**>(&in->h_hist),
                    l.hist_bytes + sizeof(DevScalars) + sizeof(pa::RealScalars)) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void**>(&in->h_table),
                    (size_t)l.n_levels * sizeof(pa::TableEntry)) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void**>(&in->h_ovl), 65 * 8) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void**>(&in->h_lovl), (size_t)(3 * l.N + 1) * 8) !=
          hipSuccess)
    return fail(PA_EDEVICE);
  in->h_sc = reinterpret_cast<DevScalars*>(reinterpret_cast<uint8_t*>(in->h_hist) + l.hist_bytes);
  in->h_rs = reinterpret_cast<pa::RealScalars*>(in->h_sc + 1);
  if (hipHostMalloc(reinterpret_cast<void**>(&in->h_eta2), 2 * sizeof(unsigned long long)) !=
          hipSuccess ||
      hipEventCreateWithFlags(&in->ev_step, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&in->ev_fam[0], hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&in->ev_fam[1], hipEventDisableTiming) != hipSuccess)
    return fail(PA_EDEVICE);
  if (l.model == PA_MODEL_GAUSS16 &&
      (hipHostMalloc(reinterpret_cast<void**>(&in->h_gthr), (size_t)(pa::kGaussDEMax + 1) * 8) !=
           hipSuccess ||
       hipEventCreateWithFlags(&in->gthr_copied, hipEventDisableTiming) != hipSuccess ||
       hipEventRecord(in->gthr_copied, in->stream) != hipSuccess))
    return fail(PA_EDEVICE);

  // phase 1 of the colour passes reads each site's neighbours in the LDS tile
  // image: +-J by their offset in it, Gaussian models by LDS address
  std::vector<pa::PlaneSite> psites(l.N);
  if (l.model == PA_MODEL_PM) {
    pa::PmSite* const q = reinterpret_cast<pa::PmSite*>(psites.data());
    for (uint32_t cm = 0; cm < l.N; ++cm)
      for (uint32_t h = 0; h < 2; ++h) {
        pa::PmSite& e = q[8 * (cm >> 2) + 4 * h + (cm & 3u)];
        for (int k = 0; k < 6; ++k) {
          const uint32_t n = in->sites[cm].nb[k];
          e.nb[k] = (uint16_t)(8u * ((n & 3u) * (l.N / 4) + (n >> 2)) + 4u * h);
        }
        e.jneg = in->sites[cm].jneg;
      }
  } else {
    for (uint32_t cm = 0; cm < l.N; ++cm) {
      pa::PlaneSite& q = psites[cm];
      for (int k = 0; k < 6; ++k) q.nb8[k] = pa::kTileLdsBase + 8u * in->sites[cm].nb[k];
      q.jneg = in->sites[cm].jneg;
      q.pad = 0;
    }
  }
  // tables and scalars (synchronous copies from pageable host memory)
  DevScalars sc{};
  sc.R_tilde = l.R;
  const pa::RealScalars rs0{};
  if (hipMemcpyAsync(w + l.off_sites, in->sites.data(), l.N * sizeof(SiteEntry),
                     hipMemcpyHostToDevice, in->stream) != hipSuccess ||
      hipMemcpyAsync(w + l.off_cm, in->cm_of_site.data(), l.N * 2, hipMemcpyHostToDevice,
                     in->stream) != hipSuccess ||
      hipMemcpyAsync(w + l.off_psites, psites.data(), l.N * sizeof(pa::PlaneSite),
                     hipMemcpyHostToDevice, in->stream) != hipSuccess ||
      hipMemcpyAsync(w + l.off_rowj, in->rowj.data(), in->rowj.size() * 8, hipMemcpyHostToDevice,
                     in->stream) != hipSuccess ||
      (!in->rowk.empty() &&
       hipMemcpyAsync(w + l.off_rowk, in->rowk.data(), in->rowk.size(), hipMemcpyHostToDevice,
                      in->stream) != hipSuccess) ||
      hipMemcpyAsync(P.sc, &sc, sizeof(sc), hipMemcpyHostToDevice, in->stream) != hipSuccess ||
      hipMemcpyAsync(P.rs, &rs0, sizeof(rs0), hipMemcpyHostToDevice, in->stream) != hipSuccess ||
      (real && hipMemcpyAsync(w + l.off_rhe, rhe->data(), rhe->size() * 8, hipMemcpyHostToDevice,
                              in->stream) != hipSuccess) ||
      (!gaddr.empty() && hipMemcpyAsync(w + l.off_gaddr, gaddr.data(), gaddr.size() * 2,
                                        hipMemcpyHostToDevice, in->stream) != hipSuccess) ||
      hipMemcpyAsync(in->d_pops, &in->dev, sizeof(DevPop), hipMemcpyHostToDevice, in->stream) !=
          hipSuccess ||
      hipMemcpyAsync(in->d_meta, &in->meta, sizeof(MetaU32), hipMemcpyHostToDevice, in->stream) !=
          hipSuccess ||
      hipStreamSynchronize(in->stream) != hipSuccess)
    return fail(PA_EDEVICE);
  if (pa::launch_init(P, 0, in->stream) != hipSuccess) return fail(PA_EDEVICE);
  // Gaussian couplings: the energy word (E16 or E32) is formed from the spins
  if ((l.model == PA_MODEL_GAUSS16 || real) &&
      pa::launch_energy(one_set(in, plain_step(0)), group_of(in, in->d_meta->etiles, mt.etiles[1]),
                        l.layout, l.L, l.model, false, in->stream) != hipSuccess)
    return fail(PA_EDEVICE);
  if ((p->flags & PA_FLAG_TIME_SWEEPS) &&
      (hipEventCreate(&in->sweep_ev[0]) != hipSuccess ||
       hipEventCreate(&in->sweep_ev[1]) != hipSuccess))
    return fail(PA_EDEVICE);
  in->cur = 0;
  in->R_tilde = l.R;
  *out = in;
  return PA_OK;
}

// he[cm][y] of PA_MODEL_GAUSS from couplings k (units 2^-32): for the site at
// colour-major index cm and its couplings k_0..k_5 to the neighbours
// +x,-x,+y,-y,+z,-z, he = sum_k k_k (1 - 2 y_k) over the bits y_k of y.
std::vector<long long> real_he_table(uint32_t L, const std::vector<long long>& k) {
  const uint32_t N = L * L * L, half = N / 2;
  std::vector<long long> he((size_t)N * pa::kRealPatterns);
  for (uint32_t z = 0; z < L; ++z)
    for (uint32_t y = 0; y < L; ++y)
      for (uint32_t x = 0; x < L; ++x) {
        const uint32_t s = x + L * (y + L * z);
        const uint32_t cm = ((x + y + z) & 1u) * half + (s >> 1);
        const uint32_t xm = (x + L - 1) % L, ym = (y + L - 1) % L, zm = (z + L - 1) % L;
        const long long kb[6] = {k[0 * N + s], k[0 * N + (xm + L * (y + L * z))],
                                 k[1 * N + s], k[1 * N + (x + L * (ym + L * z))],
                                 k[2 * N + s], k[2 * N + (x + L * (y + L * zm))]};
        for (uint32_t pat = 0; pat < pa::kRealPatterns; ++pat) {
          long long v = 0;
          for (int b = 0; b < 6; ++b) v += ((pat >> b) & 1u) ? -kb[b] : kb[b];
          he[(size_t)cm * pa::kRealPatterns + pat] = v;
        }
      }
  return he;
}

}  // namespace

extern "C" {

int pa_init_instance(const pa_params* p, const int8_t* J_host, void* d_workspace, size_t ws_bytes,
                     void* hip_stream, pa_instance** out) {
  if (p && p->model == PA_MODEL_GAUSS) return PA_EINVAL;  // real couplings: pa_init_instance_real
  if (p && J_host && p->L >= 4 && p->L <= (uint32_t)pa::kMaxL) {
    const uint32_t N = p->L * p->L * p->L;
    for (uint32_t b = 0; b < 3 * N; ++b) {
      if (p->model == PA_MODEL_PM && J_host[b] != 1 && J_host[b] != -1) return PA_EINVAL;
      if (p->model == PA_MODEL_GAUSS16 &&
          (J_host[b] < -pa::kGaussKMax || J_host[b] > pa::kGaussKMax))
        return PA_EINVAL;
    }
  }
  return init_instance(p, J_host, nullptr, d_workspace, ws_bytes, hip_stream, out);
}

int pa_init_instance_real(const pa_params* p, const double* J_host, void* d_workspace,
                          size_t ws_bytes, void* hip_stream, pa_instance** out) {
  if (!out) return PA_EINVAL;
  *out = nullptr;
  if (!p || !J_host || p->model != PA_MODEL_GAUSS) return PA_EINVAL;
  if (p->L < 4 || p->L > (uint32_t)pa::kMaxL || (p->L & 1u)) return PA_EINVAL;
  const uint32_t N = p->L * p->L * p->L;
  // each coupling to the nearest multiple of 2^-32 (ties to even: the
  // default rounding of nearbyint), as the integer k = J 2^32
  std::vector<long long> k(3 * (size_t)N);
  for (uint32_t b = 0; b < 3 * N; ++b) {
    const double J = J_host[b];
    if (!std::isfinite(J) || !(std::fabs(J) < 8.0)) return PA_EINVAL;
    k[b] = (long long)std::nearbyint(std::ldexp(J, 32));
  }
  const std::vector<long long> he = real_he_table(p->L, k);
  // the lattice tables need couplings only for the +-J bit words, unused here
  const std::vector<int8_t> ones(3 * (size_t)N, (int8_t)1);
  return init_instance(p, ones.data(), &he, d_workspace, ws_bytes, hip_stream, out);
}

int pa_export_energies(pa_instance* in, double* E_host) {
  if (int rc0 = enter(in)) return rc0;
  if (!E_host) return PA_EINVAL;
  int rc = materialize(in);
  if (rc) return rc;
  const DevPop& P = in->dev;
  PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars), hipMemcpyDeviceToHost, in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  const uint32_t R = in->h_sc->R_tilde;
  in->R_tilde = R;
  if (R == 0) return PA_OK;
  if (P.model == pa::kModelReal) {
    std::vector<long long> e(R);
    PA_HIP(in, hipMemcpy(e.data(), P.U[in->cur], (size_t)R * 8, hipMemcpyDeviceToHost));
    for (uint32_t r = 0; r < R; ++r) E_host[r] = std::ldexp((double)e[r], -32);
  } else {
    std::vector<uint32_t> u(R);
    PA_HIP(in, hipMemcpy(u.data(), P.U[in->cur], (size_t)R * 4, hipMemcpyDeviceToHost));
    for (uint32_t r = 0; r < R; ++r)
      E_host[r] = P.model == pa::kModelGauss16 ? (double)(int32_t)u[r] / 16.0
                                               : 2.0 * (double)u[r] - 3.0 * (double)P.N;
  }
  return PA_OK;
}

int pa_free(pa_instance* in) {
  if (!in) return PA_EINVAL;
  (void)hipStreamSynchronize(in->stream);
  if (in->h_hist) (void)hipHostFree(in->h_hist);
  if (in->h_table) (void)hipHostFree(in->h_table);
  if (in->h_ovl) (void)hipHostFree(in->h_ovl);
  if (in->h_lovl) (void)hipHostFree(in->h_lovl);
  if (in->h_gthr) (void)hipHostFree(in->h_gthr);
  if (in->gthr_copied) (void)hipEventDestroy(in->gthr_copied);
  for (hipEvent_t e : in->sweep_ev)
    if (e) (void)hipEventDestroy(e);
  for (hipEvent_t e : {in->ev_step, in->ev_fam[0], in->ev_fam[1]})
    if (e) (void)hipEventDestroy(e);
  if (in->h_eta2) (void)hipHostFree(in->h_eta2);
  delete in;
  return PA_OK;
}

int pa_debug_inject(pa_instance* in, uint32_t what, uint32_t arg) {
  if (!in || !(in->flags & PA_FLAG_FAULT_HOOK)) return PA_EINVAL;
  if (!usable(in)) return PA_ESTATE;
  if (what == PA_INJECT_FAIL_AFTER) {
    in->fail_countdown = (int64_t)arg;
    return PA_OK;
  }
  if (what != PA_INJECT_ENERGY) return PA_EINVAL;
  int rc = materialize(in);
  if (rc) return rc;
  PA_HIP(in, hipMemcpyAsync(in->h_sc, in->dev.sc, sizeof(DevScalars), hipMemcpyDeviceToHost,
                            in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  if (arg >= in->h_sc->R_tilde) return PA_EINVAL;
  uint32_t* word = in->dev.U[in->cur] + arg;
  uint32_t v = 0;
  PA_HIP(in, hipMemcpy(&v, word, 4, hipMemcpyDeviceToHost));
  v += 1u;
  PA_HIP(in, hipMemcpy(word, &v, 4, hipMemcpyHostToDevice));
  in->hist_valid = false;
  return PA_OK;
}

int pa_sweep(pa_instance* in, double beta, uint32_t n_sweeps) {
  if (int rc0 = enter(in)) return rc0;
  if (!(beta >= 0.0) || !std::isfinite(beta)) return PA_EINVAL;
  if (n_sweeps == 0) return PA_OK;
  if (in->sweeps + n_sweeps > 0xFFFFFFFFull) return PA_EINVAL;  // sweep counter is 32-bit
  pa::PopStep ps = plain_step(in->cur);
  PA_HIP(in, set_thresholds(in, beta, &ps));
  ps.t0 = (uint32_t)in->sweeps;
  ps.n_sweeps = n_sweeps;
  ps.gather = in->pending_gather ? 1u : 0u;
  PA_HIP(in, launch_sweep_of(in, ps));
  in->cur ^= 1u;
  in->pending_gather = false;
  in->hist_valid = false;
  in->sweeps += n_sweeps;
  return check_energy(in);
}

int pa_resample(pa_instance* in, double beta_next, pa_obs* step_out) {
  if (int rc0 = enter(in)) return rc0;
  if (!std::isfinite(beta_next)) return PA_EINVAL;
  int rc = check_energy(in);
  if (rc) return rc;
  if (!in->hist_valid || in->pending_gather) {
    rc = fetch_hist(in, false);
    if (rc) return rc;
  }
  Table t;
  rc = queue_resample(in, beta_next, &t);
  if (rc) return rc;
  PA_HIP(in, hipMemcpyAsync(in->h_sc, in->dev.sc, sizeof(DevScalars) + sizeof(pa::RealScalars),
                            hipMemcpyDeviceToHost, in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  if (in->h_sc->err == 2) return dev_fail(in);
  if (in->h_sc->err) return PA_ECAPACITY;  // population untouched
  finish_real_table(in, &t, beta_next - in->beta, in->R_tilde);
  commit_resample(in, t, beta_next, in->R_tilde);
  if (step_out) {
    std::memset(step_out, 0, sizeof(*step_out));
    step_out->beta = in->beta;
    step_out->dbeta = in->last_dbeta;
    step_out->lnQ = t.lnQ;
    step_out->beta_F = -((double)in->dev.N * std::log(2.0) + in->sum_lnQ);
    step_out->eps_expected = in->last_eps;
    step_out->R_tilde = in->R_tilde;
    step_out->n_culled = in->last_n_culled;
    step_out->step = in->step;
    step_out->sweeps_done = in->sweeps;
    step_out->sum_lnQ = in->sum_lnQ;
  }
  return PA_OK;
}

int pa_anneal_step(pa_instance* in, double eps_target, double beta_max, uint32_t n_sweeps,
                   double* beta_next, pa_obs* out) {
  if (int rc0 = enter(in)) return rc0;
  if (!beta_next) return PA_EINVAL;
  uint32_t done = 0;
  const int rc = anneal_steps(in, eps_target, beta_max, *beta_next, n_sweeps, 1, out, &done);
  if (rc == PA_OK) *beta_next = in->beta;
  return rc;
}

int pa_anneal_run(pa_instance* in, double eps_target, double beta_max, uint32_t n_sweeps,
                  uint32_t max_steps, pa_obs* obs, uint32_t* steps_done) {
  if (int rc0 = enter(in)) return rc0;
  if (!steps_done || !(eps_target >= 0.0)) return PA_EINVAL;
  *steps_done = 0;
  if (max_steps == 0) return PA_OK;
  return anneal_steps(in, eps_target, beta_max, 0.0, n_sweeps, max_steps, obs, steps_done);
}

int pa_choose_beta(pa_instance* in, double eps_target, double beta_max, double* beta_next) {
  if (int rc0 = enter(in)) return rc0;
  if (!beta_next || !std::isfinite(eps_target) || !std::isfinite(beta_max) || eps_target < 0.0)
    return PA_EINVAL;
  if (!(beta_max > in->beta)) return PA_EINVAL;
  if (int rc = check_energy(in)) return rc;
  if (!in->hist_valid || in->pending_gather) {
    int rc = fetch_hist(in, false);
    if (rc) return rc;
  }
  return choose_from_hist(in, eps_target, beta_max, beta_next);
}

int pa_observables(pa_instance* in, pa_obs* out) {
  if (int rc0 = enter(in)) return rc0;
  if (!out) return PA_EINVAL;
  int rc = check_energy(in);
  if (rc) return rc;
  rc = fetch_hist(in, true);
  if (rc) return rc;
  fill_observables(in, out);
  return PA_OK;
}

int pa_overlap_hist(pa_instance* a, pa_instance* b, uint32_t nbins, uint64_t* hist_out) {
  if (!usable(a) || !usable(b)) return PA_ESTATE;
  if (int rc0 = enter(a)) return rc0;
  if (int rc0 = enter(b)) return rc0;
  if (nbins != 65 || !hist_out || a == b) return PA_EINVAL;
  if (a->dev.L != b->dev.L || a->dev.layout != b->dev.layout) return PA_EINVAL;
  int rc = materialize(a);
  if (rc) return rc;
  rc = materialize(b);
  if (rc) return rc;
  PA_HIP(b, hipStreamSynchronize(b->stream));
  PA_HIP(a, pa::launch_fill_u32(reinterpret_cast<uint32_t*>(a->dev.ovl_hist), 0u, 130, a->stream));
  PA_HIP(a, pa::launch_overlap_pair(a->dev, b->dev, a->cur, b->cur, a->stream));
  PA_HIP(a, hipMemcpyAsync(a->h_ovl, a->dev.ovl_hist, 65 * 8, hipMemcpyDeviceToHost, a->stream));
  PA_HIP(a, hipStreamSynchronize(a->stream));
  for (int i = 0; i < 65; ++i) hist_out[i] = a->h_ovl[i];
  return PA_OK;
}

int pa_link_overlap_hist(pa_instance* a, pa_instance* b, uint32_t nbins, uint64_t* hist_out) {
  if (!usable(a) || !usable(b)) return PA_ESTATE;
  if (int rc0 = enter(a)) return rc0;
  if (int rc0 = enter(b)) return rc0;
  if (!hist_out || a == b) return PA_EINVAL;
  if (a->dev.L != b->dev.L || a->dev.layout != b->dev.layout) return PA_EINVAL;
  if (nbins != 3 * a->dev.N + 1) return PA_EINVAL;
  int rc = materialize(a);
  if (rc) return rc;
  rc = materialize(b);
  if (rc) return rc;
  PA_HIP(b, hipStreamSynchronize(b->stream));
  PA_HIP(a, pa::launch_fill_u32(a->dev.lovl_part, 0u, (size_t)pa::kLinkCopies * nbins,
                                a->stream));
  PA_HIP(a, pa::launch_link_overlap(a->dev, b->dev, a->cur, b->cur, a->dev.lovl_part,
                                    a->dev.lovl_hist, a->stream));
  PA_HIP(a, hipMemcpyAsync(a->h_lovl, a->dev.lovl_hist, (size_t)nbins * 8, hipMemcpyDeviceToHost,
                           a->stream));
  PA_HIP(a, hipStreamSynchronize(a->stream));
  for (uint32_t i = 0; i < nbins; ++i) hist_out[i] = a->h_lovl[i];
  return PA_OK;
}

int pa_link_overlap_hist_noalloc(pa_instance* a, pa_instance* b, uint32_t nbins,
                                 uint64_t* hist_out) {
  if (!usable(a) || !usable(b)) return PA_ESTATE;
  if (int rc0 = enter(a)) return rc0;
  if (int rc0 = enter(b)) return rc0;
  if (!hist_out || a == b) return PA_EINVAL;
  if (a->dev.L != b->dev.L || a->dev.layout != b->dev.layout) return PA_EINVAL;
  if (nbins != 3 * a->dev.N + 1) return PA_EINVAL;
  if (nbins > PA_NOALLOC_MAX_BINS) return PA_ENOMEM;  // beyond the fixed array
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return PA_EDEVICE;
  if (dev != a->device || dev != b->device) return PA_EINVAL;
  uint32_t* const part = scratch_of(dev);
  if (!part) return PA_EDEVICE;
  unsigned long long* const hist = reinterpret_cast<unsigned long long*>(part + kScratchPartWords);
  int rc = materialize(a);
  if (rc) return rc;
  rc = materialize(b);
  if (rc) return rc;
  PA_HIP(b, hipStreamSynchronize(b->stream));
  // the partial counts start at zero (the array keeps the last call's)
  PA_HIP(a, pa::launch_fill_u32(part, 0u, (size_t)pa::kLinkCopies * nbins, a->stream));
  PA_HIP(a, pa::launch_link_overlap(a->dev, b->dev, a->cur, b->cur, part, hist, a->stream));
  PA_HIP(a, hipMemcpyAsync(a->h_lovl, hist, (size_t)nbins * 8, hipMemcpyDeviceToHost, a->stream));
  PA_HIP(a, hipStreamSynchronize(a->stream));
  for (uint32_t i = 0; i < nbins; ++i) hist_out[i] = a->h_lovl[i];
  return PA_OK;
}

// Replicas whose canonical spins (one byte each) fit in a spin buffer: a multiple
// of 32, as the capacity is one of 256.
static uint32_t staged_replicas(const DevPop& P) {
  return P.layout == PA_LAYOUT_BITPACK64 ? P.capacity / 8 : P.capacity;
}

// Bytes of the tiles that hold R replicas.
static size_t tiles_bytes(const DevPop& P, uint32_t R) {
  return (size_t)((R + 63) / 64) * P.N * (P.layout == PA_LAYOUT_BITPACK64 ? 8 : 64);
}

// Spins of R replicas from the bytes of their tiles to the canonical layout on the
// host, and (bit-packed) back into zeroed bytes.
static void unpack_spins(const pa_instance* in, const uint8_t* tiles, uint32_t R, int8_t* out) {
  const uint32_t N = in->dev.N;
  for (uint32_t r = 0; r < R; ++r, out += N) {
    const uint32_t lane = r & 63u;
    if (in->dev.layout == PA_LAYOUT_BITPACK64) {
      const uint8_t* const t = tiles + (size_t)(r >> 6) * N * 8 + (lane >> 3);
      for (uint32_t s = 0; s < N; ++s)
        out[s] = (int8_t)(1 - 2 * ((t[8 * in->cm_of_site[s]] >> (lane & 7u)) & 1));
    } else {
      const uint8_t* const t = tiles + (size_t)(r >> 6) * N * 64 + lane;
      for (uint32_t s = 0; s < N; ++s) out[s] = (int8_t)t[64 * in->cm_of_site[s]] < 0 ? -1 : 1;
    }
  }
}

static void pack_spins(const pa_instance* in, const int8_t* spins, uint32_t R, uint8_t* tiles) {
  const uint32_t N = in->dev.N;
  for (uint32_t r = 0; r < R; ++r, spins += N) {
    const uint32_t lane = r & 63u;
    uint8_t* const t = tiles + (size_t)(r >> 6) * N * 8 + (lane >> 3);
    for (uint32_t s = 0; s < N; ++s)
      t[8 * in->cm_of_site[s]] |= (uint8_t)((spins[s] < 0 ? 1u : 0u) << (lane & 7u));
  }
}

// Spins below which an export and an import convert on the host.  On the device each
// piece (up to eight in the bit-packed layout) costs a launch and a copy of its own,
// 20 to 30 us; the host takes about 0.4 ns a spin (us on the host / on the device, out:
// bit-packed L = 4, 128000 spins 89 / 185, L = 6, 432000 spins 215 / 223, L = 8,
// 512000 spins 252 / 218; int8 L = 6, 15120 spins 40 / 50, L = 4, 32000 spins 57 / 50; in:
// bit-packed L = 6, 432000 spins 219 / 254, L = 4, 640000 spins 250 / 239; int8 never
// more than 3 us faster on the host).
static bool export_on_host(const DevPop& P, uint32_t R) {
  return (uint64_t)R * P.N < (P.layout == PA_LAYOUT_BITPACK64 ? 430000u : 30000u);
}
static bool import_on_host(const DevPop& P, uint32_t R) {
  return P.layout == PA_LAYOUT_BITPACK64 && (uint64_t)R * P.N < 640000u;
}

int pa_export_state(pa_instance* in, int8_t* spins_host, uint32_t* U_host, uint32_t* family_host,
                    uint32_t* R_tilde) {
  if (int rc0 = enter(in)) return rc0;
  if (!R_tilde) return PA_EINVAL;
  if (U_host && in->dev.model == pa::kModelReal) return PA_EINVAL;  // pa_export_energies
  int rc = materialize(in);
  if (rc) return rc;
  const DevPop& P = in->dev;
  PA_HIP(in, hipMemcpyAsync(in->h_sc, P.sc, sizeof(DevScalars), hipMemcpyDeviceToHost, in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  const uint32_t R = in->h_sc->R_tilde;
  in->R_tilde = R;
  *R_tilde = R;
  if (U_host && R)
    PA_HIP(in, hipMemcpy(U_host, P.U[in->cur], (size_t)R * 4, hipMemcpyDeviceToHost));
  if (family_host && R)
    PA_HIP(in, hipMemcpy(family_host, P.fam[in->cur], (size_t)R * 4, hipMemcpyDeviceToHost));
  if (spins_host && R && export_on_host(P, R)) {
    std::vector<uint8_t> tiles(tiles_bytes(P, R));
    PA_HIP(in, hipMemcpy(tiles.data(), P.spins[in->cur], tiles.size(), hipMemcpyDeviceToHost));
    unpack_spins(in, tiles.data(), R, spins_host);
  } else if (spins_host && R) {
    // the population's other buffer is free between calls: converted there and
    // copied out, as many replicas at a time as it holds
    const uint32_t per = staged_replicas(P);
    int8_t* const stage = static_cast<int8_t*>(P.spins[in->cur ^ 1u]);
    for (uint32_t r0 = 0; r0 < R; r0 += per) {
      const uint32_t rows = std::min(per, R - r0);
      PA_HIP(in, pa::launch_export_spins(P, in->cur, stage, R, r0, r0 + rows, in->stream));
      PA_HIP(in, hipMemcpyAsync(spins_host + (size_t)r0 * P.N, stage, (size_t)rows * P.N,
                                hipMemcpyDeviceToHost, in->stream));
    }
    PA_HIP(in, hipStreamSynchronize(in->stream));
  }
  return PA_OK;
}

int pa_export_counts(pa_instance* in, uint32_t* counts_host, uint32_t* offsets_host,
                     uint32_t* n_old) {
  if (int rc0 = enter(in)) return rc0;
  if (!n_old) return PA_EINVAL;
  *n_old = in->last_R_old;
  if (in->step == 0) return PA_ESTATE;
  PA_HIP(in, hipStreamSynchronize(in->stream));
  const size_t n = in->last_R_old;
  if (counts_host && n)
    PA_HIP(in, hipMemcpy(counts_host, in->dev.counts, n * 4, hipMemcpyDeviceToHost));
  if (offsets_host && n)
    PA_HIP(in, hipMemcpy(offsets_host, in->dev.offsets, n * 4, hipMemcpyDeviceToHost));
  return PA_OK;
}

int pa_import_state(pa_instance* in, const int8_t* spins_host, const uint32_t* family_host,
                    uint32_t R_tilde, uint64_t sweeps_done, uint32_t step, double beta,
                    double sum_lnQ) {
  if (int rc0 = enter(in)) return rc0;
  const DevPop& P = in->dev;
  if (!spins_host || !family_host || R_tilde > P.cap_limit || !std::isfinite(beta) ||
      !std::isfinite(sum_lnQ) || sweeps_done > 0xFFFFFFFFull)
    return PA_EINVAL;
  for (uint32_t i = 0; i < R_tilde; ++i) {
    if (family_host[i] >= P.R) return PA_EINVAL;
    if (i && family_host[i] < family_host[i - 1]) return PA_EINVAL;  // labels must be sorted
  }
  // every spin is +1 or -1: s + 1 is 2 or 0
  const size_t n_spins = (size_t)R_tilde * P.N;
  uint8_t other = 0;
  for (size_t i = 0; i < n_spins; ++i) other |= (uint8_t)(spins_host[i] + 1) & (uint8_t)~2u;
  if (other != 0) return PA_EINVAL;
  int rc = materialize(in);  // drop nothing silently: finish a pending copy first
  if (rc) return rc;
  PA_HIP(in, hipStreamSynchronize(in->stream));
  if (R_tilde && import_on_host(P, R_tilde)) {
    std::vector<uint8_t> tiles(tiles_bytes(P, R_tilde), 0);
    pack_spins(in, spins_host, R_tilde, tiles.data());
    PA_HIP(in, hipMemcpy(P.spins[in->cur], tiles.data(), tiles.size(), hipMemcpyHostToDevice));
  } else {
    // staged in the population's other buffer and converted, as many replicas at a
    // time as it holds; the last slots of the last tile are cleared
    const uint32_t slots = (R_tilde + 63) / 64 * 64, per = staged_replicas(P);
    int8_t* const stage = static_cast<int8_t*>(P.spins[in->cur ^ 1u]);
    for (uint32_t r0 = 0; r0 < slots; r0 += per) {
      const uint32_t r1 = std::min(r0 + per, slots);
      if (r0 < R_tilde)
        PA_HIP(in, hipMemcpyAsync(stage, spins_host + (size_t)r0 * P.N,
                                  (size_t)(std::min(r1, R_tilde) - r0) * P.N,
                                  hipMemcpyHostToDevice, in->stream));
      PA_HIP(in, pa::launch_import_spins(P, in->cur, stage, R_tilde, r0, r1, in->stream));
    }
    PA_HIP(in, hipStreamSynchronize(in->stream));
  }
  if (R_tilde)
    PA_HIP(in, hipMemcpy(P.fam[in->cur], family_host, (size_t)R_tilde * 4, hipMemcpyHostToDevice));
  DevScalars sc{};
  sc.R_tilde = R_tilde;
  PA_HIP(in, hipMemcpy(P.sc, &sc, sizeof(sc), hipMemcpyHostToDevice));
  PA_HIP(in, pa::launch_energy(one_set(in, plain_step(in->cur)),
                               group_of(in, in->d_meta->etiles, in->meta.etiles[1]), P.layout,
                               P.L, P.model, false, in->stream));
  PA_HIP(in, hipStreamSynchronize(in->stream));
  in->R_tilde = R_tilde;
  in->sweeps = sweeps_done;
  in->step = step;
  in->beta = beta;
  in->sum_lnQ = sum_lnQ;
  in->pending_gather = false;
  in->hist_valid = false;
  in->last_R_old = 0;
  return PA_OK;
}

int pa_autotune_sweep(pa_instance* in, double beta, uint32_t n_sweeps, uint32_t repeats,
                      uint32_t* split_out, float* ms_out) {
  if (int rc0 = enter(in)) return rc0;
  if (in->pending_gather) return PA_ESTATE;
  if (!(beta >= 0.0) || !std::isfinite(beta)) return PA_EINVAL;
  if (n_sweeps == 0 || repeats == 0 || repeats > 1000) return PA_EINVAL;
  // Trial sweeps at the caller's inverse temperature read the population's
  // buffer and write the other one; the population, its counters and the
  // current buffer are left as they were.
  pa::PopStep ps = plain_step(in->cur);
  if (set_thresholds(in, beta, &ps) != hipSuccess) return dev_fail(in);
  ps.t0 = (uint32_t)in->sweeps;
  ps.n_sweeps = n_sweeps;
  ps.gather = 0;
  const uint64_t tiles = ((uint64_t)in->R_tilde + 63) / 64;
  const uint32_t cand[2] = {4u, 8u};
  float ms[2] = {0.0f, 0.0f};
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return dev_fail(in);
  }
  int rc = PA_OK;
  const pa::BatchDev B = one_set(in, ps);
  auto launch = [&](uint32_t split) {
    const uint32_t form = pa::sweep_form(in->dev.model, in->dev.L, split, tiles);
    return pa::launch_sweep(B, sweep_group(in, form), in->dev.layout, in->dev.L, form,
                            in->dev.model, in->stream) == hipSuccess;
  };
  // two untimed launches of each form (clocks and caches settle), then the
  // timed launches alternate between the forms so that drift hits both alike
  bool ok = launch(cand[0]) && launch(cand[1]) && launch(cand[0]) && launch(cand[1]);
  for (uint32_t r = 0; ok && r < repeats; ++r)
    for (int c = 0; ok && c < 2; ++c) {
      float t = 0.0f;
      ok = hipEventRecord(e0, in->stream) == hipSuccess && launch(cand[c]) &&
           hipEventRecord(e1, in->stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
           hipEventElapsedTime(&t, e0, e1) == hipSuccess;
      ms[c] += t;
    }
  if (!ok) rc = dev_fail(in);
  ms[0] /= (float)repeats;
  ms[1] /= (float)repeats;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != PA_OK) return rc;
  const uint32_t best = ms[1] < ms[0] ? cand[1] : cand[0];
  pa::sweep_split_record(in->dev.model, in->dev.layout, in->dev.L, tiles, best);
  if (split_out) *split_out = best;
  if (ms_out) {
    ms_out[0] = ms[0];
    ms_out[1] = ms[1];
  }
  return PA_OK;
}

size_t pa_autotune_layout_workspace_bytes(const pa_params* p) {
  if (!p) return 0;
  size_t most = 0;
  for (uint32_t lay : {(uint32_t)PA_LAYOUT_INT8, (uint32_t)PA_LAYOUT_BITPACK64}) {
    pa_params q = *p;
    q.layout = lay;
    q.flags = 0;
    Layout l;
    if (!make_layout(&q, &l)) return 0;
    most = std::max(most, l.total);
  }
  return most;
}

int pa_autotune_layout(const pa_params* p, const int8_t* J_host, void* d_workspace,
                       size_t ws_bytes, void* hip_stream, double beta, uint32_t n_sweeps,
                       uint32_t repeats, uint32_t* layout_out, float* ms_out) {
  if (!p || !J_host || !d_workspace) return PA_EINVAL;
  const size_t need = pa_autotune_layout_workspace_bytes(p);
  if (need == 0) return PA_EINVAL;
  if (ws_bytes < need) return PA_ENOMEM;
  if (!(beta >= 0.0) || !std::isfinite(beta)) return PA_EINVAL;
  if (n_sweeps == 0 || repeats == 0 || repeats > 1000) return PA_EINVAL;
  const uint32_t lays[2] = {(uint32_t)PA_LAYOUT_INT8, (uint32_t)PA_LAYOUT_BITPACK64};
  float best_ms[2] = {0.0f, 0.0f};
  for (int i = 0; i < 2; ++i) {
    // a throwaway population of each layout in the caller's workspace; the
    // split autotuner times both sweep forms on it and records the faster
    pa_params q = *p;
    q.layout = lays[i];
    q.flags = 0;
    pa_instance* in = nullptr;
    if (int rc = pa_init_instance(&q, J_host, d_workspace, ws_bytes, hip_stream, &in)) return rc;
    float ms[2] = {0.0f, 0.0f};
    const int rc = pa_autotune_sweep(in, beta, n_sweeps, repeats, nullptr, ms);
    const int rc_free = pa_free(in);
    if (rc != PA_OK) return rc;
    if (rc_free != PA_OK) return rc_free;
    best_ms[i] = std::min(ms[0], ms[1]);
  }
  const uint32_t best = best_ms[1] <= best_ms[0] ? lays[1] : lays[0];
  pa::layout_record(p->model, p->L, ((uint64_t)p->R + 63) / 64, best);
  if (layout_out) *layout_out = best;
  if (ms_out) {
    ms_out[0] = best_ms[0];
    ms_out[1] = best_ms[1];
  }
  return PA_OK;
}

}  // extern "C"
