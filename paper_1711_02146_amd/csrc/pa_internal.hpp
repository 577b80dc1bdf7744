// pa_internal.hpp -- types shared by the HIP kernels and the host side of
// libpa (the C-ABI implementation).  Nothing here is visible to callers.
//
// Method: Amey & Machta, arXiv:1711.02146 (Sec. II annealing loop, Eqs. 1-2
// resampling, Sec. II.A model and observables, Sec. III.A rho_t).
//
// Every kernel works on a set of populations: a device array of DevPop plus a
// Group that maps each workgroup to (member population, block within it).  A
// single instance is a set of one.  Per-launch parameters come either by value
// (calls on one instance) or from a device array indexed by a device step
// counter, so that one captured graph can be replayed for every temperature
// step of a batch.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#define PA_HD __host__ __device__
#include "pa_search.hpp"

namespace pa {

// Philox stream tags (fourth counter word): one per use of the generator.
constexpr uint32_t kTagInit = 0x494E4954u;  // initial spins
constexpr uint32_t kTagMet = 0x4D455452u;   // Metropolis acceptance draws
constexpr uint32_t kTagRes = 0x52455341u;   // copy-count draws
constexpr uint32_t kTagJ = 0x434F5550u;     // +-J couplings (pa_make_couplings_pm)

constexpr int kWave = 64;          // wavefront width on gfx950; one spin tile = 64 replicas
constexpr int kBlockCounts = 256;  // slots per block in the copy-count / scatter kernels
constexpr int kHistSlots = 4096;   // slots per block of the histogram kernel
constexpr int kWindowLdsLevels = 16384;  // largest E16 window counted in LDS (64 KiB)
constexpr int kMaxL = 16;
// k_sweep (Gaussian couplings, L >= 12): per wave, one byte for each of 64 sites x 64
// replicas, the neighbour pattern (phase 1 of the colour pass: one site per lane).
constexpr uint32_t kPlaneAreaBytes = 64 * 64;
constexpr uint32_t kOverlapTiles = 8;  // 64-pair tiles (one wave each) per workgroup of k_overlap
constexpr uint32_t kLinkCopies = 32;  // partial link-overlap histograms (see launch_link_overlap)
// Energy models.  kModelPm: J = +-1, the energy word of a replica is U, the
// number of unsatisfied bonds (E = 2U - 3N).  kModelGauss16: J = k / 16 with
// k in [-127, 127], the energy word is E16 = -sum_b k_b s_i s_j (E = E16 / 16),
// stored as int32.
constexpr uint32_t kModelPm = 0;
constexpr uint32_t kModelGauss16 = 1;
// kModelReal: real Gaussian couplings (Sec. II.A) carried on the grid 2^-32
// with |J| < 8.  The energy word is the int64 E32 = E 2^32, exact: every sum
// of at most 3N such couplings fits in 49 bits.  Per site (colour-major cm)
// and per pattern y of its six "neighbour differs" bits (bit k: s_i != s_k,
// k in the order +x,-x,+y,-y,+z,-z), he[cm][y] = sum_k k_k (1 - 2 y_k) with
// k_k = J_k 2^32: flipping s_i changes E32 by 2 he, and the site's bond
// energy is -he before and +he after the flip.
constexpr uint32_t kModelReal = 2;
constexpr uint32_t kRealPatterns = 64;  // patterns y per site
// Rows (sites) past the last of the per-(site, pattern) tables: the Gaussian
// colour pass reads one group of four sites past a 64-site chunk ahead, whose
// entries it never uses.
constexpr uint32_t kPatternPadRows = 64;
// Workgroups of the kModelReal weight reductions (grid-stride over the
// replicas), one per CU: a reduction of three sums over R = 5e5 words takes 17
// us on 256 workgroups, 21 us on 128 and 29 us on 1024 (each workgroup's arrival
// costs a device-scope fence and atomic).
constexpr uint32_t kRealSumBlocks = 256;
constexpr int kGaussKMax = 127;
constexpr int kGaussDEMax = 2 * 6 * kGaussKMax;  // largest |dE16| of one flip

// One lattice site in colour-major order (cm): colour-0 sites first, then
// colour-1 sites, each in lexicographic order; for even L, cm = c*N/2 + (site >> 1).
// nb[k] are the colour-major indices of the six neighbours (+x,-x,+y,-y,+z,-z),
// bit k of jneg is set when the coupling to neighbour k is -1, site is the
// lexicographic index.  16 bytes: one scalar load per site.
struct SiteEntry {
  uint16_t nb[6];
  uint16_t jneg;
  uint16_t site;
};
static_assert(sizeof(SiteEntry) == 16, "SiteEntry must be 16 bytes");

// LDS address of the tile image in k_sweep: right after its first eight words, which
// sit at address 0 (the kernel checks both).
constexpr uint32_t kTileLdsBase = 64;

// The same site for phase 1 of k_sweep's colour passes (lane = site), laid out so
// that nothing needs unpacking: the LDS addresses kTileLdsBase + 8 nb[k] of
// the six neighbours' words, and the coupling bits.  32 bytes: two 16-byte
// loads per lane.
struct PlaneSite {
  uint32_t nb8[6];
  uint32_t jneg;
  uint32_t pad;
};
static_assert(sizeof(PlaneSite) == 32, "PlaneSite must be 32 bytes");

// The +-J sweep (k_sweep_pm): LDS address of the tile image, after the 4 KB
// threshold table, and the bytes of a wave's plane area (32 groups of four
// sites x 64 replicas, one byte each).
constexpr uint32_t kPmImage = 4096;
constexpr uint32_t kPmPlaneBytes = 32 * 64;
// Forms of the +-J sweep (see PmShape): 4 or 8 waves on one tile, or, for L <= 8,
// four waves on several tiles: waves and tiles per workgroup.
constexpr uint32_t kPmPacked = 1;
__host__ __device__ constexpr uint32_t pm_waves(uint32_t split) { return split == 8 ? 8 : 4; }
__host__ __device__ constexpr uint32_t pm_tiles(uint32_t L, uint32_t split) {
  return split != kPmPacked ? 1 : L <= 6 ? 4 : L == 8 ? 2 : 1;
}

// The Gaussian sweep with its table in LDS (k_sweep_gauss, L <= 10): waves and tiles
// per workgroup, bytes of a wave's plane area (16 sites x 64 replicas, one byte
// each), waves per SIMD that its registers are budgeted for (as many as the LDS lets
// run at L = 10, one workgroup of 16 waves), and the workgroups that fill 256 CUs.  With
// 128 registers L = 8 on several tiles keeps 39 to 53 more in scratch memory (152 to 208
// bytes a lane); the other sizes and the one-tile forms keep none there.
constexpr uint32_t kGaussLds = 2;     // several tiles per workgroup
constexpr uint32_t kGaussLdsOne = 3;  // one tile, for launches that leave the chip idle
constexpr uint32_t kGaussPlaneBytes = 16 * 64;
__host__ __device__ constexpr uint32_t gauss_waves(uint32_t L) { return L == 10 ? 16 : 8; }
__host__ __device__ constexpr uint32_t gauss_tiles(uint32_t L, uint32_t form) {
  return form == kGaussLdsOne ? 1 : L == 4 ? 8 : L == 6 ? 4 : 2;
}
constexpr int kGaussWavesPerEu = 4;
inline uint32_t gauss_resident(uint32_t L) {
  return 256 * 4 * (uint32_t)kGaussWavesPerEu / gauss_waves(L);
}

// A site for one 32-replica half of a lane in phase 1 of the +-J colour pass:
// the byte offsets of the six neighbours' words of that half in the tile's
// image and the coupling bits.  The table holds, for each group of four consecutive sites, the four
// sites for the low half, then for the high half: a lane reads 64 bytes in a row.
struct PmSite {
  uint16_t nb[6];
  uint32_t jneg;
};
static_assert(sizeof(PmSite) == 16 && 2 * sizeof(PmSite) == sizeof(PlaneSite),
              "a site takes 32 bytes in either table");

// Device-resident scalars of one population.
struct DevScalars {
  uint32_t R_tilde;       // size of the current population
  uint32_t R_next;        // size after the pending copy step (written by the scan)
  uint32_t err;           // 1: the pending copy step would exceed the capacity;
                          // 2: a kernel found its LDS layout unusable
  uint32_t n_culled;      // replicas with zero copies in the last resampling step
  unsigned long long sum_eta2;  // sum over families of eta^2
  uint32_t check_bad;     // energy check: replicas whose stored word differs from the spins'
  uint32_t dead;          // batch runs: set when a step overflowed; later steps skip it
  int32_t E_lo, E_hi;     // kModelGauss16: lowest / highest E16 of the population
  uint32_t pad[6];
};
static_assert(sizeof(DevScalars) == 64, "DevScalars is 64 bytes");

// Device scalars of a kModelReal population (after DevScalars in the same
// block, so one copy brings both to the host).  The reductions over replicas
// finish in the last workgroup to arrive (counter `done`, reset by it).
struct RealScalars {
  long long E_min;             // lowest energy word (k_rstats)
  unsigned long long sumE_lo;  // sum of the energy words, a 128-bit two's-complement
  long long sumE_hi;           //   integer (low and high word)
  uint32_t n_at_min;           // replicas at E_min
  uint32_t done;               // workgroups arrived at the current reduction
  double S;                    // sum of the weights of dbeta (Eq. 2, fixed point, rounded)
  double eps;                  // culled fraction (Sec. III.C) of the last copy-count pass
  double lo;                   // end of the constant-culling search: its lower end
  int32_t result;              // 0 running, 1 whole range, 2 bisected (lo), -1 impossible
  uint32_t pad;
};
static_assert(sizeof(RealScalars) == 64, "RealScalars is 64 bytes");

// State of the constant-culling search of a kModelReal population: the search
// and the sums of the weights at its candidates.
struct RealSearch {
  CullSearch s;
  double S[kCullLanes];
};
static_assert(sizeof(RealSearch) % 8 == 0, "copied in 8-byte words");

// One workgroup's share of a kModelReal reduction.
struct RealPartial {
  unsigned long long lo;  // fixed-point sum (unsigned) or energy sum (signed), low word
  unsigned long long hi;  //   high word
  long long m;            // lowest energy word
  uint32_t c;             // replicas at m
  uint32_t pad;
};
static_assert(sizeof(RealPartial) == 32, "RealPartial is 32 bytes");

// One energy level of the resampling table (Sec. II copy rule): a replica
// at that level gets fl copies, and one more iff a 53-bit draw is below T.
// The two live together so that the table goes to the device in one copy.
struct TableEntry {
  unsigned long long T;  // ceil(frac(tau_j) 2^53)
  uint32_t fl;           // floor(tau_j)
  uint32_t pad;
};
static_assert(sizeof(TableEntry) == 16, "TableEntry is 16 bytes");

// The occupied range of a resampling table passed by value to the copy-count
// kernel of a single population, when it fits: no separate upload (and no
// dispatch between the upload and the kernel).  Entry e[j - j0] is level j.
constexpr uint32_t kInlineLevels = 224;
struct InlineTable {
  uint32_t j0, n;
  uint32_t pad[2];
  TableEntry e[kInlineLevels];
};
static_assert(sizeof(InlineTable) == 16 + 16 * kInlineLevels, "InlineTable layout");

// Device pointers of one population (all inside its workspace).
struct DevPop {
  uint32_t L, N, R, capacity;   // capacity: slots per buffer, a multiple of kBlockCounts
  uint32_t layout;              // PA_LAYOUT_INT8 or PA_LAYOUT_BITPACK64
  uint32_t n_levels;            // 3N + 1
  uint32_t n_blocks;            // capacity / kBlockCounts
  uint32_t cap_limit;           // a resampled population may not exceed this (<= capacity)
  uint64_t seed;
  void* spins[2];               // tile-major spin buffers (see pa.h)
  uint32_t* U[2];
  uint32_t* fam[2];
  uint32_t* counts;             // n_i of the last resampling step
  uint32_t* offsets;            // exclusive scan of counts
  uint32_t* src;                // new slot -> old slot of the pending copy step
  uint32_t* block_sums;         // per block of kBlockCounts slots
  uint32_t* block_culled;
  uint32_t* hist;               // n_levels
  struct TableEntry* table;     // n_levels: the resampling table by energy level
  const SiteEntry* sites;       // N entries, colour-major
  const PlaneSite* psites;      // Gaussian models: N entries, colour-major (phase 1 of the colour
                                // passes)
  const PmSite* pmsites;        // kModelPm, in their place: 2 N entries [N / 4][2][4]
  const uint16_t* cm_of_site;   // N entries: lexicographic site -> colour-major index
  const unsigned long long* rowj;  // 2 L^2 row words: bit 6q + k set iff the bond from
                                   // site q of row (colour, y, z) to neighbour k is -1
  unsigned long long* ovl_hist; // 65 bins, scratch of the overlap histogram
  unsigned long long* lovl_hist;  // 3N + 1 bins, scratch of the link-overlap histogram
  uint32_t* lovl_part;            // kLinkCopies x (3N + 1) partial link-overlap counts
  DevScalars* sc;
  uint32_t model;               // kModelPm or kModelGauss16
  uint32_t rowk_stride;         // kModelGauss16: bytes per row of rowk (6 L/2 rounded up to 4)
  const int8_t* rowk;           // kModelGauss16: 2 L^2 rows; byte 6q + k of a row is the
                                // coupling k of its site q to neighbour k (J = k / 16)
  const unsigned long long* gthr;  // kModelGauss16: thr[d] = floor(2^32 exp(-beta d / 16)),
                                   // d = 0..kGaussDEMax, for the coming sweep
  const uint16_t* gaddr;            // kModelGauss16: 16 max(he16[cm][y], 0), N x 64, with he16
                                   // the he of kModelReal in units 1/16: the byte offset of the
                                   // move's threshold in the dE16 table (dE16 = 2 he16)
  const long long* rhe;            // kModelReal: he[cm][y], N x 64 (see kModelReal)
  unsigned long long* rthr;        // kModelReal: Metropolis threshold of (cm, y) for the
                                   // coming sweep, N x 64
  uint32_t* rthr32;                // kModelReal: min(thr, 2^32 - 1) of the same (cm, y): the
                                   // sweep's table (see pattern_thr)
  RealScalars* rs;                 // kModelReal: scalars of the weight reductions
  RealPartial* rpart;              // kModelReal: one per workgroup of kBlockCounts slots, and
                                   // kCullLanes per reduction workgroup
  RealSearch* rsearch;             // kModelReal: the constant-culling search
};

// Parameters of one population for one launch.
struct PopStep {
  unsigned long long thr[3];  // Metropolis thresholds (dE = 4, 8, 12): accept iff word < thr
  const double* erow;         // device table path: erow[d] = exp(-dbeta * 2d), d = 0..3N
  uint32_t t0;                // population sweep counter at the first sweep
  uint32_t n_sweeps;
  uint32_t gather;            // 1: the sweep applies the pending copy step (size R_next)
  uint32_t cur;               // buffer holding the population at the start of the launch
  uint32_t step;              // resampling step index k (copy-count Philox counter)
  uint32_t flags;             // kStepSticky: an overflow marks the population dead; kStepHist
  double dbeta;               // kModelReal: the resampling step of the copy-count pass
};
static_assert(sizeof(PopStep) == 64, "PopStep is 64 bytes");
constexpr uint32_t kStepSticky = 1u;
// kStepHist (+-J): the scan also clears the energy histogram and the family
// sum, for the histogram and family kernels that follow the sweep (no
// separate clearing launch).
constexpr uint32_t kStepHist = 2u;

// What a batch records for one population at one temperature step.
struct StepRecord {
  double S;                // sum_j h_j w_j of the resampling table (Eq. 2, shifted)
  double eps;              // culling fraction of the step (Sec. III.C)
  long long sumE;          // sum over the post-sweep population of E (integer)
  unsigned long long sum_eta2;
  int32_t jmin;            // lowest occupied level before resampling
  uint32_t R_old;          // population size before resampling
  uint32_t R_new;          // population size after resampling and sweeps
  uint32_t n_culled;
  int32_t E_min;           // lowest energy after the sweeps
  uint32_t status;         // 0 ok, 1 capacity overflow (population dead from here on),
                           // 2 the sweep kernel found its LDS layout unusable (dead)
  uint32_t n_at_E_min;     // replicas at E_min
  uint32_t pad;
};
static_assert(sizeof(StepRecord) == 64, "StepRecord is 64 bytes");

// A set of populations as the kernels see it.
struct BatchDev {
  const DevPop* pops;         // n_pops descriptors
  const PopStep* steps;       // per-step parameters [n][n_pops], or nullptr: use `single`
  const uint32_t* step_ctr;   // index of the current step into `steps`
  StepRecord* records;        // [n][n_pops] results of batch steps, or nullptr
  unsigned long long* qhist;  // [n][n_pairs][65] overlap histograms, or nullptr
  uint32_t n_pops;
  uint32_t n_pairs;
  PopStep single;             // parameters of a call on one population
};

// Workgroup -> population map of one launch: member m owns workgroups
// start[m] .. start[m+1]-1 and is population pop[m] of the set.
struct Group {
  const uint32_t* pop;
  const uint32_t* start;  // n + 1 entries, start[0] = 0
  uint32_t n;
  uint32_t blocks;        // start[n]
};

// Launchers (pa_kernels.hip).  All are asynchronous on `stream`.
hipError_t launch_fill_u32(uint32_t* p, uint32_t value, size_t n, hipStream_t stream);

// Diagnostics (pa_probe_ceilings): kProbeThreads lanes, each writing one word
// of `out`; the VALU probe issues kProbeValuOpsPerIter instructions per
// iteration (form 0: v_add_u32, form 1: v_bfe_u32), the Philox probe makes
// `calls` Metropolis Philox calls (4 draws each).
constexpr uint32_t kProbeThreads = 2048 * 256;
constexpr int kProbeValuOpsPerIter = 32;
hipError_t launch_probe_valu(uint32_t* out, uint32_t iters, uint32_t form, hipStream_t stream);
hipError_t launch_probe_philox(uint32_t* out, uint32_t calls, hipStream_t stream);
// The code objects of every lattice size onto the current device (each is one object,
// which HIP otherwise loads at its first launch, inside a caller's sweep, step, graph
// capture or call that must not allocate: 1.2 to 2 ms; all of them 10 ms).
hipError_t load_code();
hipError_t launch_init(const DevPop& P, uint32_t cur, hipStream_t stream);
// the slots r0 .. r1 - 1 (multiples of 32), [replica][site] int8 in device memory,
// from buffer cur (R: replicas of the population) and back into it
hipError_t launch_export_spins(const DevPop& P, uint32_t cur, int8_t* out, uint32_t R,
                               uint32_t r0, uint32_t r1, hipStream_t stream);
hipError_t launch_import_spins(const DevPop& P, uint32_t cur, const int8_t* in, uint32_t R,
                               uint32_t r0, uint32_t r1, hipStream_t stream);
hipError_t launch_zero_acc(const BatchDev& B, const Group& per_pop, hipStream_t stream);
hipError_t launch_hist(const BatchDev& B, const Group& g, uint32_t max_levels,
                       hipStream_t stream);
hipError_t launch_table(const BatchDev& B, const Group& per_pop, hipStream_t stream);
hipError_t launch_counts(const BatchDev& B, const Group& g, hipStream_t stream);
// the same with the table's occupied range passed by value (single populations)
hipError_t launch_counts_inline(const BatchDev& B, const Group& g, const InlineTable& t,
                                hipStream_t stream);
// offsets, new sizes and copy maps (g: the populations' slot blocks)
hipError_t launch_scan_scatter(const BatchDev& B, const Group& g, hipStream_t stream);
// sweep launch over the populations of one (layout, L, model) group in the form
// `split` (see sweep_form); g's blocks are sweep_blocks (one population) or
// blocks_sweep(capacity, sweep_tiles(model, L, split)) per population
hipError_t launch_sweep(const BatchDev& B, const Group& g, uint32_t layout, uint32_t L,
                        uint32_t split, uint32_t model, hipStream_t stream);
// histogram and family sum of the sets' new populations (g: blocks_hist_family
// workgroups each)
hipError_t launch_hist_family(const BatchDev& B, const Group& g, uint32_t max_levels,
                              hipStream_t stream);
hipError_t launch_family(const BatchDev& B, const Group& g, hipStream_t stream);
hipError_t launch_record(const BatchDev& B, const Group& per_pop, hipStream_t stream);
// overlap histograms of a batch step's pairs (blocks_overlap workgroups each)
hipError_t launch_overlap(const BatchDev& B, const Group& pairs, const uint32_t* pair_pops,
                          uint32_t layout, hipStream_t stream);
// the same for two instances, their current buffers cur_a and cur_b, into
// a.ovl_hist (cleared first)
hipError_t launch_overlap_pair(const DevPop& a, const DevPop& b, uint32_t cur_a, uint32_t cur_b,
                               hipStream_t stream);
// energy word of every replica of buffer cur recomputed from its spins: stored
// (check == false), or compared with the stored word, the number of replicas
// that differ added to sc->check_bad (check == true)
hipError_t launch_energy(const BatchDev& B, const Group& g, uint32_t layout, uint32_t L,
                         uint32_t model, bool check, hipStream_t stream);
// link-overlap histogram of slot i of a against slot i of b, i < min of their
// R~ (read on the device): the pairs count into kLinkCopies partial histograms
// part[kLinkCopies][3N + 1] (u32, cleared by the host first), which are then
// summed into hist[D], D = 0..3N
hipError_t launch_link_overlap(const DevPop& a, const DevPop& b, uint32_t cur_a, uint32_t cur_b,
                               uint32_t* part, unsigned long long* hist, hipStream_t stream);
// kModelGauss16: E_lo / E_hi of every member (zero_acc resets them first) and the
// histogram h[E16 - E_lo] (global atomics; the host clears the window first),
// both over the current buffer of a call on single instances
// kModelGauss16 (groups of kHistSlots slots per workgroup): the population's
// E16 range into E_lo / E_hi, then the histogram over the n_win-level window.
hipError_t launch_minmax(const BatchDev& B, const Group& g, hipStream_t stream);
hipError_t launch_hist_window(const BatchDev& B, const Group& g, uint32_t n_win,
                              hipStream_t stream);
hipError_t launch_advance(uint32_t* step_ctr, hipStream_t stream);

// kModelReal (pa_real.hip), single populations, on the current buffer:
// thresholds of every (site, pattern) at beta for the coming sweep
hipError_t launch_real_thresholds(const DevPop& P, double beta, hipStream_t stream);
// E_min, replicas at E_min and the sum of the energy words into P.rs
hipError_t launch_real_stats(const BatchDev& B, const Group& slots, hipStream_t stream);
// the sum S of the weights exp(-dbeta (E - E_min)) at the step's dbeta into P.rs->S
hipError_t launch_real_sum(const BatchDev& B, const Group& slots, hipStream_t stream);
// the constant-culling search (Sec. III.C, pa_search.hpp) over the remaining
// range: its start (after launch_real_stats), then rounds of two launches, the
// sums of the weights at the round's candidates and their culled masses with
// the decision, until P.rs->result is set (launches after that leave at once).
// Each launch runs on `blocks` workgroups (at most kRealSumBlocks) over one
// population, whose buffers it takes as arguments, so that its first loads need
// no descriptor read before them.
struct CullArgs {
  const long long* E;     // energy words of the population's current buffer
  const DevScalars* sc;   // R_tilde
  RealScalars* rs;        // E_min, the arrival counter, the result
  RealSearch* search;
  RealPartial* rpart;     // kCullLanes x blocks partials
  uint32_t R;             // target population size
  uint32_t capacity;      // slots per buffer (every slot below it is allocated)
};
hipError_t launch_real_cull_start(const CullArgs& a, double rem, double target,
                                  hipStream_t stream);
hipError_t launch_real_cull_round(const CullArgs& a, uint32_t blocks, hipStream_t stream);
// copy counts of the step (after launch_real_sum at its dbeta): counts, block
// sums and culled counts as k_counts, and the culled fraction into P.rs->eps
// (`slots`: at most kRealSumBlocks workgroups, each over every nb-th slot block)
hipError_t launch_real_counts(const BatchDev& B, const Group& slots, hipStream_t stream);

// Blocks each population needs in each kind of launch.
inline uint32_t blocks_hist(uint32_t capacity) { return (capacity + kHistSlots - 1) / kHistSlots; }
constexpr uint32_t kFamilyBlocks = 512;  // workgroups of a population that sum its families
inline uint32_t blocks_hist_family(uint32_t capacity) {
  return blocks_hist(capacity) + std::min(capacity / kBlockCounts, kFamilyBlocks);
}
inline uint32_t blocks_overlap(uint32_t capacity) {
  return (capacity / 64 + kOverlapTiles - 1) / kOverlapTiles;
}
inline uint32_t blocks_slots(uint32_t capacity) { return capacity / kBlockCounts; }
// One block per `per_block` tiles, rounded up to a multiple of 8 so that every
// population of a launch starts at a block number divisible by the XCD count
// (the extra blocks find no replicas and leave).
inline uint32_t blocks_sweep(uint32_t capacity, uint32_t per_block) {
  return ((capacity / 64 + per_block - 1) / per_block + 7) / 8 * 8;
}
// Tiles per workgroup of a sweep launch.
inline uint32_t sweep_tiles(uint32_t model, uint32_t L, uint32_t split) {
  return model == kModelPm ? pm_tiles(L, split) : split == kGaussLds ? gauss_tiles(L, split) : 1;
}
// Workgroups of a sweep launch of one population.
inline uint32_t sweep_blocks(uint32_t model, uint32_t L, uint32_t split, uint32_t capacity) {
  const uint32_t all = blocks_sweep(capacity, sweep_tiles(model, L, split));
  return model != kModelPm && (split == kGaussLds || split == kGaussLdsOne)
             ? std::min(all, gauss_resident(L))
             : all;
}
// Waves per workgroup of a sweep launch over `tiles` tiles of linear size L, from
// timings on MI355X (10 sweeps, beta = 1).
// +-J: eight waves on a tile while the launch leaves the chip idle (ms per
// launch with 8 / 4 waves: L = 4, 313 tiles 0.036 / 0.047, 782 tiles 0.059 /
// 0.044; L = 8, 157 tiles 0.059 / 0.070, 313 tiles 0.087 / 0.087; L = 10, 313
// tiles 0.140 / 0.152, 782 tiles 0.247 / 0.243) and from L = 12 up, where eight
// waves still have a full chunk each (L = 12, 3125 tiles 1.152 / 1.175; L = 16,
// 1563 tiles 1.52 / 1.92); at L = 6, whose walk per wave is short either way, where a
// launch leaves most CUs a tile each (8 tiles 0.050 / 0.048, 64 tiles 0.044 / 0.047, 256
// tiles 0.043 / 0.047, 320 tiles 0.063 / 0.054, 1563 tiles 0.186 / 0.132).
// Gaussian models, L <= 10: several tiles per workgroup (4) once that fills the
// chip, one (8) below (ms per launch of 10 sweeps with several / one, real
// couplings: L = 4, 768 tiles 0.055 / 0.046, 1024 tiles 0.054 / 0.062; L = 6, 313
// tiles 0.098 / 0.055, 1024 tiles 0.102 / 0.102, 1536 tiles 0.134 / 0.148; L = 8,
// 1024 tiles 0.165 / 0.176, 1536 tiles 0.266 / 0.256, 2048 tiles 0.327 / 0.351: several
// tiles are ahead where their rounds, of 1024 tiles, are full; one line at 1600).  At
// L = 10 a workgroup fills a CU either way, a round of 256 workgroups takes 5 parts
// of time with two tiles each against 3 with one (512 tiles 0.152 / 0.168, 768
// tiles 0.293 / 0.256, 1024 tiles 0.292 / 0.327, 7813 tiles 2.27 / 2.45), and the
// rounds decide.  From L = 12 up (k_sweep: the table does not fit) eight waves.
inline uint32_t sweep_split_default(uint32_t model, uint32_t L, uint64_t tiles) {
  if (model == kModelPm) {
    if (L == 6) return tiles >= 48 && tiles <= 256 ? 8u : 4u;
    const uint64_t few = L == 4 ? 512 : L == 8 ? 256 : 768;
    return L >= 12 || tiles < few ? 8u : 4u;
  }
  if (L == 10) return 5 * ((tiles + 511) / 512) < 3 * ((tiles + 255) / 256) ? 4u : 8u;
  const uint64_t few = L == 4 ? 900 : L == 6 ? 1100 : 1600;
  return L >= 12 || tiles < few ? 8u : 4u;
}
// The kernel form of a choice of 4 or 8.  Gaussian models, L <= 10: the kernel with
// its table in LDS, on several tiles or one.  Otherwise waves per workgroup; +-J on four waves
// packs several tiles per workgroup where there are enough of them (ms per
// launch packed / one tile per workgroup: L = 4, 313 tiles 0.044 / 0.047, 7813
// tiles 0.157 / 0.333; L = 6, 782 tiles 0.104 / 0.086, 1563 tiles 0.128 / 0.132,
// 7813 tiles 0.386 / 0.498; L = 8, 1563 tiles 0.240 / 0.219, 3125 tiles 0.384 /
// 0.382, 7813 tiles 0.824 / 0.873).
inline uint32_t sweep_form(uint32_t model, uint32_t L, uint32_t split, uint64_t tiles) {
  const uint64_t enough = L == 4 ? 0 : L == 6 ? 1500 : 3200;
  if (model != kModelPm) return L > 10 ? split : split == 4 ? kGaussLds : kGaussLdsOne;
  return split == 4 && L <= 8 && tiles >= enough ? kPmPacked : split;
}
// The form a launch uses: sweep_form of the choice set for (model, layout, L, size
// class of `tiles`) or measured there in this process (by sizes inside the class, see
// pa_tune.cpp), else of the default.
uint32_t sweep_split_for(uint32_t model, uint32_t layout, uint32_t L, uint64_t tiles);
// a choice measured at `tiles`, and one set for its size class
void sweep_split_record(uint32_t model, uint32_t layout, uint32_t L, uint64_t tiles,
                        uint32_t split);
void sweep_split_set(uint32_t model, uint32_t layout, uint32_t L, uint64_t tiles, uint32_t split);

// Spin layout of a population created with the library's choice, when the
// autotuner has not timed its shape: bit-packed (one bit per spin, 64
// replicas per word) for every shape; values are PA_LAYOUT_INT8 = 1 and
// PA_LAYOUT_BITPACK64 = 2.
inline uint32_t layout_default(uint32_t, uint32_t, uint64_t) { return 2u; }
// The autotuner's layout for (model, L, size class of `tiles`) when one was
// measured or pinned in this process, else layout_default (pa_tune.cpp).
uint32_t layout_for(uint32_t model, uint32_t L, uint64_t tiles);
void layout_record(uint32_t model, uint32_t L, uint64_t tiles, uint32_t layout);

}  // namespace pa
