// Host side of libones: argument validation, workspace layout, launch sequencing.
// The boundary is declared and documented in include/ones.h.
#include "ones.h"
#include "ones_device.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

// Scratch of ones_generation_static: one copy per GPU, held by every device that runs the
// library until the process ends.  Host code must not use this name as an address: the
// per-device address comes from hipGetSymbolAddress (static_scratch_of below).
static __device__ __align__(256) unsigned char scratch[ONES_STATIC_SCRATCH_BYTES];

namespace {

using namespace ones;

thread_local char g_hip_msg[256] = "HIP call failed";

int hip_fail(hipError_t e, const char *what) {
  snprintf(g_hip_msg, sizeof(g_hip_msg), "HIP call failed: %s: %s", what, hipGetErrorString(e));
  return ONES_E_HIP;
}
#define HIP_TRY(expr)                                         \
  do {                                                        \
    hipError_t e__ = (expr);                                  \
    if (e__ != hipSuccess) return hip_fail(e__, #expr);       \
  } while (0)

template <typename F>
int guarded(F &&body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc &) {
    snprintf(g_hip_msg, sizeof(g_hip_msg), "out of host memory");
  } catch (...) {
    snprintf(g_hip_msg, sizeof(g_hip_msg), "unexpected C++ exception");
  }
  return ONES_E_HIP;
}

size_t align_up(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

// Device address of the static scratch array on the current device, resolved once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
char *g_scratch_ptr[kMaxDevices];

int static_scratch_of(int device, char **out) {
  if (device < 0 || device >= kMaxDevices) {
    snprintf(g_hip_msg, sizeof(g_hip_msg), "device ordinal %d outside 0..%d", device, kMaxDevices - 1);
    return ONES_E_HIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    void *ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));   // for the device that is current
    g_scratch_ptr[device] = static_cast<char *>(ptr);
  }
  *out = g_scratch_ptr[device];
  return ONES_OK;
}

// Scratch of the selection: nothing in it outlives the generations of one ones_generation call
// except the splitters, the threshold and the cleared counter sets, which the next call may use
// (ctx->splitters_valid).  Offsets from the block's base, which lies in the caller's workspace
// or, for ones_generation_static, in the library's static array.
struct ScratchLayout {
  size_t split, split_slot, thresh, bcount[2], ties[2], bkeys, bidx, skeys, sidx, sbucket, total;
};

struct Layout {
  size_t genes, fit_row, slot_score, row_of, parent_row[2], spare, occupied[2], sel, fsync, xkeys, scratch, start, most, draws, lift, info[2], abl, cc, d, Y[kDrawRing], terms[kDrawRing];
  size_t export_err, export_sel, export_fit, unpacked, rY, alpha, beta, processed, time_rank, total;
  ScratchLayout S;
};

// Buckets of the selection: about 16 survivors each, at most kMaxBuckets.  A bucket stores eight
// times its fair share of the 3P/4 children and mutants (at least 256, a power of two); the
// surplus goes to a spill list that can hold a whole pool (the general selection drops every
// candidate).  The general selection re-divides the same bucket space among its own number of
// buckets.
struct BucketPlan { uint32_t nb, seg, spill; };
constexpr uint32_t kMinBucketPool = 256;
// Largest population whose selection ones_generation_static takes into the static array: the bound
// callers know (beyond it a bucket's storage doubles); its scratch is checked against the array too.
constexpr uint32_t kStaticMaxPopulation = 87380;
uint32_t pow2_at_least(uint32_t v) { uint32_t n = 1; while (n < v) n <<= 1; return n; }
BucketPlan bucket_plan(uint32_t P) {
  if (P < kMinBucketPool) return BucketPlan{0, 0, 0};      // tiny pools: one short sort is as fast
  const uint32_t K = P / 4;
  BucketPlan bp;
  bp.nb = std::min<uint32_t>(kMaxBuckets, std::max<uint32_t>(1, K / 16));
  bp.spill = P;                                            // the general selection may spill a whole pool
  bp.seg = std::min(pow2_at_least(std::max<uint32_t>(256, 8 * ((3 * K + bp.nb - 1) / bp.nb))), pow2_at_least(P) / 2);
  return bp;
}

// Pools whose generations run in one launch per ones_generation call (ones_fused.hip).  The
// launch is a cooperative one, which costs about 20 us where an ordinary launch costs 2.5, so
// calls of one or two generations are cheaper as two ordinary launches per generation.
constexpr int32_t kFusedMinGenerations = 3;
// The same for larger pools (ones_resident.hip).  What a call of four generations gains by one launch, up to 30 %, pays
// for that launch; under probability sampling, where the launched kernels rank a small pool by counting, only longer calls do,
// and a pool of 257 to 1024 on few rows of slots never (speed of calls of 4, 10, 16 and 30 generations against launched ones:
// pool 128 on 200 slots 0.93, 1.07, 1.15, 1.24; 260 0.84, 0.89, 0.90, 0.94, on 500 slots 0.93, 0.99, 1.01, 1.05;
// 1024 0.91, 0.99, 1.01, 1.05, on 500 slots 0.98, 1.06, 1.07, 1.10; 1500 0.99, 1.12, 1.18, 1.22; 4096 1.16 from 4 on; of calls
// of 6, 8, 10, 16 and 32: pool 64 on 100 slots 0.94, 0.99, 1.05, 1.13, 1.24, on 500 1.06, 1.12, 1.17, 1.26, 1.40;
// 192 0.91, 0.95, 0.98, 1.03, 1.10 and 0.96, 0.98, 1.02, 1.07, 1.14; 256 0.90, 0.92, 0.95, 0.99, 1.05 and 0.95, 0.97, 1.00, 1.04, 1.11).
// Where neither the table has changed nor draws are made, launched generations select through buckets, and four to six of
// a large pool on many slots are the faster ones (calls of 4, 6 and 10 generations, 16384 on 512 slots 0.90, 0.97, 1.36; 12000 on
// 512 0.93, 1.01, 1.36; 16384 on 200 1.17, 1.11, 1.25; 8192 on 512 1.05, 1.13, 1.48).
int32_t resident_min_generations(uint32_t P, uint32_t Jp, bool sampled, bool table_changed) {
  if (!sampled && !table_changed && P > 8192 && Jp > 4u * kLanes) return 8;
  if (!sampled || P > 2048) return 4;
  const bool many_rows = Jp > 4u * kLanes;
  if (P > 1024) return 6;
  if (P > 256) return many_rows ? 16 : INT32_MAX;
  if (P > 128) return many_rows ? 10 : 16;
  return many_rows ? 6 : 8;
}
// A search starts from random genomes, and while its pool is as mixed as that, many children beat the K-th survivor.
// Pools above 8192 are faster by generation then, the larger and the more slots the longer (16384 candidates on 512 slots, the
// first 50 generations: 1282 us, 1338 with one launch for those after the 28th, 1459 in one launch; two calls of 20 by
// generation and in one launch: 625 and 546 against 767 and 596; 12000 on 600 642 and 554, 773 and 638; 12000 on 200 488 and 437,
// 519 and 383; 9000 on 420 541 and 485, 531 and 403).  Smaller pools gain by one launch from the first generation on (8192:
// 1.1 for the first 20 on 1000 slots, 1.2 on 100), and those that would be launched for a few generations only as well.
int64_t resident_from(uint32_t P, uint32_t Jp) {
  const uint32_t n = P > 8192u ? 8 * (Jp / kLanes) * (P - 8192u) / 8192u : 0u;
  return n < 7 ? 0 : n;
}
// Of a call that begins earlier, so many generations have to come after that one: a launch behind queued ones waits for
// them, and 4 to 16 do not make up for it (a call of 20 that ends with four: 0.88 on 100 slots, with eight 0.94 on 200).
constexpr int32_t kResidentRest = 24;
// The same after a table in which `changed` of the n slots changed hands: the generations that its pool stays mixed.  Beyond
// four rows of slots, and from a sixth of them on (16384 candidates on 512 slots, two calls of 20 behind a table with new
// jobs on a sixth of them: 525 and 500 us by generation, 645 and 515 in one launch each; on a quarter 543 and 506, 713 and
// 545; on a half 707 and 525, 769 and 646).  An eighth gains as well (520 and 606 the first call), but a table whose jobs the
// pool has met before leaves it as settled as it was, and then one launch takes 323 of 431.  Behind one that changes more than
// a half, launched generations are crowded themselves (all 899 and 547, 787 and 695; 14000 on 700, three quarters, 50
// generations: 1661 and 1594), and one launch is the faster way for smaller pools, whose children the list holds (9000 on 420,
// a quarter: 481 and 442, 453 and 370), and on up to four rows (12000 on 200, three in ten: 428 and 570 against 384 and 392).
int64_t mixed_by(uint32_t P, uint32_t Jp, uint32_t changed, uint32_t n) {
  if (Jp <= 4u * kLanes || 6 * changed < n || 2 * changed > n) return 0;
  const int64_t mixed = resident_from(P, Jp) * 2 * changed / n;
  return mixed < 12 ? 0 : mixed;
}
bool fused_pool(uint32_t P, uint32_t Jp) { return Jp == static_cast<uint32_t>(kLanes) && P <= kFusedMaxPool; }
bool resident_pool(uint32_t P, uint32_t Jp) {
  return !fused_pool(P, Jp) && P <= static_cast<uint32_t>(kResidentMaxPool) && words_of(static_cast<int>(Jp / kLanes)) <= kResidentMaxWords;
}
size_t exchange_bytes(uint32_t P, uint32_t Jp) { return fused_pool(P, Jp) ? fused_exchange_bytes(P) : resident_pool(P, Jp) ? resident_exchange_bytes(P) : 0; }
int ring_places(uint32_t P, uint32_t Jp) { return resident_pool(P, Jp) ? kDrawRing : kDrawAhead; }

ScratchLayout make_scratch_layout(uint32_t P) {
  ScratchLayout S;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes); return at; };
  const BucketPlan bp = bucket_plan(P);
  S.split = take(kMaxBuckets * 8); S.split_slot = take(kMaxBuckets * 4); S.thresh = take(8);
  S.bcount[0] = take(kBucketCounters * 4); S.bcount[1] = take(kBucketCounters * 4);
  const size_t ties = bp.nb ? (static_cast<size_t>(kTieClasses) * tie_words(P / 4) + kTieMask) * 4 : 0;
  S.ties[0] = take(ties); S.ties[1] = take(ties);
  S.bkeys = take(static_cast<size_t>(bp.nb) * bp.seg * 8);
  S.bidx = take(static_cast<size_t>(bp.nb) * bp.seg * 4);
  S.skeys = take(static_cast<size_t>(bp.spill) * 8);
  S.sidx = take(static_cast<size_t>(bp.spill) * 4);
  S.sbucket = take(static_cast<size_t>(bp.spill) * 4);
  S.total = off;
  return S;
}

// Pool slots that ones_export unpacks at a time (16 MiB of batch sizes).
uint32_t unpack_slots(uint32_t P, uint32_t Jp) { return std::min<uint32_t>(P, (16u << 20) / (Jp * 4)); }

Layout make_layout(uint32_t P, uint32_t Jp) {
  Layout L;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes); return at; };
  const size_t rows = static_cast<size_t>(P) + P / 4;      // a pool of P slots lives in P + K physical rows
  const size_t row_bytes = static_cast<size_t>(words_of(Jp / kLanes)) * kLanes * 4;
  L.genes = take(rows * row_bytes);
  L.fit_row = take(rows * 8);
  L.slot_score = take(static_cast<size_t>(P) * 8);
  L.row_of = take(static_cast<size_t>(P) * 4);
  L.spare = take(static_cast<size_t>(P / 4) * 4);
  L.parent_row[0] = take(static_cast<size_t>(P / 4) * 4);
  L.parent_row[1] = take(static_cast<size_t>(P / 4) * 4);
  L.occupied[0] = take((rows + 31) / 32 * 4);     // bitmaps of the rows the survivors keep
  L.occupied[1] = take((rows + 31) / 32 * 4);
  L.sel = take(static_cast<size_t>(P / 4) * 4);
  // single-launch generations of small pools: error words, scores, ranks and draws exchanged
  L.fsync = take(256);
  L.xkeys = take(exchange_bytes(P, Jp));
  // the selection's scratch: splitters, counters, bucket storage, spill list
  L.S = make_scratch_layout(P);
  L.scratch = take(L.S.total);
  L.start = take(row_bytes); L.most = take(row_bytes); L.draws = take(row_bytes); L.lift = take(row_bytes);
  L.info[0] = take(Jp * 4); L.info[1] = take(Jp * 4);
  L.abl = take(Jp * 8); L.cc = take(Jp * 8); L.d = take(Jp * 8);
  // remaining work and the term table built from it, a ring of pairs at equal distances:
  // under probability sampling the draws of that many generations are made in one launch, and
  // generation g is scored with pair g mod their number
  for (int k = 0; k < ring_places(P, Jp); ++k) { L.Y[k] = take(Jp * 8); L.terms[k] = take(static_cast<size_t>(Jp) * kMaxTermEntries * 8); }
  // ones_export: error words, survivors, scores by slot and the batch sizes of a run of pool slots on their way
  // to the host, next to each other
  L.export_err = take(8); L.export_sel = take(static_cast<size_t>(P / 4) * 4); L.export_fit = take(static_cast<size_t>(P) * 8);
  L.unpacked = take(static_cast<size_t>(unpack_slots(P, Jp)) * Jp * 4);
  L.rY = take(Jp * 8);                            // the table's remaining work, for when sampling is switched off
  L.alpha = take(Jp * 8); L.beta = take(Jp * 8); L.processed = take(Jp * 8);
  L.time_rank = take(Jp * 4);
  L.total = off;
  return L;
}

// Host transfers go through one pinned staging buffer, which the kernels read and write themselves.  At its beginning lie the
// arrays of the call that runs: a job table, the parameters of the draws or the ranks of the executed times, as they lie
// in the workspace, or a placement.  Behind them HostWords and the winner's batch sizes and GPUs.
struct HostWords { uint32_t flag, winner, err[2]; double fit; };      // see HostSignal and WinnerOut
struct StageLayout { size_t rawinfo, a, c, d, Y, place_slot, place_batch, words, batch, gpus, total; };
// A state of up to so much is exported that way too, through a buffer of its own that the first export allocates (a larger one
// is copied).
constexpr size_t kStagedExport = 256u << 10;
size_t export_bytes(const Layout &L, uint32_t P, uint32_t Jp) { return L.unpacked + static_cast<size_t>(P) * Jp * 4 - L.export_err; }
StageLayout make_stage_layout(const Layout &L, uint32_t Jp, uint32_t G) {
  StageLayout S;
  size_t off = 0, end = 0;
  auto take = [&](size_t bytes) { size_t at = off; off = align_up(off + bytes); end = std::max(end, off); return at; };
  S.rawinfo = take(Jp * 4); S.a = take(Jp * 8); S.c = take(Jp * 8); S.d = take(Jp * 8); S.Y = take(Jp * 8);
  off = 0;
  S.place_slot = take(static_cast<size_t>(G) * 4); S.place_batch = take(static_cast<size_t>(G) * 4);
  off = 0;
  take(std::max(L.processed + static_cast<size_t>(Jp) * 8 - L.alpha, static_cast<size_t>(Jp) * 4));
  off = end;
  S.words = take(sizeof(HostWords)); S.batch = take(Jp * 4); S.gpus = take(Jp * 4);
  S.total = end;
  return S;
}

int check_config(const ones_config *cfg) {
  if (!cfg) return ONES_E_INVALID_ARG;
  if (cfg->n_gpus < 0 || cfg->n_gpus > ONES_MAX_GPUS) return ONES_E_INVALID_ARG;
  if (cfg->n_slots < 0 || cfg->n_slots > ONES_MAX_SLOTS) return ONES_E_INVALID_ARG;
  if (cfg->population <= 0 || cfg->population % 4 != 0 || cfg->population > ONES_MAX_POPULATION)
    return ONES_E_INVALID_ARG;
  if (!(cfg->mutation_rate >= 0.0 && cfg->mutation_rate <= 1.0)) return ONES_E_INVALID_ARG;
  if (!(cfg->crossover_rate >= 0.0 && cfg->crossover_rate <= 1.0)) return ONES_E_INVALID_ARG;
  return ONES_OK;
}

// A rate becomes a threshold on a uniform 32-bit word: min(2^32 - 1, floor(rate * 2^32)).
uint32_t rate_threshold(double rate) {
  const double v = std::floor(rate * 4294967296.0);
  return v >= 4294967295.0 ? 0xFFFFFFFFu : static_cast<uint32_t>(v);
}

int log2_pow2(int32_t v) {           // -1 unless v is a power of two
  if (v <= 0 || (v & (v - 1)) != 0) return -1;
  return 31 - __builtin_clz(static_cast<uint32_t>(v));
}

int check_param(double v) {
  if (!std::isfinite(v)) return ONES_E_NONFINITE;
  if (v < 0.0) return ONES_E_INVALID_ARG;
  if (v > ONES_MAX_PARAM) return ONES_E_BOUNDS;
  return ONES_OK;
}

struct HostJobs {                     // validated, padded staging copy of a job table
  std::vector<uint32_t> rawinfo;
  std::vector<double> a, c, d, Y;
  std::vector<int64_t> id;
  uint32_t term_E = 2;                // waiting + GPU-count codes up to the largest bmax / gpu_max_batch
  uint64_t demand = 0;                // GPUs that all jobs together take at their limits
};

int stage_jobs(int Jn, int Jp, const ones_jobs *jobs, HostJobs &h) {
  h.rawinfo.assign(Jp, 0u);
  h.a.assign(Jp, 0.0); h.c.assign(Jp, 0.0); h.d.assign(Jp, 0.0); h.Y.assign(Jp, 0.0);
  h.id.assign(Jp, 0);
  h.term_E = 2;
  h.demand = 0;
  if (Jn > 0 && (!jobs || !jobs->job_id || !jobs->active || !jobs->bmin || !jobs->bmax ||
                 !jobs->gpu_max_batch || !jobs->a || !jobs->c || !jobs->d || !jobs->remaining))
    return ONES_E_INVALID_ARG;
  for (int j = 0; j < Jn; ++j) {
    h.id[j] = jobs->job_id[j];
    if (!jobs->active[j]) continue;
    const int lo = log2_pow2(jobs->bmin[j]), hi = log2_pow2(jobs->bmax[j]);
    const int mu = log2_pow2(jobs->gpu_max_batch[j]);
    if (lo < 0 || hi < 0 || mu < 0) return ONES_E_NOT_POW2;
    if (lo > hi || hi > 30 || hi - mu > 20) return ONES_E_BOUNDS;
    int rc;
    if ((rc = check_param(jobs->a[j])) || (rc = check_param(jobs->c[j])) ||
        (rc = check_param(jobs->d[j])) || (rc = check_param(jobs->remaining[j])))
      return rc;
    h.rawinfo[j] = static_cast<uint32_t>(lo) | (static_cast<uint32_t>(hi) << 5) |
                   (static_cast<uint32_t>(mu) << 10) | (1u << 15);
    h.a[j] = jobs->a[j]; h.c[j] = jobs->c[j]; h.d[j] = jobs->d[j]; h.Y[j] = jobs->remaining[j];
    h.term_E = std::max<uint32_t>(h.term_E, static_cast<uint32_t>(std::max(0, hi - mu)) + 2);
    h.demand += 1u << std::max(0, hi - mu);
  }
  return ONES_OK;
}

struct EventPair { hipEvent_t start, stop; };

}  // namespace

struct ones_ctx {
  ones_config cfg;
  uint32_t P, K, Jn, Jp, R, G;
  uint32_t T_mut, T_x;
  hipStream_t stream;
  char *ws;
  char *stage;                // pinned host staging buffer, free between calls
  char *stage_dev;            // the same buffer as the device addresses it
  StageLayout S;
  char *export_stage, *export_stage_dev;    // the same for ones_export, once it is used (kStagedExport)
  uint32_t signals;           // HostSignal: the value of the last one
  uint32_t winner;            // the last generation's winner comes with this signal (a whole call in one launch), or 0: it does not
  Layout L;
  int cur;                    // the survivors of the current generation are in parent_row[cur ^ 1]
  int occ;                    // which bitmap holds the survivors' rows, unless
  bool rows_assigned;         // row_of and spare hold the rows of the next generation's slots
  int info_now, info_stored;  // which info array belongs to the job table, and to the one the genomes are stored under
  bool table_changed;         // job table replaced since the current generation was computed
  bool no_schedule;           // ... by ones_set_jobs: the winner is not a schedule under the new table
  bool new_jobs_first;        // option: the generation after ones_set_jobs serves the arrived jobs first
  bool sampling;              // remaining work drawn per generation (Alg. 1) instead of the table's
  int y_cur;                  // which remaining-work array and term table the last generation was scored with
  int64_t drawn_from, drawn_to;  // the ring holds the draws of generations [drawn_from, drawn_to) (equal: none)
  bool per_gpu;               // uniform crossover over the GPUs instead of the jobs (ones_set_crossover)
  bool has_times;             // executed times known (ones_set_processed_time): their ranks are on the device
  BucketPlan bp;              // nb == 0: pool small enough for the single-chunk sort
  int bucket_phase;           // which counter set the next bucketed generation fills
  int cleared_phase;          // a phase whose counters and bitmaps are cleared in the workspace's scratch
  bool splitters_valid;       // the workspace's selection scratch holds the splitters of the current survivors
                              // and cleared counter sets: a bucketed generation may follow
  bool poisoned;              // a launch failed in the middle of a generation: the state is inconsistent
  bool fused;                 // small pool: all generations of a call in one cooperative launch
  bool resident;              // ... the same for larger pools, as far as the job table leaves room (resident_plan)
  int64_t settled;            // ... from this generation on
  uint32_t fused_generations; // generations those launches have run so far
  uint32_t fused_changes;     // ... of them generations that also exchanged the survivors' scores
  uint32_t fused_draws;       // ... of them generations with a drawn remaining work
  uint32_t spin_limit;        // polls before a device-wide wait gives up
  int device;                 // the device the context was created on
  char *static_scratch;       // this device's copy of the library's static scratch array
  int n_cus;
  uint32_t term_E;            // entries per job of the term table
  uint64_t demand;            // GPUs that the table's jobs take at their limits
  int64_t t;                  // generation counter
  std::vector<int64_t> ids;   // job identity per slot, to detect slots that change hands
  // measurement
  bool profiling;
  int profile_every;          // bracket the kernels of every profile_every-th generation
  int64_t profile_tick;
  std::vector<EventPair> evolve_ev, select_ev;
  size_t evolve_used, select_used;

  template <typename T> T *at(size_t off) const { return reinterpret_cast<T *>(ws + off); }
  JobTable table(int which) const {     // with the remaining work and term table number `which`
    return JobTable{at<uint32_t>(L.start), at<uint32_t>(L.most), at<uint32_t>(L.draws), at<uint32_t>(L.lift),
                    at<uint32_t>(L.info[info_now]), at<uint32_t>(L.info[info_stored]), at<double>(L.abl), at<double>(L.cc), at<double>(L.d), at<double>(L.Y[which]),
                    at<double>(L.terms[which]), term_E};
  }
  JobTable table() const { return table(y_cur); }
  template <typename T> T *staged(size_t off) const { return reinterpret_cast<T *>(stage + off); }
  template <typename T> T *mapped(size_t off) const { return reinterpret_cast<T *>(stage_dev + off); }     // for kernels
  volatile HostWords *host_words() const { return staged<volatile HostWords>(S.words); }
  HostWords *host_words_dev() const { return mapped<HostWords>(S.words); }
};

namespace {

HostSignal next_signal(ones_ctx *c) {
  c->signals += 1;
  return HostSignal{c->at<uint32_t>(c->L.fsync) + 8, &c->host_words_dev()->flag, c->signals};
}
// For a launch that runs a whole call.
WinnerOut next_winner(ones_ctx *c) {
  HostWords *words = c->host_words_dev();
  return WinnerOut{c->mapped<int32_t>(c->S.batch), c->mapped<int32_t>(c->S.gpus), &words->fit, &words->winner, words->err, c->Jn, next_signal(c)};
}
// Waits for the last signal.  The poll leaves a longer wait to the runtime, which reports what goes wrong on the device.
// (The runtime clears up after launches as they come, and after the last some hundred when it is next asked to wait: 0.1 to 0.6 ms
// that ones_destroy or the next ones_init pays once.  Asked every 16 signals to, an epoch took 5 to 15 us more, every 64 2 to 4.)
constexpr std::chrono::milliseconds kPollTime(4);
using PollClock = std::chrono::steady_clock;
bool poll_signal(const ones_ctx *c, PollClock::time_point from) {
  do {
    for (int i = 0; i < 256; ++i) {
      if (c->host_words()->flag == c->signals) {
        std::atomic_thread_fence(std::memory_order_acquire);
        return true;
      }
      __builtin_ia32_pause();
    }
  } while (PollClock::now() - from < kPollTime);
  return false;
}
int wait_signal(ones_ctx *c) {
  if (!poll_signal(c, PollClock::now())) HIP_TRY(hipStreamSynchronize(c->stream));
  return ONES_OK;
}
// Waits for the whole stream where the last signal is that of an earlier call: what the caller has put behind that call's launch
// is waited for too, and an error of it returned.  Once the signal is there the stream is mostly done within 5 us, which
// hipStreamQuery tells for less than hipStreamSynchronize (an epoch of 64 candidates 87 us, 98; a kernel of its own that signals,
// as the calls that launch one anyway do, 95).  Behind an ordinary launch the query is the dearer one (55 against 40).
int wait_stream(ones_ctx *c) {
  const auto from = PollClock::now();
  hipError_t e = hipErrorNotReady;
  if (poll_signal(c, from)) {
    while ((e = hipStreamQuery(c->stream)) == hipErrorNotReady && PollClock::now() - from < kPollTime) __builtin_ia32_pause();
    if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();       // no error of this thread's
  }
  if (e != hipSuccess) HIP_TRY(hipStreamSynchronize(c->stream));
  return ONES_OK;
}

int upload_table(ones_ctx *c, const HostJobs &h) {
  const size_t n4 = static_cast<size_t>(c->Jp) * 4, n8 = static_cast<size_t>(c->Jp) * 8;
  const StageLayout &S = c->S;
  memcpy(c->stage + S.rawinfo, h.rawinfo.data(), n4);
  memcpy(c->stage + S.a, h.a.data(), n8);
  memcpy(c->stage + S.c, h.c.data(), n8);
  memcpy(c->stage + S.d, h.d.data(), n8);
  memcpy(c->stage + S.Y, h.Y.data(), n8);
  RawJobs raw{c->mapped<uint32_t>(S.rawinfo), c->mapped<double>(S.a), c->mapped<double>(S.c), c->mapped<double>(S.d), c->mapped<double>(S.Y)};
  c->term_E = h.term_E;
  c->demand = h.demand;
  HIP_TRY(launch_table_change(raw, c->table(), c->at<double>(c->L.rY), c->Jp, next_signal(c), c->stream));
  return wait_signal(c);                        // the staging buffer is free again
}

// `bytes` (a multiple of 16) of the staging buffer's beginning to the workspace.
int fetch_staged(ones_ctx *c, size_t to, size_t bytes) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != c->device) {    // a kernel needs the context's device to be current, a copy does not
    HIP_TRY(hipMemcpyAsync(c->ws + to, c->stage, bytes, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return ONES_OK;
  }
  const uint32_t n = static_cast<uint32_t>(bytes / 16);
  HIP_TRY(launch_fetch(c->stage_dev, c->ws + to, n, next_signal(c), c->stream));
  return wait_signal(c);                        // the staging buffer is free again
}

int timed(ones_ctx *c, std::vector<EventPair> &pool, size_t &used, bool begin) {
  if (!c->profiling || c->profile_tick % c->profile_every != 0) return ONES_OK;
  if (begin) {
    if (used == pool.size()) {
      EventPair e;
      HIP_TRY(hipEventCreate(&e.start));
      HIP_TRY(hipEventCreate(&e.stop));
      pool.push_back(e);
    }
    HIP_TRY(hipEventRecord(pool[used].start, c->stream));
  } else {
    HIP_TRY(hipEventRecord(pool[used].stop, c->stream));
    ++used;
  }
  return ONES_OK;
}

// Distance of two places of the ring of draws (make_layout), in doubles.
uint32_t ring_stride(const ones_ctx *c) { return static_cast<uint32_t>((c->L.Y[1] - c->L.Y[0]) / 8); }

// The ring holds the draws of `least` generations from t on, and, if they have to be made, those of up to `ahead`.
int make_draws(ones_ctx *c, uint32_t t, int least, int ahead) {
  if (c->drawn_from <= static_cast<int64_t>(t) && static_cast<int64_t>(t) + least <= c->drawn_to) return ONES_OK;
  const Progress pr{c->at<double>(c->L.alpha), c->at<double>(c->L.beta), c->at<double>(c->L.processed)};
  const uint32_t count = static_cast<uint32_t>(std::min<int64_t>(ahead, 0x100000000ll - static_cast<int64_t>(t)));
  HIP_TRY(launch_sample_remaining(pr, c->table(0), ring_stride(c), ring_places(c->P, c->Jp), c->Jn, c->Jp, static_cast<uint32_t>(c->cfg.seed),
                                  static_cast<uint32_t>(c->cfg.seed >> 32), t, count, c->stream));
  c->drawn_from = t;
  c->drawn_to = static_cast<int64_t>(t) + count;
  return ONES_OK;
}

// A launch that is being recorded into a graph must not need a resident grid.
bool capturing(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(s, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

// scratch: base of the selection's scratch block (the workspace's, or the static array);
// splitters_valid: that block holds the current survivors' splitters and cleared counters.
int run_generation(ones_ctx *c, uint32_t t, char *scratch, bool &splitters_valid, bool events) {
  EvolveArgs a;
  const ScratchLayout &S = c->L.S;
  auto sc = [&](size_t off) { return scratch + off; };
  const int next = t == 0 ? c->cur : c->cur ^ 1;
  a.genes = c->at<uint32_t>(c->L.genes);
  a.fit_row = c->at<double>(c->L.fit_row);
  a.parent_row = c->at<uint32_t>(c->L.parent_row[next]);
  a.row_of = c->at<uint32_t>(c->L.row_of);
  a.spare = c->at<uint32_t>(c->L.spare);
  a.occupied = c->at<uint32_t>(c->L.occupied[c->occ]);          // set by the last selection, unless it assigned the rows
  a.assigned = c->rows_assigned ? 1u : 0u;
  c->winner = 0;
  // Under probability sampling this generation is scored with its own place of the ring of
  // remaining-work arrays and term tables: a launch of an earlier generation has filled it
  // already, or the draws of this and the next generations are made now.
  const bool sampled = t != 0 && c->sampling;
  const int y_this = sampled ? static_cast<int>(t % ring_places(c->P, c->Jp)) : c->y_cur;
  a.tab = c->table(y_this);
  a.G = c->G; a.P = c->P; a.K = c->K; a.Jp = c->Jp;
  a.key0 = static_cast<uint32_t>(c->cfg.seed);
  a.key1 = static_cast<uint32_t>(c->cfg.seed >> 32);
  a.t = t; a.T_mut = c->T_mut; a.T_x = c->T_x;
  // same table: the survivors are fixed points of the repair.  Under probability sampling their
  // scores still change with every draw of the remaining work, so they are scored again.
  const bool same_table = t != 0 && !c->table_changed;
  a.rescore = same_table && sampled ? 1u : 0u;
  a.new_first = c->new_jobs_first && c->no_schedule ? 1u : 0u;   // the table's "arrived" marks are fresh
  a.per_gpu = c->per_gpu ? 1u : 0u;
  a.coin_stride = 0;                                             // the launcher sets it
  a.walk = walk_pays(c->Jp, c->G, c->demand, false) ? 1u : 0u;
  a.fault = c->at<uint32_t>(c->L.fsync) + 2;
  a.slot_score = c->at<double>(c->L.slot_score);
  a.time_rank = c->has_times ? c->at<uint32_t>(c->L.time_rank) : nullptr;
  // quantile buckets: only when the survivors reappear with the scores they had
  const bool buckets = same_table && !sampled && c->bp.nb != 0 && splitters_valid;
  a.occupied_other = buckets ? nullptr : c->at<uint32_t>(c->L.occupied[c->occ ^ 1]);
  a.bk.nb = buckets ? c->bp.nb : 0;
  a.bk.seg = c->bp.seg;
  a.bk.split = a.bk.split_next = reinterpret_cast<uint64_t *>(sc(S.split));
  a.bk.thresh = a.bk.thresh_next = reinterpret_cast<uint64_t *>(sc(S.thresh));
  a.bk.count = reinterpret_cast<uint32_t *>(sc(S.bcount[c->bucket_phase]));
  a.bk.keys = reinterpret_cast<uint64_t *>(sc(S.bkeys));
  a.bk.idx = reinterpret_cast<uint32_t *>(sc(S.bidx));
  a.bk.spill_keys = reinterpret_cast<uint64_t *>(sc(S.skeys));
  a.bk.spill_idx = reinterpret_cast<uint32_t *>(sc(S.sidx));
  a.bk.spill_bucket = reinterpret_cast<uint32_t *>(sc(S.sbucket));
  a.bk.split_slot = reinterpret_cast<uint32_t *>(sc(S.split_slot));
  a.bk.ties = reinterpret_cast<uint32_t *>(sc(S.ties[c->bucket_phase]));
  // the selection notes the rows the survivors keep, the next generation's parents
  RowPlan rp;
  rp.row_of = a.row_of;
  rp.parents = a.parent_row;
  rp.parent_next = c->at<uint32_t>(c->L.parent_row[next ^ 1]);
  rp.occupied = a.occupied_other;
  int rc;
  if (sampled && (rc = make_draws(c, t, 1, kDrawAhead))) return rc;
  if (events && (rc = timed(c, c->evolve_ev, c->evolve_used, true))) return rc;
  HIP_TRY(launch_evolve(a, static_cast<int>(c->R), same_table, c->n_cus, c->stream));
  if (events && (rc = timed(c, c->evolve_ev, c->evolve_used, false))) return rc;
  if (events && (rc = timed(c, c->select_ev, c->select_used, true))) return rc;
  if (buckets) {
    HIP_TRY(launch_bucket_select(a.fit_row, a.bk, rp, c->K,
                                 reinterpret_cast<uint32_t *>(sc(S.bcount[c->bucket_phase ^ 1])),
                                 reinterpret_cast<uint32_t *>(sc(S.ties[c->bucket_phase ^ 1])),
                                 c->at<int32_t>(c->L.sel), c->stream));
    c->bucket_phase ^= 1;
    if (scratch == c->ws + c->L.scratch) c->cleared_phase = c->bucket_phase;
  } else {
    BucketArgs store = a.bk;                       // same storage; always the first counter set
    store.nb = c->bp.nb;
    store.count = reinterpret_cast<uint32_t *>(sc(S.bcount[0]));
    // the launch scored the whole pool (initial population, refresh under a new table, survivors
    // scored again under a new draw): its scores by slot are complete
    const bool all_scored = t == 0 || !same_table || a.rescore != 0;
    HIP_TRY(launch_select(a.fit_row, all_scored ? a.slot_score : nullptr, rp, c->P, c->K, store,
                          c->at<int32_t>(c->L.sel), c->stream));
    splitters_valid = false;
    if (c->bp.nb != 0 && !sampled && same_table) {
      // Splitters for the bucketed generations that follow; clears both counter sets.  Under sampling
      // no bucketed generation can follow.  Nor after an initial population or a refresh under a new
      // table: the scores of such survivors say little about where their children will fall (nearly
      // all children of a random population beat its best members and would crowd into the first
      // bucket, more than a workgroup sorts in LDS), so the generation after it is ranked in full
      // once more and the buckets start from survivors that the search itself produced.
      HIP_TRY(launch_splitters(a.fit_row, a.row_of, c->at<int32_t>(c->L.sel), c->K, c->bp.nb,
                               reinterpret_cast<uint64_t *>(sc(S.split)), reinterpret_cast<uint64_t *>(sc(S.thresh)),
                               reinterpret_cast<uint32_t *>(sc(S.bcount[0])),
                               reinterpret_cast<uint32_t *>(sc(S.bcount[1])), reinterpret_cast<uint32_t *>(sc(S.ties[0])),
                               static_cast<uint32_t>((S.bkeys - S.ties[0]) / 4), c->stream));
      splitters_valid = true;
    }
  }
  if (events && (rc = timed(c, c->select_ev, c->select_used, false))) return rc;
  c->cur = next;
  c->rows_assigned = buckets;
  if (!buckets) c->occ ^= 1;
  c->y_cur = y_this;
  c->info_stored = c->info_now;     // every genome of the new pool was made under the current table
  c->table_changed = false;
  c->no_schedule = false;
  c->profile_tick += 1;
  return ONES_OK;
}

}  // namespace

extern "C" {

int32_t ones_padded_jobs(int32_t n_slots) {
  const int32_t n = n_slots < 1 ? 1 : n_slots;
  return kLanes * ((n + kLanes - 1) / kLanes);
}

size_t ones_workspace_bytes(const ones_config *cfg) {
  if (check_config(cfg) != ONES_OK) return 0;
  return make_layout(static_cast<uint32_t>(cfg->population), static_cast<uint32_t>(ones_padded_jobs(cfg->n_slots))).total;
}

static int init_impl(ones_ctx **out, const ones_config *cfg, const ones_jobs *jobs, void *d_workspace,
                     size_t workspace_bytes, void *hip_stream) {
  if (!out) return ONES_E_INVALID_ARG;
  int rc = check_config(cfg);
  if (rc) return rc;
  const int Jp = ones_padded_jobs(cfg->n_slots);
  HostJobs h;
  if ((rc = stage_jobs(cfg->n_slots, Jp, jobs, h))) return rc;
  const Layout L = make_layout(static_cast<uint32_t>(cfg->population), static_cast<uint32_t>(Jp));
  if (!d_workspace) return ONES_E_INVALID_ARG;
  if (workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(d_workspace) & 255u) != 0)
    return ONES_E_WORKSPACE_TOO_SMALL;
  std::unique_ptr<ones_ctx, void (*)(ones_ctx *)> owner(new ones_ctx(), ones_destroy);   // freed on every way out but the last
  ones_ctx *c = owner.get();
  c->cfg = *cfg;
  c->P = static_cast<uint32_t>(cfg->population); c->K = c->P / 4;
  c->Jn = static_cast<uint32_t>(cfg->n_slots); c->Jp = static_cast<uint32_t>(Jp); c->R = c->Jp / kLanes;
  c->G = static_cast<uint32_t>(cfg->n_gpus);
  c->T_mut = rate_threshold(cfg->mutation_rate);
  c->T_x = rate_threshold(cfg->crossover_rate);
  c->stream = static_cast<hipStream_t>(hip_stream);
  c->ws = static_cast<char *>(d_workspace);
  c->L = L;
  c->stage = nullptr;
  c->stage_dev = nullptr;
  c->export_stage = c->export_stage_dev = nullptr;
  {
    void *pinned = nullptr;
    c->S = make_stage_layout(L, c->Jp, c->G);
    HIP_TRY(hipHostMalloc(&pinned, c->S.total, hipHostMallocDefault));
    c->stage = static_cast<char *>(pinned);
    c->host_words()->flag = c->host_words()->winner = c->signals = c->winner = 0;
    void *mapped = nullptr;
    HIP_TRY(hipHostGetDevicePointer(&mapped, pinned, 0));
    c->stage_dev = static_cast<char *>(mapped);
  }
  c->cur = 0; c->t = 0;
  c->occ = 0;
  c->rows_assigned = false;
  c->info_now = c->info_stored = 0;
  c->table_changed = false;
  c->no_schedule = false;
  c->new_jobs_first = false;
  c->sampling = false;
  c->y_cur = 0;
  c->drawn_from = c->drawn_to = 0;
  c->has_times = false;
  c->per_gpu = false;
  c->bp = bucket_plan(c->P);
  c->bucket_phase = c->cleared_phase = 0;
  c->splitters_valid = false;
  c->poisoned = false;
  c->fused = c->resident = false;
  c->fused_generations = 0;
  c->fused_changes = 0;
  c->fused_draws = 0;
  c->spin_limit = 1u << 22;   // a few seconds of polling
  c->ids = h.id;
  {
    int dev = 0;
    hipDeviceProp_t prop;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipGetDeviceProperties(&prop, dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
    c->n_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    c->device = dev;
    c->static_scratch = nullptr;
    if ((rc = static_scratch_of(dev, &c->static_scratch))) return rc;
    // the single-launch path needs a launch whose workgroups are all resident at once
    c->fused = fused_pool(c->P, c->Jp) && prop.cooperativeLaunch != 0 &&
               fused_grid_limit(c->P) <= static_cast<uint32_t>(c->n_cus);
    c->resident = resident_pool(c->P, c->Jp) && prop.cooperativeLaunch != 0;
    c->settled = resident_from(c->P, c->Jp);
  }
  c->profiling = false; c->profile_every = 1; c->profile_tick = 0; c->evolve_used = c->select_used = 0;
  {
    const uint32_t words = (c->P + c->K + 31) / 32;
    hipError_t e = launch_zero_words(c->at<uint32_t>(c->L.occupied[0]), words, c->stream);
    if (e == hipSuccess) e = launch_zero_words(c->at<uint32_t>(c->L.occupied[1]), words, c->stream);
    if (e == hipSuccess) e = launch_zero_words(c->at<uint32_t>(c->L.fsync), 64, c->stream);
    const size_t exchange = exchange_bytes(c->P, c->Jp);
    if (e == hipSuccess && exchange != 0)   // the exchange buffers of the single-launch paths: every tag starts at 0
      e = launch_zero_words(c->at<uint32_t>(c->L.xkeys), static_cast<uint32_t>(exchange / 4), c->stream);
    if (e == hipSuccess && c->resident && c->bp.nb != 0)   // bitmaps of the buckets that may follow a launch of theirs
      e = launch_zero_words(c->at<uint32_t>(c->L.scratch + L.S.ties[0]), static_cast<uint32_t>((L.S.bkeys - L.S.ties[0]) / 4), c->stream);
    if (e != hipSuccess) return hip_fail(e, "launch_zero_words");
  }
  if ((rc = upload_table(c, h)) ||
      (rc = run_generation(c, 0, c->ws + c->L.scratch, c->splitters_valid, false)))
    return rc;
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  *out = owner.release();
  return ONES_OK;
}

static int set_jobs_impl(ones_ctx *c, const ones_jobs *jobs) {
  if (!c) return ONES_E_INVALID_ARG;
  HostJobs h;
  int rc = stage_jobs(static_cast<int>(c->Jn), static_cast<int>(c->Jp), jobs, h);
  if (rc) return rc;
  uint32_t changed = 0;
  for (uint32_t j = 0; j < c->Jn; ++j)
    if (h.id[j] != c->ids[j]) {                                  // the slot changed hands
      changed += 1;
      h.rawinfo[j] |= 1u << 17;
      if ((h.rawinfo[j] >> 15) & 1u) h.rawinfo[j] |= 1u << 16;   // an active job arrived in it
    }
  // the genomes stay as they are stored; info_stored says how to read them until the next generation
  c->info_now = c->info_stored ^ 1;
  if ((rc = upload_table(c, h))) return rc;
  c->ids = h.id;
  c->table_changed = true;
  c->no_schedule = true;
  c->winner = 0;
  c->settled = std::max(c->settled, c->t + mixed_by(c->P, c->Jp, changed, c->Jn));
  c->drawn_from = c->drawn_to = 0;   // the draws made ahead built their term tables from the old job table
  return ONES_OK;
}

static int set_progress_impl(ones_ctx *c, const double *alpha, const double *beta, const double *processed) {
  if (!c) return ONES_E_INVALID_ARG;
  if (!alpha && !beta && !processed) {
    if (c->sampling) {
      // back to the table's remaining work (still staged on the device); every score is stale
      HIP_TRY(hipMemcpyAsync(c->ws + c->L.Y[c->y_cur], c->ws + c->L.rY, static_cast<size_t>(c->Jp) * 8,
                             hipMemcpyDeviceToDevice, c->stream));
      HIP_TRY(launch_build_terms(c->table(), c->Jp, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      c->sampling = false;
      c->drawn_from = c->drawn_to = 0;
      c->table_changed = true;
    }
    return ONES_OK;
  }
  if (!alpha || !beta || !processed) return ONES_E_INVALID_ARG;
  for (uint32_t j = 0; j < c->Jn; ++j) {
    if (!std::isfinite(alpha[j]) || !std::isfinite(beta[j]) || !std::isfinite(processed[j])) return ONES_E_NONFINITE;
    if (alpha[j] < 1.0 || beta[j] < 1.0 || processed[j] < 0.0) return ONES_E_INVALID_ARG;
    if (alpha[j] > ONES_MAX_PARAM || beta[j] > ONES_MAX_PARAM || processed[j] > ONES_MAX_PARAM) return ONES_E_BOUNDS;
  }
  const Layout &L = c->L;
  double *ha = c->staged<double>(0), *hb = c->staged<double>(L.beta - L.alpha), *hp = c->staged<double>(L.processed - L.alpha);
  for (uint32_t j = 0; j < c->Jp; ++j) {
    const bool real = j < c->Jn;
    ha[j] = real ? alpha[j] : 1.0; hb[j] = real ? beta[j] : 1.0; hp[j] = real ? processed[j] : 0.0;
  }
  if (int rc = fetch_staged(c, L.alpha, L.processed + static_cast<size_t>(c->Jp) * 8 - L.alpha)) return rc;
  c->sampling = true;
  c->drawn_from = c->drawn_to = 0;   // the draws made ahead used the old parameters
  return ONES_OK;
}

static int set_new_jobs_first_impl(ones_ctx *c, int32_t on) {
  if (!c) return ONES_E_INVALID_ARG;
  c->new_jobs_first = on != 0;
  return ONES_OK;
}

static int set_crossover_impl(ones_ctx *c, int32_t mode) {
  if (!c || (mode != ONES_CROSSOVER_JOBS && mode != ONES_CROSSOVER_GPUS)) return ONES_E_INVALID_ARG;
  if (mode == ONES_CROSSOVER_GPUS && c->G > static_cast<uint32_t>(kMaxCoinGpus)) return ONES_E_BOUNDS;
  c->per_gpu = mode == ONES_CROSSOVER_GPUS;
  return ONES_OK;
}

static int set_processed_time_impl(ones_ctx *c, const double *t_processed) {
  if (!c) return ONES_E_INVALID_ARG;
  if (!t_processed) { c->has_times = false; return ONES_OK; }
  for (uint32_t j = 0; j < c->Jn; ++j) {
    int rc = check_param(t_processed[j]);
    if (rc) return rc;
  }
  // position of every slot in ascending (time, slot) order; the padding slots count as time 0
  std::vector<uint32_t> order(c->Jp);
  uint32_t *rank = c->staged<uint32_t>(0);
  for (uint32_t j = 0; j < c->Jp; ++j) order[j] = j;
  auto time_of = [&](uint32_t j) { return j < c->Jn ? t_processed[j] : 0.0; };
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return time_of(x) < time_of(y); });
  for (uint32_t pos = 0; pos < c->Jp; ++pos) rank[order[pos]] = pos;
  if (int rc = fetch_staged(c, c->L.time_rank, static_cast<size_t>(c->Jp) * 4)) return rc;
  c->has_times = true;
  return ONES_OK;
}

static int export_remaining_impl(ones_ctx *c, double *remaining_out) {
  if (!c || !remaining_out) return ONES_E_INVALID_ARG;
  HIP_TRY(hipStreamSynchronize(c->stream));
  if (c->Jn) HIP_TRY(hipMemcpy(remaining_out, c->ws + c->L.Y[c->y_cur], static_cast<size_t>(c->Jn) * 8, hipMemcpyDeviceToHost));
  return ONES_OK;
}

// The problem as the kernels of a whole call see it.
static EvolveArgs whole_call_args(const ones_ctx *c) {
  EvolveArgs a{};
  a.genes = c->at<uint32_t>(c->L.genes);
  a.fit_row = c->at<double>(c->L.fit_row);
  a.row_of = c->at<uint32_t>(c->L.row_of);
  a.spare = c->at<uint32_t>(c->L.spare);
  a.assigned = c->rows_assigned ? 1u : 0u;
  a.tab = c->table();
  a.G = c->G; a.P = c->P; a.K = c->K; a.Jp = c->Jp;
  a.key0 = static_cast<uint32_t>(c->cfg.seed);
  a.key1 = static_cast<uint32_t>(c->cfg.seed >> 32);
  a.t = static_cast<uint32_t>(c->t);
  a.T_mut = c->T_mut; a.T_x = c->T_x;
  a.new_first = c->new_jobs_first && c->no_schedule ? 1u : 0u;
  a.time_rank = c->has_times ? c->at<uint32_t>(c->L.time_rank) : nullptr;
  a.per_gpu = c->per_gpu ? 1u : 0u;
  a.walk = walk_pays(c->Jp, c->G, c->demand, true) ? 1u : 0u;
  a.fault = c->at<uint32_t>(c->L.fsync) + 2;
  return a;
}

// What run_fused and run_resident return when the runtime refuses the launch: nothing has run and no state has changed,
// and the kernels of one generation, which any GPU runs, take the call.
constexpr int kLaunchRefused = 1;
static int refused(ones_ctx *c, bool &whole_calls) {
  whole_calls = false;              // not asked for again by this context
  c->signals -= 1;                  // nor will the signal come
  (void)hipGetLastError();
  return kLaunchRefused;
}

// All n generations in one cooperative launch (small pools).
static int run_fused(ones_ctx *c, uint32_t n, bool events) {
  FusedArgs fa{};
  fa.ev = whole_call_args(c);
  fa.parent_rows = c->at<uint32_t>(c->L.parent_row[c->cur ^ 1]);
  fa.sel = c->at<int32_t>(c->L.sel);
  fused_exchange(c->at<uint64_t>(c->L.xkeys), c->P, fa);
  fa.changes_before = c->fused_changes;
  fa.draws_before = c->fused_draws;
  fa.sampled = c->sampling ? 1u : 0u;
  fa.pr = Progress{c->at<double>(c->L.alpha), c->at<double>(c->L.beta), c->at<double>(c->L.processed)};
  fa.n_slots = c->Jn;
  fa.y_out = c->at<double>(c->L.Y[c->y_cur]);      // what ones_export_remaining reads
  fa.sync = c->at<uint32_t>(c->L.fsync);
  fa.generations_before = c->fused_generations;
  fa.n_generations = n;
  fa.first_changed = c->table_changed ? 1u : 0u;
  fa.spin_limit = c->spin_limit;
  int rc;
  if (events && (rc = timed(c, c->evolve_ev, c->evolve_used, true))) return rc;
  fa.winner = next_winner(c);
  if (launch_fused(fa, c->stream) != hipSuccess) return refused(c, c->fused);
  if (events && (rc = timed(c, c->evolve_ev, c->evolve_used, false))) return rc;
  c->winner = capturing(c->stream) ? 0 : c->signals;   // (when a recorded launch will run is not known)
  c->fused_generations += n;
  c->fused_changes += c->sampling ? n : fa.first_changed;
  if (c->sampling) {
    c->fused_draws += n;
    c->drawn_from = c->drawn_to = 0;   // the ring may hold tables this launch wrote over (y_out); the two-launch path draws again
  }
  c->rows_assigned = true;
  c->info_stored = c->info_now;
  c->table_changed = false;
  c->no_schedule = false;
  c->splitters_valid = false;       // the two-launch path ranks the pool in full before it uses buckets again
  c->profile_tick += 1;
  return ONES_OK;
}

// The next n generations in one cooperative launch (pools beyond those of run_fused).  Under probability
// sampling n is at most kDrawRing, and their draws are in the ring.  Without, the launch leaves the survivors' splitters
// in the workspace's scratch for ones_generation, whichever entry point made it: it needs no scratch itself.
static int run_resident(ones_ctx *c, uint32_t n, const ResidentPlan &plan) {
  ResidentArgs ra{};
  ra.ev = whole_call_args(c);
  const ScratchLayout &S = c->L.S;
  char *scratch = c->ws + c->L.scratch;
  ra.n_buckets = c->sampling ? 0 : c->bp.nb;
  ra.split = reinterpret_cast<uint64_t *>(scratch + S.split);
  ra.thresh = reinterpret_cast<uint64_t *>(scratch + S.thresh);
  for (int set = 0; set < 2; ++set) ra.count[set] = reinterpret_cast<uint32_t *>(scratch + S.bcount[set]);
  ra.ev.coin_stride = plan.coin_stride;
  ra.ev.walk = plan.walk;
  ra.ev.term_lds = c->term_E;
  if (c->sampling) ra.ev.tab = c->table(static_cast<int>((c->t + 1) % kDrawRing));
  resident_exchange(c->at<uint64_t>(c->L.xkeys), c->P, ra);
  ra.parent_rows = c->at<uint32_t>(c->L.parent_row[c->cur ^ 1]);
  ra.sel = c->at<int32_t>(c->L.sel);
  ra.sync = c->at<uint32_t>(c->L.fsync);
  ra.generations_before = c->fused_generations;
  ra.sampled = c->sampling ? 1u : 0u;
  ra.ring_terms = c->at<double>(c->L.terms[0]);
  ra.ring_stride = ring_stride(c);
  ra.n_generations = n;
  ra.first_changed = c->table_changed ? 1u : 0u;
  ra.spin_limit = c->spin_limit;
  ra.paired = plan.paired; ra.unit_waves = plan.unit_waves; ra.child_items = plan.child_items;
  ra.segment = plan.segment; ra.list = plan.list; ra.table_lds = plan.table_lds;
  ra.winner = next_winner(c);
  hipError_t launched;
  switch (words_of(static_cast<int>(c->R))) {
    case 1: launched = launch_resident_words1(ra, plan, c->stream); break;
    case 2: launched = launch_resident_words2(ra, plan, c->stream); break;
    case 3: launched = launch_resident_words3(ra, plan, c->stream); break;
    default: launched = launch_resident_words4(ra, plan, c->stream); break;
  }
  if (launched != hipSuccess) return refused(c, c->resident);
  c->winner = c->signals;
  c->fused_generations += n;
  if (c->sampling) c->y_cur = static_cast<int>((c->t + n) % kDrawRing);
  c->rows_assigned = true;
  c->info_stored = c->info_now;
  c->table_changed = false;
  c->no_schedule = false;
  c->splitters_valid = ra.n_buckets != 0;
  c->bucket_phase = c->cleared_phase;       // (the launch clears both sets of counters, but no bitmaps)
  c->profile_tick += 1;
  return ONES_OK;
}

static int poisoned_error() {
  snprintf(g_hip_msg, sizeof(g_hip_msg), "an earlier launch failed in the middle of a generation; destroy the context");
  return ONES_E_HIP;
}

static int generation_impl(ones_ctx *c, int32_t n_generations, bool in_static_scratch) {
  if (!c || n_generations < 0) return ONES_E_INVALID_ARG;
  if (c->t + n_generations > 0xFFFFFFFFll) return ONES_E_INVALID_ARG;
  if (c->poisoned) return poisoned_error();
  char *block = c->ws + c->L.scratch;
  bool static_valid = false;      // the static array holds whatever the last call on this GPU left
  if (in_static_scratch) {
    if (c->P > kStaticMaxPopulation || c->L.S.total > ONES_STATIC_SCRATCH_BYTES) return ONES_E_STATIC_LIMIT;
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != c->device) return ONES_E_INVALID_ARG;
    block = c->static_scratch;
    if (n_generations > 0) c->splitters_valid = false;   // the workspace's splitters fall behind
  }
  if (c->fused && n_generations >= kFusedMinGenerations) {
    // uses no scratch at all: every workgroup ranks the pool in its LDS
    const int rc = run_fused(c, static_cast<uint32_t>(n_generations), !in_static_scratch);
    if (rc != kLaunchRefused) {
      if (rc) { c->poisoned = true; return rc; }
      c->t += n_generations;
      return ONES_OK;
    }
  }
  int32_t left = n_generations;
  bool &splitters_valid = in_static_scratch ? static_valid : c->splitters_valid;
  auto launched_generation = [&] {
    const int rc = run_generation(c, static_cast<uint32_t>(c->t + 1), block, splitters_valid, !in_static_scratch);
    if (rc) { c->poisoned = true; return rc; }
    c->t += 1;
    left -= 1;
    return static_cast<int>(ONES_OK);
  };
  ResidentPlan plan;
  const int32_t least = resident_min_generations(c->P, c->Jp, c->sampling, c->table_changed);
  const bool by_kernel = c->profiling && !in_static_scratch;       // the measurement hook sees evolve and select launches
  if (c->resident && left >= least && !by_kernel && resident_plan(whole_call_args(c), c->sampling, c->n_cus, plan) &&
      !capturing(c->stream)) {
    if (!c->sampling && c->t < c->settled) {
      const int64_t rest = c->t + left - c->settled;
      while (left > (rest < kResidentRest ? 0 : rest))
        if (const int rc = launched_generation()) return rc;
    }
    while (left >= least) {
      int32_t n = left;
      if (c->sampling) {
        // a launch takes as many generations as the ring has places: where an earlier call left fewer draws they are made
        // again, a small launch, so that how a call is run depends on the call only (30 generations of 4096 candidates on
        // 200 slots after five calls of one: 560 us, where the three draws that those leave had them all launched 904)
        const int32_t draws = std::min<int32_t>(left, kDrawRing);
        const int rc = make_draws(c, static_cast<uint32_t>(c->t + 1), draws, draws);
        if (rc) { c->poisoned = true; return rc; }
        n = static_cast<int32_t>(std::min<int64_t>(left, c->drawn_to - (c->t + 1)));
        if (n < least) break;
      }
      const int rc = run_resident(c, static_cast<uint32_t>(n), plan);
      if (rc == kLaunchRefused) break;
      if (rc) { c->poisoned = true; return rc; }
      c->t += n;
      left -= n;
    }
  }
  while (left > 0)
    if (const int rc = launched_generation()) return rc;
  return ONES_OK;
}

// A device-wide wait of a single-launch generation gave up (it never does on a healthy device):
// the population is inconsistent from then on.
static int wait_gave_up(ones_ctx *c) {
  c->poisoned = true;
  snprintf(g_hip_msg, sizeof(g_hip_msg), "a device-wide wait inside the generation kernel gave up; destroy the context");
  return ONES_E_HIP;
}

// A kernel had to pull a row index back into the genome array: the row bookkeeping is wrong
// (a defect of the library, never of the caller's input).
static int row_fault(ones_ctx *c) {
  c->poisoned = true;
  snprintf(g_hip_msg, sizeof(g_hip_msg), "internal error: a genome row index was out of range; destroy the context");
  return ONES_E_HIP;
}

// Rows of the current generation's survivors, best first.
static const uint32_t *survivor_rows(const ones_ctx *c) { return c->at<uint32_t>(c->L.parent_row[c->cur ^ 1]); }

// What a kernel found wrong, once its error words are there.
static int check_error_words(ones_ctx *c) {
  if (c->host_words()->err[0]) return wait_gave_up(c);
  return c->host_words()->err[1] ? row_fault(c) : ONES_OK;
}

static int best_impl(ones_ctx *c, int32_t *batch_out, int32_t *gpus_out, double *fitness_out) {
  if (!c) return ONES_E_INVALID_ARG;
  if (c->poisoned) return poisoned_error();
  HostWords *words = c->host_words_dev();
  bool there = false;
  if (c->winner != 0 && c->winner == c->signals) {
    // the launch that ran the last call, which is this context's last one, leaves the winner in the pinned buffer
    if (int rc = wait_stream(c)) return rc;
    there = c->host_words()->winner == c->winner;
    if (!there) c->winner = 0;      // it has given up
  }
  if (!there) {
    // one launch and one wait, no copy (a few hundred bytes to a few kilobytes)
    HIP_TRY(launch_best(c->at<uint32_t>(c->L.genes), c->at<double>(c->L.fit_row), survivor_rows(c), c->at<uint32_t>(c->L.info[c->info_stored]),
                        c->at<uint32_t>(c->L.info[c->info_now]), c->Jn, c->Jp, c->mapped<int32_t>(c->S.batch), c->mapped<int32_t>(c->S.gpus),
                        &words->fit, c->at<uint32_t>(c->L.fsync) + 1, words->err, next_signal(c), c->stream));
    if (int rc = wait_signal(c)) return rc;
  }
  if (int rc = check_error_words(c)) return rc;
  if (batch_out && c->Jn) memcpy(batch_out, c->stage + c->S.batch, c->Jn * 4);
  if (gpus_out && c->Jn) memcpy(gpus_out, c->stage + c->S.gpus, c->Jn * 4);
  if (fitness_out) *fitness_out = c->host_words()->fit;
  return ONES_OK;
}

static int placement_impl(ones_ctx *c, int32_t *slot_of_gpu, int32_t *batch_of_gpu) {
  if (!c || c->no_schedule) return ONES_E_INVALID_ARG;
  if (c->poisoned) return poisoned_error();
  const size_t n4 = static_cast<size_t>(c->G) * 4;
  HIP_TRY(launch_placement(c->at<uint32_t>(c->L.genes), survivor_rows(c), c->at<uint32_t>(c->L.info[c->info_now]), c->Jn, c->Jp, c->G,
                           c->mapped<int32_t>(c->S.place_slot), c->mapped<int32_t>(c->S.place_batch), c->at<uint32_t>(c->L.fsync) + 1,
                           c->host_words_dev()->err, next_signal(c), c->stream));
  if (int rc = wait_signal(c)) return rc;
  if (int rc = check_error_words(c)) return rc;
  if (slot_of_gpu && c->G) memcpy(slot_of_gpu, c->stage + c->S.place_slot, n4);
  if (batch_of_gpu && c->G) memcpy(batch_of_gpu, c->stage + c->S.place_batch, n4);
  return ONES_OK;
}

// A state of up to this size comes to the host in one copy (each costs about 10 us), through a buffer; of up to kStagedExport
// without any.
constexpr size_t kOneCopyExport = 1u << 20;

static int export_impl(ones_ctx *c, int32_t *genes, double *fit, int32_t *sel, int64_t *generation) {
  if (!c) return ONES_E_INVALID_ARG;
  if (c->poisoned) { HIP_TRY(hipStreamSynchronize(c->stream)); return poisoned_error(); }
  // candidates live in physical rows, their genes as codes: the device puts scores and genomes in slot order
  const Layout &L = c->L;
  ExportArgs x{c->at<uint32_t>(L.genes), c->at<double>(L.fit_row), c->at<uint32_t>(L.row_of), c->at<int32_t>(L.sel),
                     survivor_rows(c), c->at<uint32_t>(L.info[c->info_stored]), c->at<uint32_t>(L.fsync) + 1, c->P, c->K, c->Jp,
                     c->at<double>(L.export_fit), c->at<int32_t>(L.export_sel), c->at<uint32_t>(L.export_err),
                     c->at<int32_t>(L.unpacked), HostSignal{}};
  const size_t fit_bytes = static_cast<size_t>(c->P) * 8, sel_bytes = static_cast<size_t>(c->K) * 4;
  const size_t row_bytes = static_cast<size_t>(c->Jp) * 4, genes_bytes = c->P * row_bytes;
  const uint32_t most = unpack_slots(c->P, c->Jp);
  const size_t all_bytes = genes ? L.unpacked + genes_bytes - L.export_err : L.export_fit + fit_bytes - L.export_err;
  const bool one_copy = all_bytes <= kOneCopyExport && most == c->P;
  bool staged = genes && export_bytes(L, c->P, c->Jp) <= kStagedExport;
  if (staged && !c->export_stage) {
    void *pinned = nullptr, *dev = nullptr;
    staged = hipHostMalloc(&pinned, export_bytes(L, c->P, c->Jp), hipHostMallocDefault) == hipSuccess;
    if (staged && hipHostGetDevicePointer(&dev, pinned, 0) != hipSuccess) { (void)hipHostFree(pinned); staged = false; }
    if (staged) { c->export_stage = static_cast<char *>(pinned); c->export_stage_dev = static_cast<char *>(dev); }
    else (void)hipGetLastError();                     // copied, then
  }
  const size_t head_bytes = one_copy ? all_bytes : L.export_sel + sel_bytes - L.export_err;
  std::unique_ptr<char[]> copied;
  const char *head = c->export_stage;
  if (staged) {
    auto mapped = [&](size_t off) { return c->export_stage_dev + (off - L.export_err); };
    x.fit_out = reinterpret_cast<double *>(mapped(L.export_fit));
    x.sel_out = reinterpret_cast<int32_t *>(mapped(L.export_sel));
    x.err_out = reinterpret_cast<uint32_t *>(mapped(L.export_err));
    x.genes_out = reinterpret_cast<int32_t *>(mapped(L.unpacked));
    x.done = next_signal(c);
    HIP_TRY(launch_export_genes(x, 0, c->P, true, c->stream));
    if (int rc = wait_signal(c)) return rc;
  } else {
    if (genes && one_copy) HIP_TRY(launch_export_genes(x, 0, c->P, true, c->stream));
    else HIP_TRY(launch_export_scores(x, c->stream));
    copied.reset(new char[head_bytes]);
    head = copied.get();
    HIP_TRY(hipMemcpyAsync(copied.get(), c->ws + L.export_err, head_bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  auto fetched = [&](size_t off) { return head + (off - L.export_err); };
  uint32_t words[2] = {0, 0};
  memcpy(words, fetched(L.export_err), 8);
  if (words[0]) return wait_gave_up(c);
  if (words[1]) return row_fault(c);
  if (sel) memcpy(sel, fetched(L.export_sel), sel_bytes);
  if (one_copy) {
    if (fit) memcpy(fit, fetched(L.export_fit), fit_bytes);
    if (genes) memcpy(genes, fetched(L.unpacked), genes_bytes);
  } else {
    if (fit) HIP_TRY(hipMemcpy(fit, c->ws + L.export_fit, fit_bytes, hipMemcpyDeviceToHost));
    for (uint32_t first = 0; genes && first < c->P; first += most) {
      const uint32_t count = std::min(most, c->P - first);
      HIP_TRY(launch_export_genes(x, first, count, false, c->stream));
      HIP_TRY(hipMemcpyAsync(genes + static_cast<size_t>(first) * c->Jp, c->ws + L.unpacked, count * row_bytes,
                             hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
    }
  }
  if (generation) *generation = c->t;
  return ONES_OK;
}

static int profile_enable_impl(ones_ctx *c, int32_t on) {
  if (!c) return ONES_E_INVALID_ARG;
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->profiling = on > 0;
  c->profile_every = on > 0 ? on : 1;
  c->profile_tick = 0;
  c->evolve_used = c->select_used = 0;
  return ONES_OK;
}

static int profile_read_impl(ones_ctx *c, double *evolve_ms, int64_t *evolve_launches, double *select_ms,
                      int64_t *select_launches) {
  if (!c) return ONES_E_INVALID_ARG;
  HIP_TRY(hipStreamSynchronize(c->stream));
  double em = 0.0, sm = 0.0;
  for (size_t i = 0; i < c->evolve_used; ++i) {
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, c->evolve_ev[i].start, c->evolve_ev[i].stop));
    em += ms;
  }
  for (size_t i = 0; i < c->select_used; ++i) {
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, c->select_ev[i].start, c->select_ev[i].stop));
    sm += ms;
  }
  if (evolve_ms) *evolve_ms = em;
  if (evolve_launches) *evolve_launches = static_cast<int64_t>(c->evolve_used);
  if (select_ms) *select_ms = sm;
  if (select_launches) *select_launches = static_cast<int64_t>(c->select_used);
  return ONES_OK;
}

static int update_limits_impl(int32_t n_slots, const ones_limit_inputs *in, double sigma, int32_t *limit) {
  if (n_slots < 0 || n_slots > ONES_MAX_SLOTS) return ONES_E_INVALID_ARG;
  if (n_slots > 0 && (!in || !limit || !in->state || !in->bmin || !in->bcap || !in->gpu_max_batch ||
                      !in->last_batch || !in->finished_epoch || !in->elapsed))
    return ONES_E_INVALID_ARG;
  if (!std::isfinite(sigma)) return ONES_E_NONFINITE;
  if (sigma < 0.0) return ONES_E_INVALID_ARG;
  std::vector<int32_t> next(static_cast<size_t>(n_slots), 0);
  for (int32_t j = 0; j < n_slots; ++j) {
    const uint8_t state = in->state[j];
    if (state > 3) return ONES_E_INVALID_ARG;
    if (state == 0) continue;
    if (log2_pow2(in->bmin[j]) < 0 || log2_pow2(in->bcap[j]) < 0 || log2_pow2(in->gpu_max_batch[j]) < 0)
      return ONES_E_NOT_POW2;
    if (in->bmin[j] > in->bcap[j] || in->bcap[j] > (1 << 30)) return ONES_E_BOUNDS;
    int64_t r = limit[j];
    if (state == 1) {                              // Start
      r = in->gpu_max_batch[j];
    } else {
      if (r < 1) return ONES_E_INVALID_ARG;
      if (state == 2) {                            // Resume
        if (in->last_batch[j] < 0) return ONES_E_INVALID_ARG;
        r = in->last_batch[j] > 0 ? std::min<int64_t>(r, in->last_batch[j]) : r / 2;
      } else {                                     // Scale-up with the Scale-down penalty
        const double T = in->elapsed[j];
        if (!std::isfinite(T)) return ONES_E_NONFINITE;
        if (T < 0.0) return ONES_E_INVALID_ARG;
        if (sigma * T > 1e15) return ONES_E_BOUNDS;
        if (in->finished_epoch[j]) {
          const int64_t penalty = static_cast<int64_t>(std::ceil(sigma * T + 1.0));
          r = (2 * r + penalty - 1) / penalty;
        }
      }
    }
    r = std::min<int64_t>(std::max<int64_t>(r, in->bmin[j]), in->bcap[j]);
    next[j] = 1 << (63 - __builtin_clzll(static_cast<unsigned long long>(r)));   // largest power of two <= r
  }
  if (n_slots) memcpy(limit, next.data(), static_cast<size_t>(n_slots) * 4);
  return ONES_OK;
}

// The entry points proper: nothing is thrown across the C boundary (the staging vectors may run out of host
// memory).

int ones_init(ones_ctx **out, const ones_config *cfg, const ones_jobs *jobs, void *d_workspace, size_t workspace_bytes, void *hip_stream) {
  return guarded([&] { return init_impl(out, cfg, jobs, d_workspace, workspace_bytes, hip_stream); });
}

int ones_set_jobs(ones_ctx *c, const ones_jobs *jobs) {
  return guarded([&] { return set_jobs_impl(c, jobs); });
}

int ones_set_crossover(ones_ctx *c, int32_t mode) {
  return guarded([&] { return set_crossover_impl(c, mode); });
}

int ones_set_processed_time(ones_ctx *c, const double *t_processed) {
  return guarded([&] { return set_processed_time_impl(c, t_processed); });
}

int ones_set_progress(ones_ctx *c, const double *alpha, const double *beta, const double *processed) {
  return guarded([&] { return set_progress_impl(c, alpha, beta, processed); });
}

int ones_set_new_jobs_first(ones_ctx *c, int32_t on) {
  return guarded([&] { return set_new_jobs_first_impl(c, on); });
}

int ones_export_remaining(ones_ctx *c, double *remaining_out) {
  return guarded([&] { return export_remaining_impl(c, remaining_out); });
}

int ones_generation(ones_ctx *c, int32_t n_generations) {
  return guarded([&] { return generation_impl(c, n_generations, false); });
}

int ones_set_wait_limit(ones_ctx *c, uint32_t polls) {
  if (!c) return ONES_E_INVALID_ARG;
  c->spin_limit = polls;
  return ONES_OK;
}

int ones_generation_static(ones_ctx *c, int32_t n_generations) {
  return guarded([&] { return generation_impl(c, n_generations, true); });
}

int ones_best(ones_ctx *c, int32_t *batch_out, int32_t *gpus_out, double *fitness_out) {
  return guarded([&] { return best_impl(c, batch_out, gpus_out, fitness_out); });
}

int ones_placement(ones_ctx *c, int32_t *slot_of_gpu, int32_t *batch_of_gpu) {
  return guarded([&] { return placement_impl(c, slot_of_gpu, batch_of_gpu); });
}

int ones_export(ones_ctx *c, int32_t *genes, double *fit, int32_t *sel, int64_t *generation) {
  return guarded([&] { return export_impl(c, genes, fit, sel, generation); });
}

int ones_profile_enable(ones_ctx *c, int32_t on) {
  return guarded([&] { return profile_enable_impl(c, on); });
}

int ones_profile_read(ones_ctx *c, double *evolve_ms, int64_t *evolve_launches, double *select_ms, int64_t *select_launches) {
  return guarded([&] { return profile_read_impl(c, evolve_ms, evolve_launches, select_ms, select_launches); });
}

int ones_update_limits(int32_t n_slots, const ones_limit_inputs *in, double sigma, int32_t *limit) {
  return guarded([&] { return update_limits_impl(n_slots, in, sigma, limit); });
}

void ones_destroy(ones_ctx *c) {
  if (!c) return;
  // A launch of ones_generation that no call has waited for still writes the winner to the pinned buffer.  (Not on a stream that is
  // being captured: that would end the capture, and what is recorded writes nothing before it is launched.)
  if (c->stage && c->host_words()->flag != c->signals && !capturing(c->stream)) (void)hipStreamSynchronize(c->stream);
  for (auto &e : c->evolve_ev) { (void)hipEventDestroy(e.start); (void)hipEventDestroy(e.stop); }
  for (auto &e : c->select_ev) { (void)hipEventDestroy(e.start); (void)hipEventDestroy(e.stop); }
  if (c->stage) (void)hipHostFree(c->stage);
  if (c->export_stage) (void)hipHostFree(c->export_stage);
  delete c;
}

const char *ones_strerror(int code) {
  switch (code) {
    case ONES_OK: return "ok";
    case ONES_E_INVALID_ARG: return "invalid argument";
    case ONES_E_NOT_POW2: return "bmin, bmax and gpu_max_batch of an active slot must be powers of two";
    case ONES_E_BOUNDS: return "batch window or model parameter out of bounds";
    case ONES_E_NONFINITE: return "NaN or infinity in a job parameter";
    case ONES_E_WORKSPACE_TOO_SMALL: return "workspace too small or not 256-byte aligned";
    case ONES_E_HIP: return g_hip_msg;
    case ONES_E_STATIC_LIMIT: return "population too large for the static scratch of ones_generation_static";
    default: return "unknown error code";
  }
}

}  // extern "C"

