// Internal interface between the host side of libones (ones_api.hip) and its kernels
// (ones_evolve.hip, ones_select.hip, ones_sample.hip).  Not installed; the public boundary is include/ones.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ones {

constexpr int kLanes = 64;          // one candidate schedule per wave64, job columns across lanes
constexpr int kMaxRows = 32;        // 2048 job slots / 64 columns
constexpr int kMaxTermEntries = 22; // waiting + GPU counts 2^0 .. 2^20
constexpr int kMaxCoinGpus = 8192;  // crossover over the GPUs: one Philox block of 128 coins per lane
#ifndef ONES_SORT_CHUNK
#define ONES_SORT_CHUNK 4096
#endif
constexpr int kSortChunk = ONES_SORT_CHUNK;   // largest pool that one workgroup sorts in LDS

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
struct Words { uint32_t w[4]; };

__device__ __forceinline__ Words philox4x32_10(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t pa = static_cast<uint64_t>(x0) * 0xD2511F53ull;
    const uint64_t pb = static_cast<uint64_t>(x2) * 0xCD9E8D57ull;
    // three-input xor in one instruction (truth table 0x96)
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), x1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), x3, k1, 0x96);
    x1 = static_cast<uint32_t>(pb);
    x3 = static_cast<uint32_t>(pa);
    x0 = n0;
    x2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Words{{x0, x1, x2, x3}};
}

// Genomes.  A gene is a byte: the code of the job's GPU count, 0 = the job waits, e + 1 = it runs on
// 2^e GPUs (at most 2^20).  After the free lift to the per-GPU max batch a running job's global batch
// is B = GPUs << bl_exp with bl_exp a property of its slot in the job table, so the code says it
// all, for the table the genome was made under.  A genome row is Q * 64 words, Q = ceil(rows / 4):
// job slot j lies in column (lane) j mod 64 and row i = j div 64, at byte i mod 4 of word
// (i div 4) * 64 + lane; the bytes of rows beyond the job slots are 0.
constexpr int words_of(int rows) { return (rows + 3) / 4; }          // Q
__host__ __device__ inline uint32_t gene_byte(uint32_t j) { return ((j / 64 / 4) * 64 + j % 64) * 4 + j / 64 % 4; }
__host__ __device__ inline uint32_t batch_of_code(uint32_t code, uint32_t bl_exp) { return ((1u << code) >> 1) << bl_exp; }

// Per-slot constants derived from the job table, over the padded slots.
struct JobTable {
  // laid out like a genome row, a byte per slot: code a waiting job resumes with and code at the
  // batch-size limit R_j (0 for an empty slot), number of outcomes of a redraw (hi - lo + 2; 0 for an
  // empty slot), outcomes 1 .. lift of which give the former
  uint32_t *start, *most, *draws, *lift;
  uint32_t *info;     // bits 0-4 lo, 5-10 (hi-lo+2), 11-15 mu, 16-20 bl_exp, 21 active, 22 arrived with this table
  // info of the table the genomes are stored under: this one, or, between ones_set_jobs and the next
  // generation, an earlier one, where bit 23 marks the slots that have changed hands since (they wait)
  uint32_t *stored;
  double   *abl;      // a * 2^bl_exp: compute time of one iteration at the local batch
  double   *cc;       // synchronisation cost per doubling of the GPU count
  double   *d;        // fixed cost per iteration
  double   *Y;        // remaining samples
  // term table: T_j c_j of slot (row, lane) running on 2^(e-1) GPUs at [(row*term_E + e)*64 + lane],
  // e = 0 (waiting, +0.0) .. term_E-1; the value the score formula gives, precomputed per table
  double   *terms;
  uint32_t  term_E;
};

__host__ __device__ inline uint32_t info_lo(uint32_t w)     { return w & 31u; }
__host__ __device__ inline uint32_t info_n(uint32_t w)      { return (w >> 5) & 63u; }
__host__ __device__ inline uint32_t info_mu(uint32_t w)     { return (w >> 11) & 31u; }
__host__ __device__ inline uint32_t info_blexp(uint32_t w)  { return (w >> 16) & 31u; }
__host__ __device__ inline uint32_t info_active(uint32_t w) { return (w >> 21) & 1u; }
__host__ __device__ inline uint32_t info_new(uint32_t w)    { return (w >> 22) & 1u; }
__host__ __device__ inline uint32_t info_reset(uint32_t w)  { return (w >> 23) & 1u; }
constexpr uint32_t kInfoReset = 1u << 23;

// Quantile buckets of the selection (valid while the job table stays the same): children and
// mutants that beat the K-th survivor are dropped into the bucket of the survivors they fall
// between.  nb == 0 switches the mechanism off.  A bucket stores up to seg offspring; the rare
// surplus goes to one shared spill list.
constexpr int kMaxBuckets = 1024;
constexpr int kSpillCounter = kMaxBuckets;       // count[kSpillCounter]: records in the spill list
constexpr int kManyFlag = kMaxBuckets + 1;       // count[kManyFlag]: a bucket was given more than kManyInBucket records
// Copies.  A pool that has been searched for a while fills with copies of one genome, or of a few, and then most children that
// beat the K-th survivor have exactly the score of many survivors.  Such a child of a class of survivors that takes up kTieRun
// splitters in a row is not stored: its slot is marked in the class's bitmap, and its rank follows from the number of
// marks before its own.  Class c's last splitter lies among splitters [c * kTieRun, (c + 1) * kTieRun), so there are at most
// kTieClasses of them and no two share a bitmap.  count[kTieCount + c]: its children; count[kTieBucket + c]: the bucket
// they would be in, of which they are the first offspring.
// (A bucket's counter takes 9 ns per child: on the stress workload, where up to 28000 children share one score while a better genome
// takes the pool over, the kernel of such a generation took up to 390 us, and the selection 127 in the median of those generations,
// 270 at most.  Now 71 and 19, 61 at most, and other generations take the 0.3 us longer that the look for the flag costs; runs of
// 16 splitters leave classes of up to 1500 children to the buckets, and 26 us.)
constexpr int kTieRun = 8, kTieClasses = kMaxBuckets / kTieRun;
constexpr int kTieFlag = kMaxBuckets + 2;        // count[kTieFlag]: there is such a child
constexpr int kTieCount = kTieFlag + 1, kTieBucket = kTieCount + kTieClasses;
static_assert(kTieClasses == 2 * kLanes, "two classes to a lane");
constexpr int kBucketCounters = kTieBucket + kTieClasses;
constexpr uint32_t kTieMask = kTieClasses / 32;      // words of the classes' bits
__host__ __device__ inline uint32_t tie_words(uint32_t K) { return (3 * K + 31) / 32; }     // of a class's bitmap, over the slots from K on
constexpr uint32_t kManyInBucket = 512;
constexpr int kRowGroupWords = 64;               // bitmap words per entry of the free-row index (one per lane)
struct BucketArgs {
  const uint64_t *split;      // [kMaxBuckets] score bits of survivor ranks c*K/nb, c = 1..nb-1, then +inf
  const uint64_t *thresh;     // [1] score bits of the K-th survivor
  uint32_t       *count;      // [kBucketCounters] offspring per bucket (spilled ones included), this generation
  uint64_t       *keys;       // [nb][seg] score bits of the bucket's offspring
  uint32_t       *idx;        // [nb][seg] their pool slots
  uint64_t       *spill_keys; // [P] surplus candidates: score bits, slot, bucket
  uint32_t       *spill_idx;
  uint32_t       *spill_bucket;
  uint32_t       *split_slot; // [kMaxBuckets] general selection: the pool slots that go with the splitters' scores
  uint32_t       *ties;       // [kTieClasses][tie_words] the children of each class, by slot, then [kTieMask] a bit per class that has
                              // any; zero when a generation begins
  uint64_t       *split_next; // splitters and threshold for the next generation (same arrays)
  uint64_t       *thresh_next;
  uint32_t        nb, seg;
};

// Boundary rank of bucket c (c = 0..nb); bucket b owns survivor ranks [bound(b), bound(b+1)).
__device__ __forceinline__ uint32_t bucket_bound(uint32_t c, uint32_t K, uint32_t nb) {
  return (c * K) / nb;          // c <= 1024, K <= 2^18: the product fits 32 bits
}

constexpr uint64_t kNoSplitter = 0x7FF0000000000000ull;       // +infinity pads the table of splitters

// Remaining work of slot j under probability sampling (Alg. 1, Eq. 7) for generation t:
// tab.Y[j] = processed[j] * (1/rho - 1), rho ~ Be(alpha[j], beta[j]), for j < Jn; then the
// slot's entries of the term table.
struct Progress {
  const double *alpha, *beta, *processed;   // [Jp]
};
// The draws depend on nothing but (seed, slot, generation), so they are made ahead, those of many
// generations in one launch: generation g's remaining work and term table sit at place g mod n of a ring of
// n (Y, terms) pairs, n = kDrawRing for pools of resident_kernel, else kDrawAhead (the kernels of one generation; the
// whole calls of fused_kernel draw for themselves).
constexpr int kDrawRing = 32;
constexpr int kDrawAhead = 8;       // generations drawn at a time for the kernels of one generation

// How a kernel tells the host that it, and so everything before it on the stream, is done: its last workgroup writes `value` to a
// word of pinned memory that the host polls.  (A kernel and a wait of this kind take 5.9 us alone, with hipStreamSynchronize 9.3; a
// copy from or to pinned memory is another 5 to 6, so these kernels read and write it themselves.)
struct HostSignal {
  uint32_t *arrived;          // workgroups that are done: zero between launches, see last_to_arrive
  uint32_t *flag;
  uint32_t  value;
};
// What a launch that runs a whole call leaves in pinned memory: the winner, as ones_best hands it out, and the error words.
struct WinnerOut {
  int32_t  *batch, *gpus;     // [n_slots]
  double   *fit;
  uint32_t *of;               // the value of the launch's signal
  uint32_t *err;              // [2]
  uint32_t  n_slots;
  HostSignal done;
};

// Whether the repair is faster if it walks along the genes near its start (see Window), on G GPUs, with jobs that would take `demand`
// of them at their limits.  Whole genomes of one or two rows of slots are shed and filled in fewer instructions than it takes
// to lay a window out and walk it (17 slots, pool 7676, sampled: an epoch of 44 generations 1037 us walking, 994 not; 103 slots, pool
// 15844, 4 generations 115 and 111; three rows: 130 slots, pool 260, 8 generations 106 and 110; four: 212 slots, pool 15848, 40
// generations 893 and 923).  And where the GPUs are enough for most jobs, few of them ask for more, and the walk leaves its window, the
// sooner the shorter the genome (six generations on 0.7, 0.9, 1 and 1.05 of the demand: 1004 slots, pool 32768 206, 230, 213 and
// 244 us walking, 227, 227, 187 and 203 not; 200 slots 139, 144, 135 and 151, 140, 136, 122 and 129; 2028 276, 303, 274 and 287,
// 311, 310, 250 and 271; speed of walking on 0.5, 0.6, 0.7 and 0.8, jobs of up to 16 GPUs: 140 slots, pool 20000 0.96, 0.95, 0.96 and 0.97, 200,
// pool 32768 1.08, 1.03, 1.01 and 0.96, 1004 1.18, 1.11, 1.07 and 1.08).  A launch that runs whole calls (whole_call) waits for its
// slowest wave in every generation, and there it pays less (200 slots, pool 8192 1.01, 0.98, 0.95 and 0.93; 500 1.05, 0.97, 0.90 and
// 0.87; 1000, pool 4096 1.02, 0.95, 0.95 and 0.91; jobs of up to 4 GPUs 1.01, 1.04, 1.02 and 0.99; 1.05, 1.03, 1.00 and 0.97; 1.08, 1.05,
// 0.99 and 0.89).
inline bool walk_pays(uint32_t Jp, uint32_t G, uint64_t demand, bool whole_call) {
  const uint32_t twentieths = whole_call ? 11 : Jp <= 256 ? 13 : Jp <= 1024 ? 17 : 19;
  return Jp > 2 * kLanes && 20ull * G <= twentieths * demand;
}

// Genomes live in physical rows; a candidate keeps its row for as long as it survives, so a
// survivor is never copied.  The pool of P slots uses P + K rows.  While a generation is computed
// the K survivors hold theirs (parent_row); 3K rows are for the new children and mutants, by slot
// (row_of), and K are spare: a survivor that must be refreshed after a table change goes to the
// spare row of its rank, and its old one is the next spare.
// Which rows the 3K slots get:
// - After a bucketed selection nearly all of them keep the row that their slot had, whose candidate
//   dropped out.  A child that survived keeps it instead; as many survivors dropped out at the end
//   of the ranking, and the selection hands the row of the last but i to the slot of the i-th best
//   surviving child.  row_of and spare hold everything (assigned).
// - After any other selection a bitmap holds the survivors' rows, and the evolve kernel looks the free
//   ones up in ascending order: the slot K + q takes the q-th, the last K are spare.
struct EvolveArgs {
  uint32_t       *genes;      // [P + K][Q * 64] genome rows
  double         *fit_row;    // [P + K] score of the genome in each row
  const uint32_t *parent_row; // [K] rows of the survivors, best first
  uint32_t       *row_of;     // [P] row of every slot of the new pool
  uint32_t       *spare;      // [K] rows no slot uses
  const uint32_t *occupied;   // bitmap over the P + K rows: the survivors' rows (unless assigned)
  uint32_t       *occupied_other;  // the other bitmap, cleared here for the coming selection (null: it uses none)
  uint32_t       assigned;    // row_of and spare hold the rows of the slots to fill
  JobTable       tab;
  uint32_t       G, P, K, Jp;
  uint32_t       key0, key1;  // seed
  uint32_t       t;           // generation counter (0 = initial population)
  uint32_t       T_mut, T_x;  // rate thresholds on a 32-bit word
  uint32_t       new_first;   // after a table change: the jobs that arrived with it are served first
  const uint32_t *time_rank;  // [Jp] with new_first: position of every slot in ascending order of executed
                              //      time, the order the other jobs are admitted in; null = visiting order
  uint32_t       rescore;     // the survivors' scores are stale (remaining work redrawn): score them again
  uint32_t       per_gpu;     // the uniform crossover scans the GPUs (Eq. 1) instead of the jobs; needs G <= kMaxCoinGpus
  uint32_t       coin_stride; // set by the launcher: bytes of LDS scratch per wave
  uint32_t       walk;        // the repair walks along the genes near its start: walk_pays, and then whether the launcher finds
                              // room in LDS for what it needs
  uint32_t       term_lds;    // set by the launcher: entries per job of the term table in LDS, 0 = none
  uint32_t       *fault;      // [1] raised when a row index had to be pulled back into the genome array
  double         *slot_score; // [P] the score of every candidate this launch scores, by pool slot (written when
                              //     the buckets are off): what the general selection reads when the launch scored
                              //     the whole pool, in place of slot -> row -> score
  BucketArgs     bk;
};

// All generations of one ones_generation call in a single launch, for pools that are small
// enough to be ranked inside every workgroup's LDS (one row of 64 job columns, at most
// kFusedMaxPool candidates).  ev describes the problem as for the evolve kernel (row_of and spare
// are written when the launch ends, and read when assigned is set); ev.t is the generation counter
// BEFORE the call (the launch runs generations ev.t + 1 .. ev.t + n_generations).
constexpr uint32_t kFusedMaxPool = 2048;
struct FusedArgs {
  EvolveArgs ev;
  uint32_t *parent_rows;    // [K] in: rows of the survivors, best first; out: of the new survivors
  int32_t  *sel;            // [K] out: survivor slots of the last generation's pool, best first
  // exchange between the workgroups, zeroed when the context is created, then only written by these launches:
  uint64_t *xkeys;          // [2][P] tagged score bits of the children by pool slot, a buffer per generation parity
  uint64_t *xsurv;          // [2][K] the same for survivors with a new score
  uint64_t *xrank;          // [P] ranks from a ranking by counting, stamped with the generation
  uint64_t *xdraw;          // [4][64] tagged draws of the remaining work (probability sampling), four generations rotating
  uint32_t *sync;           // [1] set when a poll ran out
  uint32_t generations_before;  // generations these launches have run for the context so far
  uint32_t changes_before;      // ... of them generations that also exchanged the survivors' scores
  uint32_t draws_before;        // ... of them generations with a drawn remaining work
  uint32_t sampled;             // probability sampling (Alg. 1): every generation draws the remaining work anew
  Progress pr;                  // its inputs
  uint32_t n_slots;             // Jn: slots at or beyond it have no remaining work
  double  *y_out;               // [64] out: the remaining work the last generation was scored with
  uint32_t n_generations;   // > 1
  uint32_t first_changed;   // the job table changed since the survivors were scored: the first generation refreshes them
  uint32_t spin_limit;      // polls before a wait gives up (0: gives up at once; for tests of that path)
  uint32_t table_lds;       // set by the launcher: bytes of LDS the staged job table takes
  uint32_t work_groups;     // set by the launcher: workgroups that compute candidates (the grid's first ones)
  WinnerOut winner;         // its signal is given by one workgroup
};
// Workgroups to launch for a pool of P (the launch must be co-resident: cooperative).
uint32_t fused_workgroups(uint32_t P, bool sampled);
uint32_t fused_grid_limit(uint32_t P);      // the largest grid a launch for a pool of P uses
size_t fused_exchange_bytes(uint32_t P);    // xkeys, xsurv, xrank and xdraw, consecutive
void fused_exchange(uint64_t *base, uint32_t P, FusedArgs &fa);   // their addresses
hipError_t launch_fused(const FusedArgs &fa, hipStream_t s);

// The same for pools beyond those (ones_resident.hip): at most kResidentMaxPool candidates of up to
// 256 * kResidentMaxWords job slots, as far as a compute unit's LDS holds them (resident_plan).
constexpr int kResidentMaxPool = 16384;
constexpr int kResidentMaxWords = 4;
constexpr uint32_t kResidentMaxGroups = 1024;   // workgroups of a launch: flags in the workspace
struct ResidentArgs {
  EvolveArgs ev;            // ev.bk.nb is 0: no buckets while the launch runs
  uint32_t *parent_rows;    // as in FusedArgs, as are the following, but for
  int32_t  *sel;
  uint64_t *xkeys;          // [2][P] score bits by pool slot, a buffer per generation parity
  uint32_t *xrow;           // [2][P] ... and rows
  uint64_t *flags;          // [2][kResidentMaxGroups] the generation of the context a workgroup has published the candidates of
                            // and, below it, how many of its children beat the K-th survivor
  uint64_t *lists;          // [2][P + 2 kResidentMaxGroups][2] score bits of those children; slot, row and the row's place among the
                            // workgroup's; `segment` entries per workgroup
  uint64_t *xrank;          // [K] slot and row of the survivors by rank, from a ranking by counting, stamped with the generation
  uint32_t n_buckets;       // 0, or, for the generation after the launch: buckets whose splitters, ...
  uint64_t *split, *thresh; // ... threshold ...
  uint32_t *count[2];       // ... and cleared counters the launch leaves, see BucketArgs
  uint32_t *sync;
  uint32_t generations_before;
  uint32_t sampled;
  const double *ring_terms; // the term tables of the draws, generation t's at place t mod kDrawRing, made before the launch
  uint32_t ring_stride;     // doubles between two places
  uint32_t n_generations;   // > 1; under probability sampling at most kDrawRing
  uint32_t first_changed, spin_limit;
  uint32_t paired, unit_waves, child_items, segment, list, table_lds;    // from the plan
  WinnerOut winner;         // its signal is given by all workgroups
};
// paired: a wave's item is a pair or a mutant, not a child.  unit_waves: waves of a workgroup that start with an item each;
// child_items: items of a workgroup that are no survivors, segment: children they make, list: children that beat the K-th
// survivor a workgroup can rank, all at most; walk: see EvolveArgs; table_lds: LDS bytes of the job table.
struct ResidentPlan { uint32_t groups, paired, unit_waves, child_items, segment, list, coin_stride, walk, table_lds; size_t lds; };
size_t resident_exchange_bytes(uint32_t P);     // lists, xkeys, xrank, flags and xrow, consecutive
void resident_exchange(uint64_t *base, uint32_t P, ResidentArgs &ra);      // their addresses
// How a launch for ev's pool and job table would be shaped; false: it does not fit.
bool resident_plan(const EvolveArgs &ev, bool sampled, int n_cus, ResidentPlan &plan);
hipError_t launch_resident_words1(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t s);
hipError_t launch_resident_words2(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t s);
hipError_t launch_resident_words3(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t s);
hipError_t launch_resident_words4(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t s);

// What a selection records besides the survivor list: the survivors keep their rows.
struct RowPlan {
  uint32_t       *row_of;       // [P] row of every slot of the pool being ranked
  const uint32_t *parents;      // [K] rows of the survivors of the selection before (bucketed selection)
  uint32_t       *parent_next;  // [K] rows of the new survivors, best first
  uint32_t       *occupied;     // bitmap over the P + K rows, zero on entry; survivors' rows get set (general selection)
};

// T_j c_j of a job at GPU-count code e (0 = waiting, e = 1 + log2 of the GPU count): Eq. 3
// with T = Y / X (Eq. 5) and the iteration time a*b + c*log2(g) + d at the job's local batch
// b = 2^blexp; abl = a * b.  Same operations in the same order wherever a term is computed.
__device__ __forceinline__ double term_of(double abl, double cc, double d, double Y, uint32_t blexp, uint32_t e) {
  if (e == 0) return 0.0;
  const double lg = static_cast<double>(e - 1);
  const double inv_bl = __hiloint2double(static_cast<int>((1023u - blexp) << 20), 0);
  const double t = (abl + cc * lg) + d;
  return (Y * t) * inv_bl;
}

struct RawJobs {              // uploaded by the host after validation, [Jp] each
  const uint32_t *rawinfo;    // bits 0-4 lo, 5-9 hi, 10-14 mu, 15 active, 16 arrived with this table, 17 changed hands
  const double   *a, *c, *d, *Y;
};

// launchers (each returns the hipGetLastError of its launch)
// The per-slot values and the term table from the raw table, and the slots that changed hands marked
// in tab.stored (unless the genomes are, or will be, stored under this table); one launch.  remaining: the raw table's, kept.
hipError_t launch_table_change(const RawJobs &raw, const JobTable &tab, double *remaining, uint32_t Jp, const HostSignal &done, hipStream_t s);
// n 16-byte words.
hipError_t launch_fetch(const void *from, void *to, uint32_t n, const HostSignal &done, hipStream_t s);
hipError_t launch_build_terms(const JobTable &tab, uint32_t Jp, hipStream_t s);
// ring: the job table with Y and terms pointing at place 0 of a ring of `places`, which lie
// ring_stride doubles apart; draws generations t .. t + count - 1 (count <= places).
hipError_t launch_sample_remaining(const Progress &pr, const JobTable &ring, uint32_t ring_stride, uint32_t places, uint32_t Jn,
                                   uint32_t Jp, uint32_t key0, uint32_t key1, uint32_t t, uint32_t count,
                                   hipStream_t s);
// same_table: the job table is the one the previous generation was repaired and scored with
hipError_t launch_evolve_group0(const EvolveArgs &a, int words, bool same_table, int n_cus, hipStream_t s);
hipError_t launch_evolve_group1(const EvolveArgs &a, int words, bool same_table, int n_cus, hipStream_t s);
hipError_t launch_evolve_group2(const EvolveArgs &a, int words, bool same_table, int n_cus, hipStream_t s);
hipError_t launch_evolve_group3(const EvolveArgs &a, int words, bool same_table, int n_cus, hipStream_t s);
inline hipError_t launch_evolve(const EvolveArgs &a, int rows, bool same_table, int n_cus, hipStream_t s) {
  const int words = words_of(rows);
  switch ((words - 1) / 2) {
    case 0: return launch_evolve_group0(a, words, same_table, n_cus, s);
    case 1: return launch_evolve_group1(a, words, same_table, n_cus, s);
    case 2: return launch_evolve_group2(a, words, same_table, n_cus, s);
    case 3: return launch_evolve_group3(a, words, same_table, n_cus, s);
    default: return hipErrorInvalidValue;
  }
}
// General selection (any scores).  store: the bucket storage (count, keys, idx and spill arrays,
// split and split_slot as scratch for the splitters, nb * seg entries of bucket space); used by pools
// too large for the single launch that ranks a whole pool.  slot_score: the pool's scores by slot
// when the evolve launch wrote them all, else null (they are then looked up through the rows).
hipError_t launch_select(const double *fit_row, const double *slot_score, const RowPlan &rp, uint32_t P, uint32_t K,
                         const BucketArgs &store, int32_t *sel, hipStream_t s);
hipError_t launch_zero_words(uint32_t *words, uint32_t n, hipStream_t s);
// count_next, ties_next: the other set of counters and bitmaps, cleared for the next generation.
hipError_t launch_bucket_select(const double *fit_row, const BucketArgs &bk, const RowPlan &rp, uint32_t K,
                                uint32_t *count_next, uint32_t *ties_next, int32_t *sel, hipStream_t s);
hipError_t launch_splitters(const double *fit_row, const uint32_t *row_of, const int32_t *sel, uint32_t K,
                            uint32_t nb, uint64_t *split, uint64_t *thresh, uint32_t *count0, uint32_t *count1,
                            uint32_t *ties, uint32_t ties_words, hipStream_t s);
// Eq. 1 for the winner: GPU i runs slot slot_of_gpu[i] (-1 = idle) with batch_of_gpu[i] samples;
// jobs in slot order on consecutive GPUs.  G entries each.  best: row of the winner.
hipError_t launch_placement(const uint32_t *genes, const uint32_t *best, const uint32_t *info, uint32_t Jn, uint32_t Jp,
                            uint32_t G, int32_t *slot_of_gpu, int32_t *batch_of_gpu, const uint32_t *err_in, uint32_t *err_out,
                            const HostSignal &done, hipStream_t s);
// stored: info of the table the genomes are stored under, info: of the table in force.
hipError_t launch_best(const uint32_t *genes, const double *fit_row, const uint32_t *best, const uint32_t *stored,
                       const uint32_t *info, uint32_t Jn, uint32_t Jp, int32_t *batch_out, int32_t *gpus_out,
                       double *fit_out, const uint32_t *err_in, uint32_t *err_out, const HostSignal &done, hipStream_t s);
// The state as ones_export hands it out.  The rows of the survivors, slot sel[g] in row parents[g], go by
// parents, those of the other slots by row_of.
struct ExportArgs {
  const uint32_t *genes;
  const double   *fit_row;
  const uint32_t *row_of;
  const int32_t  *sel;
  const uint32_t *parents;
  const uint32_t *stored;     // info of the table the genomes are stored under
  const uint32_t *err_in;     // [2] the error words
  uint32_t        P, K, Jp;
  double         *fit_out;    // [P] in slot order
  int32_t        *sel_out;    // [K]
  uint32_t       *err_out;    // [2]
  int32_t        *genes_out;  // [count][Jp] batch sizes of the slots [first, first + count)
  HostSignal      done;       // given by the last kernel of launch_export_genes, flag null: by none
};
// Scores, survivors and error words.
hipError_t launch_export_scores(const ExportArgs &x, hipStream_t s);
// The genomes of a run of slots; with_scores: and, the slots being the whole pool, everything else.
hipError_t launch_export_genes(const ExportArgs &x, uint32_t first, uint32_t count, bool with_scores, hipStream_t s);

}  // namespace ones
