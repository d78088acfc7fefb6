// All generations of one ones_generation call in a single launch (ONES, arXiv 2108.03645,
// Section 3.2.2), for the pools the paper itself schedules with (population = cluster size,
// Section 3.2.2 "Initialization"; 64 GPUs in Section 4.1): at most 64 job slots and
// kFusedMaxPool candidates.
//
// Two launches per generation cost more than the generation itself at this size, so here a
// co-resident grid stays on the chip for the whole call.  Per generation every wave composes,
// repairs and scores its share of the 3K children (4K candidates when every score is new: after a
// table change and under probability sampling) and publishes genome and score; every workgroup then
// collects all scores and ranks the pool by itself in its LDS: the survivors' scores and rows and the
// rows of the slots to fill are kept there redundantly, so the only data that cross workgroups are
// the genomes and one score per candidate.  While the scores stay the same the K survivors
// reappear with theirs, already in order, so the ranking is a merge of the few children that beat
// the K-th survivor into that order; when there are many of them, or every score is new, every
// workgroup ranks a share of the pool by counting and the ranks are exchanged like the scores.
//
// Exchange.  Data written by one workgroup and read by another inside the launch (genomes,
// scores, ranks) go through relaxed atomic stores and loads at device scope, which the hardware
// performs at the device's point of coherence instead of in the caches of one XCD.  There is no
// barrier: a published score carries a tag (its sign bit, which a score never uses, alternating
// with every reuse of the exchange buffer; ranks carry the generation number), a reader polls
// until every entry shows the tag of the current generation, and a wave publishes its score only
// after its genome stores have been acknowledged.  Seeing all scores of a generation therefore
// means that every wave has finished reading that generation's parents and writing its
// children, which is all the ordering the rows need.  Every poll is bounded: a workgroup that
// gives up sets an error word and leaves, and so, in time, do all others.
// What bounds a generation is this exchange: all workgroups read the same few kilobytes of the memory
// side at once, so a poll that comes too early delays those that matter.  (A generation of 1024
// candidates, 96 workgroups: 4.5 us with one poll after the other, no branch around a load and a
// pause before the first poll; 4.8 without the pause; 5.1 with a branch per load; two polls in
// flight 4.8, four 5.4.  A flag per workgroup, polled in place of the scores, reads an eighth of the
// bytes but waits for the workgroup's slowest wave first: 5.5.)
#include "ones_candidate.h"
#include "ones_exchange.h"
#include "ones_sample.h"
#include "ones_sort.h"

#include <cstddef>
#include <cstdlib>

namespace ones {
namespace {

constexpr int kFusedWaves = 8;                         // waves per workgroup
constexpr int kFusedThreads = kFusedWaves * kLanes;
constexpr uint32_t kFusedMaxWorkgroups = 192;
constexpr uint32_t kFusedMaxSampledWorkgroups = 248;   // plus the drawing ones: one per compute unit at most
constexpr uint32_t kFusedUnits = 4;          // most units (candidates) one wave computes per generation
constexpr uint32_t kMergeMax = 128;          // children beating the K-th survivor that are merged into the survivors' order
// With so many workgroups a wave waits a little before its first poll, until the others' entries are
// nearly there: 0.2 us for the scores of the children, 1.3 us where the survivors are scored too, 0.4 us
// for ranks (1024 candidates: a generation 4.8 -> 4.5 us; 2048 sampled, over the GPUs: 14.4 -> 12.3).
constexpr uint32_t kCrowd = 32;
constexpr int kGatherPer = (kFusedMaxPool + kFusedThreads - 1) / kFusedThreads;   // entries per thread when a workgroup collects P values
static_assert(kFusedMaxPool / 4 <= kFusedThreads, "a thread per survivor");

// Tag of the n-th use (n = 0, 1, ..) of a pair of exchange buffers that start out zeroed: use n
// goes to buffer n & 1 and flips the tag that buffer's entries carried before.
__device__ __forceinline__ uint64_t use_tag(uint32_t n) { return static_cast<uint64_t>(((n >> 1) & 1u) ^ 1u) << 63; }
constexpr uint64_t kTagBit = 1ull << 63;
// The draws of the remaining work are published two generations ahead, so they rotate through
// four buffers instead of two.
constexpr uint32_t kDrawBuffers = 4;
constexpr uint32_t kDrawGroups = (kLanes / 4 + kFusedWaves - 1) / kFusedWaves;   // workgroups that only draw: a wave per four slots
static_assert(kDrawGroups * kFusedWaves == kLanes / 4, "the drawing workgroups have exactly one wave per four job slots");
__device__ __forceinline__ uint64_t draw_tag(uint32_t n) { return static_cast<uint64_t>(((n / kDrawBuffers) & 1u) ^ 1u) << 63; }

// Per-workgroup copy of the search state between two generations, plus scratch of the ranking.
struct Ranks {
  uint64_t *skeys;     // [2][K] score bits of the survivors, best first (two generations alternate)
  uint16_t *srows;     // [2][K] their genome rows
  uint32_t K;
  // (pointer arithmetic instead of an array of pointers: a runtime index into such an array would
  // put this struct into scratch memory)
  __device__ __forceinline__ uint64_t *skey(int which) const { return skeys + static_cast<uint32_t>(which) * K; }
  __device__ __forceinline__ uint16_t *srow(int which) const { return srows + static_cast<uint32_t>(which) * K; }
  uint16_t *nsel;      // [K] pool slot each new survivor had in the generation just ranked
  uint16_t *frow;      // [P] the row unit u of a generation writes; the last K are spare between table changes
  uint64_t *ckey;      // [P] score bits by pool slot
  uint64_t *lkey;      // [3K] children that beat the K-th survivor
  uint16_t *lslot;     // [3K] ... their slots
  uint64_t *okey;      // [kMergeMax] ... in order
  uint16_t *oslot;     // [kMergeMax]
  uint32_t *below;     // [kMergeMax] counters of the rankings by counting
  uint32_t *bits;      // bitmap: over the P + K rows when rows are listed, over the survivors of the generation before
  uint32_t *wfree;     // free rows before each word of the bitmap
  uint16_t *drow;      // [K] rows of survivors that dropped out
  uint32_t *wcount;    // [2][kFusedWaves] counts of the waves, for prefix sums
  uint32_t *misc;      // [0] number of children that beat the K-th survivor, [1 + generation mod 3] whether there is one
  uint32_t *draws;     // [waves][kFusedUnits][4] per unit: ranks of the parents, rotation (drawn ahead)
  uint32_t *words;     // [waves][kFusedUnits][64] per unit: the gene words (drawn ahead)
  uint64_t *ukeys;     // [waves][kFusedUnits] per unit: the score, until the wave publishes it
  double   *ydraw;     // [64] remaining work of every slot as drawn for the generation being computed (Alg. 1)
  double   *model;     // [3][64] the slots' a * local batch, c and d, from which a draw gives the term table
  uint32_t *blexp;     // [64] ... and log2 of their local batch
};

inline size_t ranks_bytes(uint32_t P) {
  const size_t K = P / 4, words = (P + K + 31) / 32;
  return 4 * kLanes * 8 + kFusedWaves * kFusedUnits * 8 + 2 * K * 8 + static_cast<size_t>(P) * 8 + 3 * K * 8 + kMergeMax * 8 +
         4 * (kMergeMax + 2 * words + 2 * kFusedWaves + 4 + kFusedWaves * kFusedUnits * (4 + kLanes) + kLanes) +
         2 * (2 * K + K + P + 3 * K + kMergeMax + K) + 64;
}

__device__ __forceinline__ Ranks carve_ranks(unsigned char *base, uint32_t P) {
  const uint32_t K = P / 4, words = (P + K + 31) / 32;
  Ranks r;
  r.K = K;
  r.ydraw = reinterpret_cast<double *>(base);
  r.model = r.ydraw + kLanes;
  r.ukeys = reinterpret_cast<uint64_t *>(r.model + 3 * kLanes);
  r.skeys = r.ukeys + kFusedWaves * kFusedUnits;
  r.ckey = r.skeys + 2 * K;
  r.lkey = r.ckey + P;
  r.okey = r.lkey + 3 * K;
  r.below = reinterpret_cast<uint32_t *>(r.okey + kMergeMax);
  r.bits = r.below + kMergeMax;
  r.wfree = r.bits + words;
  r.wcount = r.wfree + words;
  r.misc = r.wcount + 2 * kFusedWaves;
  r.draws = r.misc + 4;
  r.words = r.draws + kFusedWaves * kFusedUnits * 4;
  r.blexp = r.words + kFusedWaves * kFusedUnits * kLanes;
  r.srows = reinterpret_cast<uint16_t *>(r.blexp + kLanes);
  r.nsel = r.srows + 2 * K;
  r.frow = r.nsel + K;
  r.lslot = r.frow + P;
  r.oslot = r.lslot + 3 * K;
  r.drow = r.oslot + kMergeMax;
  return r;
}

// The rows that are not the survivors' (rows[0..K)), in ascending order, as rows of the units, when
// no selection has assigned them.  Whole workgroup; ends with a barrier.
__device__ __forceinline__ void list_free_rows(const Ranks &rk, const uint16_t *rows, uint32_t P) {
  const uint32_t K = P / 4, n_rows = P + K, words = (n_rows + 31) / 32;   // at most 80 words
  for (uint32_t w = threadIdx.x; w < words; w += blockDim.x) rk.bits[w] = 0;
  __syncthreads();
  for (uint32_t g = threadIdx.x; g < K; g += blockDim.x) atomicOr(&rk.bits[rows[g] >> 5], 1u << (rows[g] & 31u));
  __syncthreads();
  // free rows before each bitmap word (one wave scans the words' counts), ...
  if (threadIdx.x < kLanes) {
    uint32_t carry = 0;
    for (uint32_t base = 0; base < words; base += kLanes) {
      const uint32_t w = base + threadIdx.x;
      const uint32_t n = w < words ? __popc(~rk.bits[w]) : 0u;   // bits beyond the last row are never looked at
      const uint32_t incl = wave_inclusive_scan(n);
      if (w < words) rk.wfree[w] = carry + incl - n;
      carry += __builtin_amdgcn_readlane(incl, kLanes - 1);
    }
  }
  __syncthreads();
  // ... then every row finds its own place in the list
  for (uint32_t row = threadIdx.x; row < n_rows; row += blockDim.x) {
    const uint32_t free_bits = ~rk.bits[row >> 5], bit = row & 31u;
    if ((free_bits >> bit) & 1u) {
      const uint32_t pos = rk.wfree[row >> 5] + __popc(free_bits & ((1u << bit) - 1u));
      if (pos < P) rk.frow[pos] = static_cast<uint16_t>(row);
    }
  }
  __syncthreads();
}

// Collects n published 64-bit entries: thread t takes entries t, t + threads, ..., polls until every one
// is ready and hands it to take.  at(e): the address of entry e.  False when the polls ran out.  No
// branch around a load: a thread reads its entries again until the wave has all of its own.
template <int kPer, typename At, typename Ready, typename Take>
__device__ __forceinline__ bool gather_per(uint32_t n, uint32_t spin_limit, At at, Ready ready, Take take) {
  uint32_t pending = 0;
  const uint64_t *src[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t e = threadIdx.x + k * kFusedThreads;
    if (e < n) pending |= 1u << k;
    src[k] = at(min(e, n - 1));
  }
  if (__ballot(pending != 0) == 0) return true;
  for (uint32_t spins = 0; spins < spin_limit; ++spins) {
    uint64_t v[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) v[k] = shared_load(src[k]);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t e = threadIdx.x + k * kFusedThreads;
      if (((pending >> k) & 1u) && ready(e, v[k])) {
        take(e, v[k]);
        pending &= ~(1u << k);
      }
    }
    if (__ballot(pending != 0) == 0) return true;
  }
  return false;
}

template <typename At, typename Ready, typename Take>
__device__ __forceinline__ bool gather(uint32_t n, uint32_t spin_limit, At at, Ready ready, Take take) {
  static_assert(kGatherPer <= 4, "entries per thread");
  switch ((n + kFusedThreads - 1) / kFusedThreads) {
    case 1: return gather_per<1>(n, spin_limit, at, ready, take);
    case 2: return gather_per<2>(n, spin_limit, at, ready, take);
    case 3: return gather_per<3>(n, spin_limit, at, ready, take);
    default: return gather_per<4>(n, spin_limit, at, ready, take);
  }
}

// What a child or mutant draws before it needs anything of its parents: the parents' ranks and
// the rotation of its repair (draw_parents), its word per gene (draw_words).  Both depend on
// (seed, generation, slot) only, so a wave draws for the coming generation while the scores of
// the current generation are still arriving.
__device__ __forceinline__ void draw_parents(const EvolveArgs &a, uint32_t t, uint32_t u, int lane, uint32_t *draws) {
  // a child of a pair shares the parents drawn for the pair's first slot, its rotation is its own:
  // lane 0 draws for the former, lane 1 for the latter
  const bool child = u < 2 * a.K;
  const uint32_t p = a.K + u;
  const Draw d = candidate_draw(a, t, child && lane == 0 ? p - (u & 1u) : p);
  if (lane == 0) { draws[0] = d.ra; draws[1] = d.rb; }
  if (lane == 1) draws[2] = d.r;
}

// The one row of job slots takes the first word of a Philox block.
template <bool kOverGpus>
__device__ __forceinline__ void draw_words(const EvolveArgs &a, uint32_t t, uint32_t u, int lane, const uint2 *prefix,
                                           uint32_t *words) {
  const uint32_t K = a.K;
  uint32_t w = 0;
  if (u >= 2 * K) w = WordSource(a, t, K + u).block(prefix, 0, lane).w[0];
  else if (!kOverGpus) w = WordSource(a, t, K + (u & ~1u)).block(prefix, 0, lane).w[0];   // both children share the pair's words
  words[lane] = w;
}

// One candidate of generation t: unit u < 2K is a child of pair u / 2, u < 3K a mutant, u >= 3K
// (only after a table change) the survivor of rank u - 3K to refresh.  srow: rows of the
// survivors by rank.  Returns the score; the repaired genes are left in c.
template <bool kSameTable, bool kOverGpus>
__device__ __forceinline__ double compose_unit(const EvolveArgs &a, uint32_t t, const Smem &s, const uint16_t *srow,
                                               uint32_t u, bool new_first, uint64_t *coins, const uint32_t *draws,
                                               const uint32_t *words, int lane, uint32_t (&c)[1]) {
  const uint32_t K = a.K;
  uint32_t r;
  auto gene_of = [&](uint32_t row) { return shared_load(a.genes + static_cast<size_t>(row) * kLanes + lane); };
  if (u < 3 * K) {
    const uint32_t ra = __builtin_amdgcn_readfirstlane(draws[0]), rb = __builtin_amdgcn_readfirstlane(draws[1]);
    r = __builtin_amdgcn_readfirstlane(draws[2]);
    const uint32_t w = words[lane];
    if (u < 2 * K) {
      const uint32_t side = u & 1u;
      uint32_t B[1];
      c[0] = gene_of(srow[ra]);
      B[0] = gene_of(srow[rb]);
      if (kOverGpus) {
        if (!kSameTable) { to_new_table<1>(s, lane, c); to_new_table<1>(s, lane, B); }
        crossover_over_gpus<1, kSameTable>(a, t, s, coins, K + (u & ~1u), lane, c, B);
        c[0] = side ? B[0] : c[0];
      } else {
        const bool swap = w < a.T_x;                 // the first child takes the second parent's gene
        c[0] = (swap != (side != 0)) ? B[0] : c[0];
        if (!kSameTable) to_new_table<1>(s, lane, c);
      }
    } else {
      c[0] = gene_of(srow[ra]);
      if (!kSameTable) to_new_table<1>(s, lane, c);
      const uint32_t k = ((w & 0xFFFFu) * (s.draws[lane] & 0xFFu)) >> 16;
      c[0] = w < a.T_mut ? codes_of_draws(s, lane, k) : c[0];
    }
  } else {
    const uint32_t p = u - 3 * K;
    r = __builtin_amdgcn_readfirstlane(candidate_draw(a, t, p).r);
    c[0] = gene_of(srow[p]);
    to_new_table<1>(s, lane, c);
  }
  if (!kSameTable && new_first) repair<1, kOneRow, true>(c, s, a.G, r, 0, lane, kLanes, a.time_rank != nullptr, nullptr, false);
  else repair<1, kOneRow, false>(c, s, a.G, r, 0, lane, kLanes, false, nullptr, false);
  return score<1, 1>(c, s, a.term_lds, lane);
}

// ------------------------------------------------------------------ ranking --------
// The rows that go with a ranking of the whole pool: the new survivors keep theirs, and the slots of
// the surviving children take the rows of the survivors that dropped out, the i-th the i-th (both
// counted in the same order by every workgroup).  changed: the pool's first K slots are refreshed
// survivors in the spare rows, and the rows they came from are spare from now on.
__device__ __forceinline__ void assign_rows(const Ranks &rk, uint32_t P, int cur, int nxt, bool changed) {
  const uint32_t K = P / 4, tid = threadIdx.x, lane = tid % kLanes, wave = tid / kLanes;
  const uint32_t words = (K + 31) / 32;
  if (tid < words) rk.bits[tid] = 0;
  __syncthreads();
  const uint32_t slot = tid < K ? rk.nsel[tid] : 0u;
  const bool child = tid < K && slot >= K;
  if (tid < K && !child) atomicOr(&rk.bits[slot / 32], 1u << (slot % 32));
  __syncthreads();
  const bool dead = tid < K && ((rk.bits[tid / 32] >> (tid % 32)) & 1u) == 0;
  const uint64_t children = __ballot(child), gone = __ballot(dead);
  if (lane == 0) {
    rk.wcount[wave] = static_cast<uint32_t>(__popcll(children));
    rk.wcount[kFusedWaves + wave] = static_cast<uint32_t>(__popcll(gone));
  }
  auto elite_row = [&](uint32_t e) { return changed ? rk.frow[3 * K + e] : rk.srow(cur)[e]; };
  __syncthreads();
  const uint64_t before = (1ull << lane) - 1ull;
  uint32_t nth_child = static_cast<uint32_t>(__popcll(children & before)), nth_gone = static_cast<uint32_t>(__popcll(gone & before));
  for (uint32_t w = 0; w < wave; ++w) { nth_child += rk.wcount[w]; nth_gone += rk.wcount[kFusedWaves + w]; }
  if (dead) rk.drow[nth_gone] = elite_row(tid);
  if (tid < K) rk.srow(nxt)[tid] = child ? rk.frow[slot - K] : elite_row(slot);
  __syncthreads();
  if (child) rk.frow[slot - K] = rk.drow[nth_child];
  if (changed && tid < K) rk.frow[3 * K + tid] = rk.srow(cur)[tid];
  __syncthreads();
}

// (Argument block: FusedArgs by value, which starts with its EvolveArgs, see kernel_args.)
static_assert(offsetof(FusedArgs, ev) == 0, "kernel_args() reads the EvolveArgs at the start of the argument block");
// kSampled: the remaining work is drawn anew for every generation (Alg. 1, Eq. 7) and the whole
// pool, survivors included, is scored with the draw.
template <bool kOverGpus, bool kSampled>
__global__ __launch_bounds__(kFusedThreads) void fused_kernel(FusedArgs fa) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const EvolveArgs &a = fa.ev;
  const uint32_t P = a.P, K = a.K, tid = threadIdx.x;
  const Smem s = carve<1>(smem_raw, a.term_lds, kFusedWaves, a.coin_stride);
  const Ranks rk = carve_ranks(smem_raw + fa.table_lds, P);
  const int lane0 = tid & (kLanes - 1);
  const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the first work_groups workgroups compute candidates; under probability sampling kDrawGroups more only draw
  const uint32_t n_groups = fa.work_groups;
  const uint32_t wave = blockIdx.x * kFusedWaves + wave_in_block, n_waves = n_groups * kFusedWaves;
  uint64_t *coins = reinterpret_cast<uint64_t *>(s.coins + static_cast<size_t>(wave_in_block) * a.coin_stride);
  // The k-th unit of this wave.  Every second round is dealt from the last wave on: where every score is new, the last waves have a
  // survivor, which is only scored, and take the few units beyond one a wave; dealt from the first on those went to waves that
  // compose a child (an epoch of 20 sampled generations of 2048 candidates, 1984 waves: 300 us, now 286).
  auto unit_of = [&](uint32_t k) { return k * n_waves + (k % 2 == 0 ? wave : n_waves - 1 - wave); };
  uint32_t *my_draws = rk.draws + wave_in_block * kFusedUnits * 4;
  uint32_t *my_words = rk.words + wave_in_block * kFusedUnits * kLanes;
  auto draw_unit_parents = [&](uint32_t t) {         // for this wave's children and mutants of generation t
    for (uint32_t k = 0, u; k < kFusedUnits && (u = unit_of(k)) < 3 * K; ++k)
      draw_parents(a, t, u, opaque(lane0), my_draws + 4 * k);
  };
  auto draw_unit_words = [&](uint32_t t) {
    for (uint32_t k = 0, u; k < kFusedUnits && (u = unit_of(k)) < 3 * K; ++k)
      draw_words<kOverGpus>(a, t, u, opaque(lane0), s.prefix, my_words + kLanes * k);
  };
  uint64_t *my_keys = rk.ukeys + wave_in_block * kFusedUnits;
  const bool crowd = n_groups >= kCrowd;
  auto give_up = [&] { if (tid == 0) shared_store(fa.sync + 1, 1u); };
  // Probability sampling.  The draw of a generation takes a long chain of fp64 operations (about
  // 5 us), so it is made two generations ahead, by workgroups that do nothing else (sixteen lanes
  // per job slot, four slots per wave), and published, tagged; every computing
  // workgroup collects the 64 values while the scores arrive and rebuilds its LDS copy of the term
  // table from them between two generations.  n: how many draws these launches have made for the context before.
  auto publish_draw = [&](uint32_t t, uint32_t n) {  // called by the kLanes / 4 waves of the drawing workgroups
    uint64_t *xd = fa.xdraw + static_cast<size_t>(n % kDrawBuffers) * kLanes;
    const uint32_t j = 4 * (wave - n_waves) + static_cast<uint32_t>(lane0) / kLanesPerSlot;
    const double Y = draw_remaining(fa.pr, fa.n_slots, a.key0, a.key1, t, j);
    if (lane0 % kLanesPerSlot == 0) shared_store(xd + j, static_cast<uint64_t>(__double_as_longlong(Y)) | draw_tag(n));
  };
  auto collect_draw = [&](uint32_t n) -> bool {      // into ydraw; false when the polls ran out
    const uint64_t *xd = fa.xdraw + static_cast<size_t>(n % kDrawBuffers) * kLanes;
    return gather(kLanes, fa.spin_limit, [&](uint32_t j) { return xd + j; },
                            [&](uint32_t, uint64_t v) { return (v & kTagBit) == draw_tag(n); },
                            [&](uint32_t j, uint64_t v) { rk.ydraw[j] = __longlong_as_double(static_cast<long long>(v & ~kTagBit)); });
  };
  auto build_terms = [&] {                           // whole workgroup, from ydraw; between two barriers of its own
    __syncthreads();
    const uint32_t E = a.term_lds;
    for (uint32_t q = tid; q < E * kLanes; q += kFusedThreads) {
      const uint32_t e = q / kLanes, j = q % kLanes;
      s.terms[e * (4 * kLanes) + j] =
          term_of(rk.model[j], rk.model[kLanes + j], rk.model[2 * kLanes + j], rk.ydraw[j], rk.blexp[j], e);
    }
    __syncthreads();
  };
  if (kSampled && blockIdx.x >= n_groups) {
    // A drawing workgroup: the draws of the first three generations at once, then the draw of
    // generation g + 2 as soon as all scores of generation g - 1 are out.  By then every workgroup
    // has built its term table of generation g - 1, hence has long read the draw of generation
    // g - 2, whose buffer the new one takes (four rotate).
    for (uint32_t g = 0; g < 3 && g < fa.n_generations; ++g) publish_draw(a.t + g + 1, fa.draws_before + g);
    for (uint32_t g = 1; g + 2 < fa.n_generations; ++g) {
      const uint32_t use = fa.generations_before + g - 1;
      const uint64_t *xk = fa.xkeys + static_cast<size_t>(use & 1u) * P + K;
      const bool seen = gather(3 * K, fa.spin_limit, [&](uint32_t i) { return xk + i; },
                               [&](uint32_t, uint64_t v) { return (v & kTagBit) == use_tag(use); }, [&](uint32_t, uint64_t) {});
      if (__syncthreads_or(seen ? 0 : 1)) return give_up();
      publish_draw(a.t + g + 3, fa.draws_before + g + 2);
    }
    return;
  }
  draw_unit_parents(a.t + 1);
  stage_table<1>(a, s, a.term_lds, fa.first_changed != 0, threadIdx.x, blockDim.x);
  // the state the last selection left: the survivors' rows and scores, the rows of the units (the
  // ranking only moves the rows)
  for (uint32_t e = tid; e < K; e += kFusedThreads) {
    const uint32_t row = checked_row(fa.parent_rows[e], P + K);
    rk.srow(0)[e] = static_cast<uint16_t>(row);
    rk.skey(0)[e] = static_cast<uint64_t>(__double_as_longlong(a.fit_row[row]));
    if (a.assigned) rk.frow[3 * K + e] = static_cast<uint16_t>(checked_row(a.spare[e], P + K));
  }
  if (a.assigned)
    for (uint32_t u = tid; u < 3 * K; u += kFusedThreads) rk.frow[u] = static_cast<uint16_t>(checked_row(a.row_of[K + u], P + K));
  if (tid < 4) rk.misc[tid] = 0;
  if (kSampled && tid < kLanes) {
    rk.model[tid] = a.tab.abl[tid];
    rk.model[kLanes + tid] = a.tab.cc[tid];
    rk.model[2 * kLanes + tid] = a.tab.d[tid];
    rk.blexp[tid] = info_blexp(a.tab.info[tid]);
  }
  __syncthreads();
  draw_unit_words(a.t + 1);
  if (!a.assigned) list_free_rows(rk, rk.srow(0), P);
  if (kSampled) {
    const bool got = collect_draw(fa.draws_before);
    if (__syncthreads_or(got ? 0 : 1)) return give_up();
    build_terms();
  }

  int cur = 0;
  for (uint32_t g = 0; g < fa.n_generations; ++g) {
    const uint32_t t = a.t + g + 1;
    const bool changed = g == 0 && fa.first_changed != 0;
    const bool new_first = changed && a.new_first != 0;
    const bool last = g + 1 == fa.n_generations;
    const bool all_new = changed || kSampled;                   // every candidate of the pool gets a new score
    const uint32_t units = all_new ? 4 * K : 3 * K;
    const uint32_t use = fa.generations_before + g;             // how often the children's exchange buffers have been used
    const uint32_t surv_use = fa.changes_before + (kSampled ? g : 0u);   // ... uses of the survivors' exchange buffers
    uint64_t *xk = fa.xkeys + static_cast<size_t>(use & 1u) * P;
    uint64_t *xs = fa.xsurv + static_cast<size_t>(surv_use & 1u) * K;
    // ---- compose, repair, score and store this wave's candidates (at most kFusedUnits of them)
    for (uint32_t k = 0, u; (u = unit_of(k)) < units; ++k) {
      const int lane = opaque(lane0);
      uint32_t c[1], row;
      double f;
      if (kSampled && !changed && u >= 3 * K) {
        // the survivor of rank u - 3K keeps genome and row; only its score changes with the draw
        row = rk.srow(cur)[u - 3 * K];
        c[0] = shared_load(a.genes + static_cast<size_t>(row) * kLanes + lane);
        f = score<1, 1>(c, s, a.term_lds, lane);
      } else {
        f = changed ? compose_unit<false, kOverGpus>(a, t, s, rk.srow(cur), u, new_first, coins, my_draws + 4 * k,
                                                     my_words + kLanes * k, lane, c)
                    : compose_unit<true, kOverGpus>(a, t, s, rk.srow(cur), u, false, coins, my_draws + 4 * k,
                                                    my_words + kLanes * k, lane, c);
        row = rk.frow[u];
        shared_store(a.genes + static_cast<size_t>(row) * kLanes + lane, c[0]);
      }
      if (lane == 0) {
        const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(f));
        my_keys[k] = bits;
        // the scores kept with the rows are only looked at after the call (to the point of coherence
        // like the rest: a plain store could linger in one XCD's cache)
        if (last) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + row, bits);
      }
    }
    // the genomes have arrived before their scores are published
    phase_fence();
    __builtin_amdgcn_s_waitcnt(0);
    phase_fence();
    if (lane0 == 0)
      for (uint32_t k = 0, u; (u = unit_of(k)) < units; ++k) {
        if (u < 3 * K) shared_store(xk + K + u, my_keys[k] | use_tag(use));
        else shared_store(xs + (u - 3 * K), my_keys[k] | use_tag(surv_use));
      }
    if (!last) {                                     // while the others' scores are on their way
      draw_unit_parents(t + 1);
      draw_unit_words(t + 1);
    }
    bool drawn = true;                               // the draw of the next generation has been out for a while
    if (kSampled && !last) drawn = collect_draw(fa.draws_before + g + 1);

    // ---- collect the scores (children and mutants i < 3K, then, when every score is new, the
    // survivors); a child that beats the K-th survivor raises a flag (an equal score loses to the
    // survivor's smaller slot).  The flags of three generations rotate, so that the next one's can be
    // cleared before the barrier: every wave is past the barrier before, hence past the use of the
    // flag of two generations ago.
    const uint64_t thresh = all_new ? 0ull : rk.skey(cur)[K - 1];
    if (crowd) { if (all_new) __builtin_amdgcn_s_sleep(48); else __builtin_amdgcn_s_sleep(8); }
    const bool ok = gather(all_new ? P : 3 * K, fa.spin_limit,
                           [&](uint32_t i) { return i < 3 * K ? xk + K + i : xs + (i - 3 * K); },
                           [&](uint32_t i, uint64_t v) { return (v & kTagBit) == (i < 3 * K ? use_tag(use) : use_tag(surv_use)); },
                           [&](uint32_t i, uint64_t v) {
                             const uint64_t key = v & ~kTagBit;
                             rk.ckey[i < 3 * K ? K + i : i - 3 * K] = key;
                             if (key < thresh) rk.misc[1 + g % 3] = 1;
                           });
    if (tid == 0) rk.misc[0] = rk.misc[1 + (g + 1) % 3] = 0;
    if (__syncthreads_or(ok && drawn ? 0 : 1)) return give_up();
    const bool any = rk.misc[1 + g % 3] != 0;

    // every wave of this workgroup is done with the term table of this generation: the next one's
    if (kSampled && !last) build_terms();

    // ---- rank the pool
    int nxt = cur ^ 1;
    bool whole = all_new;                            // rank the whole pool, a share per workgroup
    if (!all_new && !any) {
      // no child beats the K-th survivor: same survivors, same order, same rows
      if (last && blockIdx.x != 0) return;
      nxt = cur;
      if (last) for (uint32_t e = tid; e < K; e += kFusedThreads) rk.nsel[e] = static_cast<uint16_t>(e);
    } else if (!all_new) {
      // list the children that beat the K-th survivor
      for (uint32_t base = 0; base < 3 * K; base += kFusedThreads) {   // whole waves go round together
        const uint32_t i = base + tid;
        const uint64_t key = i < 3 * K ? rk.ckey[K + i] : ~0ull;
        const bool beats = key < thresh;
        const uint64_t mask = __ballot(beats);
        uint32_t at = 0;
        if (lane0 == 0 && mask != 0) at = atomicAdd(&rk.misc[0], static_cast<uint32_t>(__popcll(mask)));
        at = __builtin_amdgcn_readfirstlane(at) + static_cast<uint32_t>(__popcll(mask & ((1ull << lane0) - 1ull)));
        if (beats) { rk.lkey[at] = key; rk.lslot[at] = static_cast<uint16_t>(K + i); }
      }
      __syncthreads();
      const uint32_t M = rk.misc[0];
      // in the last generation only the first workgroup needs the ranking (it writes the state the
      // call leaves); the others stay for their share of a ranking by counting, if there is one
      if (last && blockIdx.x != 0 && M <= kMergeMax) return;
      if (M > kMergeMax) {
        whole = true;
        for (uint32_t e = tid; e < K; e += kFusedThreads) rk.ckey[e] = rk.skey(cur)[e];
      } else {
        // rank of each such child among them, the comparisons dealt to all threads
        const uint32_t Mp = pow2_at_least(M), parts = kFusedThreads / Mp, per = (M + parts - 1) / parts;
        if (tid < kMergeMax) rk.below[tid] = 0;
        __syncthreads();
        {
          const uint32_t i = tid % Mp, from = (tid / Mp) * per, to = min(from + per, M);
          if (i < M) {
            const uint64_t key = rk.lkey[i];
            const uint32_t slot = rk.lslot[i];
            uint32_t n = 0;
            for (uint32_t j = from; j < to; ++j) n += key_less(rk.lkey[j], rk.lslot[j], key, slot) ? 1u : 0u;
            if (n) atomicAdd(&rk.below[i], n);
          }
        }
        __syncthreads();
        if (tid < M) { rk.okey[rk.below[tid]] = rk.lkey[tid]; rk.oslot[rk.below[tid]] = rk.lslot[tid]; }
        __syncthreads();
        // child at position b: new rank = b + survivors with a score <= its own; its slot takes the
        // row of the last survivor but b, which drops out
        if (tid < M) {
          const uint64_t key = rk.okey[tid];
          uint32_t lo = 0, hi = K;
          while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (rk.skey(cur)[mid] <= key) lo = mid + 1; else hi = mid;
          }
          const uint32_t rank = tid + lo, u = rk.oslot[tid] - K;
          if (rank < K) {
            rk.skey(nxt)[rank] = key;
            rk.srow(nxt)[rank] = rk.frow[u];
            rk.nsel[rank] = rk.oslot[tid];
            rk.frow[u] = rk.srow(cur)[K - 1 - tid];
          }
        }
        // survivor e: new rank = e + such children with a strictly smaller score
        for (uint32_t e = tid; e < K; e += kFusedThreads) {
          const uint64_t key = rk.skey(cur)[e];
          uint32_t lo = 0, hi = M;
          while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (rk.okey[mid] < key) lo = mid + 1; else hi = mid;
          }
          const uint32_t rank = e + lo;
          if (rank < K) {
            rk.skey(nxt)[rank] = key;
            rk.srow(nxt)[rank] = rk.srow(cur)[e];
            rk.nsel[rank] = static_cast<uint16_t>(e);
          }
        }
      }
    }
    if (whole) {
      // ckey holds the whole pool's scores by slot.  This workgroup ranks its share of the slots
      // (rank = candidates below in (score, slot) order), publishes the ranks, collects all.
      // (Ranking all of them in every workgroup's LDS, by a sample sort there, takes 15 to 25 us at 2048
      // candidates where this takes 5: equal scores of neighbouring slots queue up on its counters.)
      const uint32_t lo = static_cast<uint32_t>(static_cast<uint64_t>(P) * blockIdx.x / n_groups);
      const uint32_t hi = static_cast<uint32_t>(static_cast<uint64_t>(P) * (blockIdx.x + 1) / n_groups);
      const uint32_t ns = hi - lo, parts = ns ? kFusedThreads / ns : 0u;   // 0 < parts: ns <= kMergeMax
      if (tid < kMergeMax) rk.below[tid] = 0;
      __syncthreads();
      if (ns != 0 && tid < parts * ns) {
        // thread (i, part): slot lo + i against the candidates part, part + parts, ...; candidate j is
        // below when its score is smaller, or equal with a smaller slot, i.e. smaller than the
        // score + 1 for j < slot (scores are integers below 2^63 here)
        const uint32_t i = tid % ns, part = tid / ns, slot = lo + i;
        const uint64_t key = rk.ckey[slot];
        uint32_t n = 0;
        uint32_t j = part;
        for (; j + 3 * parts < P; j += 4 * parts) {
          const uint64_t k0 = rk.ckey[j], k1 = rk.ckey[j + parts], k2 = rk.ckey[j + 2 * parts], k3 = rk.ckey[j + 3 * parts];
          n += k0 < key + (j < slot ? 1u : 0u) ? 1u : 0u;
          n += k1 < key + (j + parts < slot ? 1u : 0u) ? 1u : 0u;
          n += k2 < key + (j + 2 * parts < slot ? 1u : 0u) ? 1u : 0u;
          n += k3 < key + (j + 3 * parts < slot ? 1u : 0u) ? 1u : 0u;
        }
        for (; j < P; j += parts) n += rk.ckey[j] < key + (j < slot ? 1u : 0u) ? 1u : 0u;
        if (n) atomicAdd(&rk.below[i], n);
      }
      __syncthreads();
      const uint64_t stamp = static_cast<uint64_t>(use + 1u) << 32;     // no generation has number 0
      if (tid < ns) shared_store(fa.xrank + lo + tid, stamp | rk.below[tid]);
      if (last && blockIdx.x != 0) return;
      if (crowd) __builtin_amdgcn_s_sleep(16);
      const bool ranked = gather(P, fa.spin_limit, [&](uint32_t p) { return fa.xrank + p; },
                                 [&](uint32_t, uint64_t v) { return (v >> 32) == (stamp >> 32); },
                                 [&](uint32_t p, uint64_t v) {
                                   const uint32_t rank = static_cast<uint32_t>(v);
                                   if (rank < K) {
                                     rk.skey(nxt)[rank] = rk.ckey[p];
                                     rk.nsel[rank] = static_cast<uint16_t>(p);
                                   }
                                 });
      if (__syncthreads_or(ranked ? 0 : 1)) return give_up();
      assign_rows(rk, P, cur, nxt, changed);
    } else if (any) {
      __syncthreads();
    }
    if (last) {
      // the state the next call (of either kind) starts from.  (A call runs more than one generation,
      // so the last one is never the first under a new table: the pool's first K slots are survivors.)
      for (uint32_t e = tid; e < K; e += kFusedThreads) {
        const uint32_t row = rk.srow(cur)[e];
        a.row_of[e] = row;
        if (!all_new) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + row, rk.skey(cur)[e]);
        fa.parent_rows[e] = rk.srow(nxt)[e];
        fa.sel[e] = rk.nsel[e];
        a.spare[e] = rk.frow[3 * K + e];
      }
      for (uint32_t u = tid; u < 3 * K; u += kFusedThreads) a.row_of[K + u] = rk.frow[u];
      if (kSampled && tid < kLanes) fa.y_out[tid] = rk.ydraw[tid];   // the remaining work the last generation was scored with
      // the other workgroups have published their last and leave, or have left; the argument block is read here, see kernel_args
      const auto *late = (const __attribute__((address_space(4))) FusedArgs *)kernel_args();
      publish_winner(late->winner, a.genes, kLanes, rk.srow(nxt)[0], a.tab.info, rk.skey(nxt)[0]);
      all_arrived();
      if (tid == 0) signal_call_done(late->winner, late->sync + 1);
      return;
    }
    cur = nxt;
  }
}

size_t table_lds_bytes(const EvolveArgs &ev) {
  return (smem_bytes(1, kFusedWaves, ev.term_lds, ev.P + ev.K, ev.coin_stride) + 15) & ~size_t(15);
}

}  // namespace

uint32_t fused_workgroups(uint32_t P, bool sampled) {
  // one wave per candidate a generation computes: the 3K children, and under probability sampling the K survivors too
  const uint32_t units = (sampled ? 4 : 3) * (P / 4);
  return std::max(1u, std::min(sampled ? kFusedMaxSampledWorkgroups : kFusedMaxWorkgroups, (units + kFusedWaves - 1) / kFusedWaves));
}

uint32_t fused_grid_limit(uint32_t P) {
  return std::max(fused_workgroups(P, false), fused_workgroups(P, true) + kDrawGroups);
}

size_t fused_exchange_bytes(uint32_t P) {             // xkeys [2][P], xsurv [2][K], xrank [P], xdraw [4][64]; zeroed once
  return (static_cast<size_t>(2) * P + 2 * (P / 4) + P + kDrawBuffers * kLanes) * 8;
}

void fused_exchange(uint64_t *base, uint32_t P, FusedArgs &fa) {
  fa.xkeys = base;
  fa.xsurv = fa.xkeys + static_cast<size_t>(2) * P;
  fa.xrank = fa.xsurv + static_cast<size_t>(2) * (P / 4);
  fa.xdraw = fa.xrank + P;
}

hipError_t launch_fused(const FusedArgs &args, hipStream_t stream) {
  FusedArgs fa = args;
  if (fa.ev.Jp != static_cast<uint32_t>(kLanes) || fa.ev.P > kFusedMaxPool || fa.ev.P < 4 || fa.n_generations < 2)
    return hipErrorInvalidValue;
  const uint32_t n_wg = fused_workgroups(fa.ev.P, fa.sampled != 0);
  // every wave keeps its units of a generation in LDS, and a workgroup's share of a ranking by counting fits its counters
  if ((fa.ev.P + n_wg * kFusedWaves - 1) / (n_wg * kFusedWaves) > kFusedUnits || (fa.ev.P + n_wg - 1) / n_wg > kMergeMax)
    return hipErrorInvalidValue;
  fa.ev.bk.nb = 0;
  fa.ev.coin_stride = coin_stride(fa.ev);
  fa.ev.term_lds = fa.ev.tab.term_E;                  // 64 job columns: the term table always fits
  fa.table_lds = static_cast<uint32_t>(table_lds_bytes(fa.ev));
  const size_t lds = fa.table_lds + ranks_bytes(fa.ev.P);
  if (lds > kLdsBudget) return hipErrorInvalidValue;
  const void *fn = fa.sampled ? (fa.ev.per_gpu ? reinterpret_cast<const void *>(fused_kernel<true, true>)
                                               : reinterpret_cast<const void *>(fused_kernel<false, true>))
                              : (fa.ev.per_gpu ? reinterpret_cast<const void *>(fused_kernel<true, false>)
                                               : reinterpret_cast<const void *>(fused_kernel<false, false>));
  hipError_t rc = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (rc != hipSuccess) return rc;
  fa.work_groups = n_wg;
  const uint32_t grid = n_wg + (fa.sampled ? kDrawGroups : 0u);
  void *params[] = {&fa};
  // For tools that cannot follow a cooperative launch (rocprofv3's kernel trace ends in a fault when
  // the process exits after one): the same kernel as an ordinary launch.  Its waits stay bounded,
  // but nothing then guarantees that all workgroups are resident at once, so this is not for production.
  static const bool plain = getenv("ONES_FUSED_PLAIN_LAUNCH") != nullptr;
  if (plain) return hipLaunchKernel(fn, dim3(grid), dim3(kFusedThreads), params, lds, stream);
  // cooperative: the runtime refuses the launch unless all workgroups can be resident at once
  return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kFusedThreads), params, static_cast<unsigned int>(lds), stream);
}

}  // namespace ones
