// All generations of one ones_generation call in a single launch (ONES, arXiv 2108.03645, Section 3.2.2), for
// pools of some thousand candidates beyond those of ones_fused.hip: up to kResidentMaxPool candidates of up to
// 64 * 4 * kResidentMaxWords job slots, as far as a workgroup's LDS holds the job table and the ranking.
//
// The protocol is that of ones_fused.hip: a co-resident grid, one workgroup to a compute unit, stays on the chip
// for the whole call; its waves compose, repair and score the workgroup's share of the 3K children (4K candidates
// when every score is new) and publish genomes and scores, and every workgroup ranks the pool by itself in its LDS,
// so that one exchange separates two generations.  (Two launches a generation, the other way to do this, spend
// more on their boundaries, on staging the job table and on looking rows and scores up through memory than on the
// candidates: a pool of 8192 on 200 slots 15 us a generation, of which 2.5 compute.)
// What differs is the size: hundreds to thousands of children beat the K-th survivor of such a pool in every
// generation, too many to count against each other, and the scores of all are too much for every workgroup to read.
// A workgroup publishes those children in a list of its own, score, slot and row, with their number beside its
// flag.  The survivors are in order, so such a child finds its place among them by binary search; the children of
// each place are counted, the counts summed up, and the few children that share a place ranked among themselves.
// Only where many share one (a pool full of copies of one genome), where more children than the list holds beat the
// K-th survivor, or where every score is new, do the workgroups read the scores of all, rank a share of the pool
// each, by counting, and exchange the order in a second step.
#include "ones_candidate.h"
#include "ones_exchange.h"
#include "ones_sort.h"

#include <cstddef>
#include <cstdlib>

#ifndef ONES_RESIDENT_WORDS
#error "compile with -DONES_RESIDENT_WORDS=1..4"
#endif

namespace ones {
namespace {

constexpr int kResWaves = 16;
constexpr int kResThreads = kResWaves * kLanes;
constexpr uint32_t kResPlace = 128;          // children that share a place among the survivors, at most (an epoch of 16384 candidates on
                                             // 512 jobs, 50 generations: 1136 us, with 320 of them 1192, with 64 no difference)
constexpr uint32_t kResSample = 256;         // sample points of a pool that is ranked as a whole
constexpr uint32_t kResFirst = 128;          // ... those of them that are ranked first
constexpr uint32_t kResBound = kResFirst / 4 + 24;     // ... of which the one of this rank bounds what can survive: the K-th is a quarter
                                                       // of the way up, so at rank 32 of the 128 on average, with a deviation of 4.9
constexpr uint32_t kResLocal = 256;          // a pool of so few is ranked by every workgroup by itself
constexpr uint32_t kResInside = kResThreads / 4 * 3;   // candidates of a range that are counted against each other at once: of 16384 candidates a
                                                       // range holds 64 on average, and more than so many once in 2500 rankings
constexpr int kResListed = 3;                // listed children a thread handles, at most
[[maybe_unused]] constexpr uint32_t kResList = kResListed * kResThreads;
constexpr uint32_t kResLeastList = 2 * kResInside;        // children that the list holds at least
constexpr int kResElites = kResidentMaxPool / 4 / kResThreads;           // survivors a thread handles, at most
constexpr int kResPool = kResidentMaxPool / kResThreads;
[[maybe_unused]] constexpr size_t kResLds = kLdsBudget - 512;   // what is left beside the 256 bytes that the or over a workgroup takes
static_assert(kResidentMaxPool % (4 * kResThreads) == 0, "whole numbers of survivors and candidates per thread");
static_assert(kResidentMaxPool <= 1 << 14, "a slot and a row in 32 bits");
static_assert(kResLocal <= kResInside && kResSample <= kResInside, "one set of counters, one set of records");
static_assert(kResInside * sizeof(uint4) <= kResLeastList * 8, "records fit in the list's place");
static_assert(kResidentMaxGroups <= static_cast<uint32_t>(kResThreads), "a thread per workgroup's flag");

// ----------------------------------------------------------------- LDS -------------
struct Ranking {
  uint64_t *ckey;    // [K] score bits of the survivors, best first
  uint64_t *sample;  // [kResSample] score bits of the sample points
  uint64_t *lkey;    // [list] score bits of the listed children
  uint32_t *place;   // [max(K, kResInside)] children at each place, then their running sum; zero between uses
  uint32_t *range;   // [4] the sample point that bounds what can survive, sample points below it, candidates below and
                     // inside this workgroup's range
  uint32_t *bits;    // bitmap: over the P + K rows when rows are listed, over the survivors of the generation before
  uint32_t *wcount;  // [64] counts of the waves, for prefix sums
  uint32_t *misc;    // [1] whether a place is crowded, [2] items that waves have taken, [3] children this workgroup lists
  uint32_t *nsel;    // [kResLocal / 4] slot and row of the new survivors of a pool that every workgroup ranks by itself
  uint32_t *from;    // [workgroups] listed children of the workgroups before each
  uint32_t *draws;   // [child items][3] ranks of the parents, starts of the repairs (drawn ahead)
  uint32_t *words;   // [child items][Q * 64] what the item draws per gene (see draw_genes)
  uint16_t *lslot;   // [list] slots of the children in lkey
  uint16_t *order;   // [list] the workgroups that list them; the listed children in the order of their places; slots of sample points
  uint16_t *srow;    // [K] genome rows of the survivors
  uint16_t *rows;    // [child items][2] the rows this workgroup's children go to
  // in another's place:
  uint16_t *spare;   // [K] in ckey's, until the generation after a table change is ranked: rows of the refreshed survivors
  uint4    *records; // [kResInside] in lkey's, while the pool is ranked as a whole: score bits and slots, of sample points, then
                     // of the candidates of this workgroup's range
  uint16_t *drow;    // [K] ... and, once it is ranked: rows of survivors that dropped out
};

[[maybe_unused]] inline size_t ranking_bytes(uint32_t Q, uint32_t P, const ResidentPlan &plan) {
  const size_t K = P / 4, words = (P + K + 31) / 32;
  return 8 * (K + kResSample + std::max<size_t>(plan.list, (K + 3) / 4)) +
         4 * (std::max<size_t>(K, kResInside) + 4 + words + 64 + 4 + kResLocal / 4 + plan.groups +
              static_cast<size_t>(plan.child_items) * (3 + Q * kLanes)) +
         2 * (2 * static_cast<size_t>(plan.list) + K + 2 * plan.child_items) + 16;
}

__device__ __forceinline__ Ranking carve_ranking(unsigned char *base, uint32_t Q, uint32_t P, uint32_t groups, uint32_t list,
                                                 uint32_t child_items) {
  const uint32_t K = P / 4, words = (P + K + 31) / 32;
  Ranking r;
  r.lkey = reinterpret_cast<uint64_t *>(base);
  r.sample = r.lkey + max(list, (K + 3) / 4);
  r.ckey = r.sample + kResSample;
  r.place = reinterpret_cast<uint32_t *>(r.ckey + K);
  r.range = r.place + max(K, kResInside);
  r.bits = r.range + 4;
  r.wcount = r.bits + words;
  r.misc = r.wcount + 64;
  r.nsel = r.misc + 4;
  r.from = r.nsel + kResLocal / 4;
  r.draws = r.from + groups;
  r.words = r.draws + 3 * child_items;
  r.lslot = reinterpret_cast<uint16_t *>(r.words + child_items * Q * kLanes);
  r.order = r.lslot + list;
  r.srow = r.order + list;
  r.rows = r.srow + K;
  r.spare = reinterpret_cast<uint16_t *>(r.ckey);
  r.records = reinterpret_cast<uint4 *>(r.lkey);
  r.drow = reinterpret_cast<uint16_t *>(r.lkey);
  return r;
}

// The job table in LDS without what only the kernels of one generation need.
[[maybe_unused]] inline size_t table_bytes(uint32_t Q, uint32_t E, uint32_t stride, bool walk) {
  const size_t words = static_cast<size_t>(Q) * kLanes;
  return words * (4 * 8 * static_cast<size_t>(E) + 8 + 8 + 7 * 4) + (walk ? walk_table_bytes(Q) : 0) + static_cast<size_t>(kResWaves) * stride;
}
template <int Q>
__device__ __forceinline__ Smem carve_table(unsigned char *at, uint32_t E, bool walk) {
  constexpr uint32_t kWords = Q * kLanes;
  Smem s{};
  s.terms = reinterpret_cast<double *>(at);
  s.rank = reinterpret_cast<uint2 *>(s.terms + static_cast<size_t>(4 * kWords) * E);
  s.prefix = s.rank + kWords;
  s.start = reinterpret_cast<uint32_t *>(s.prefix + kWords);
  s.most = s.start + kWords;
  s.draws = s.most + kWords;
  s.lift = s.draws + kWords;
  s.shift = s.lift + kWords;
  s.fresh = s.shift + kWords;
  s.bl = s.fresh + kWords;
  s.start_at = reinterpret_cast<uint8_t *>(s.bl + kWords);
  s.most_at = s.start_at + 4 * kWords + kWindowAhead;
  s.coins = s.start_at + (walk ? walk_table_bytes(Q) : 0);
  return s;
}

// ----------------------------------------------------------------- work items ------
// How the candidates are dealt to the workgroups.  A wave takes an item at a time: a child of a pair or a mutant, or, in
// a pool of more of those than there are waves, a pair (its two children share what they draw) or a mutant; behind
// them, where every score is new, a survivor.  Item i is item i / groups of workgroup i mod groups.
struct Deal {
  uint32_t K, groups, me, paired, children;          // children: items that are no survivors
  __device__ __forceinline__ uint32_t first_slot(uint32_t i) const { return !paired ? K + i : i < K ? K + 2 * i : 2 * K + i; }
  __device__ __forceinline__ bool both(uint32_t i) const { return paired && i < K; }
  __device__ __forceinline__ uint32_t mine(uint32_t n) const { return n > me ? (n - me + groups - 1) / groups : 0u; }
  // place among the rows of its workgroup's children that the child in `slot` has, ~0 if it is another's
  __device__ __forceinline__ uint32_t own(uint32_t slot) const {
    const uint32_t u = slot - K, i = !paired ? u : u < 2 * K ? u / 2 : u - K;
    return i % groups != me ? ~0u : i / groups * 2 + (paired && u < 2 * K ? u % 2 : 0u);
  }
};

// What a child or mutant draws before it needs anything of its parents depends on (seed, generation, slot)
// only, so a workgroup draws for the coming generation while the scores of the current one are still arriving.
// A word per four genes: for a child of a pair 0xFF where the pair's genes are swapped; for a mutant 0x80 and the
// new code where a gene is redrawn.
template <int Q, bool kOverGpus>
__device__ __forceinline__ void draw_genes(const EvolveArgs &a, const Smem &s, uint32_t t, uint32_t p, bool both, int lane,
                                           uint32_t *draws, uint32_t *words) {
  const uint32_t K = a.K, R = a.Jp / kLanes;
  const bool child = p < 3 * K;
  const uint32_t p0 = child ? p - ((p - K) & 1u) : p;            // a pair shares what is drawn for its first slot, but for
  const Draw d = candidate_draw(a, t, lane == 0 ? p0 : both ? p + 1 : p);        // the rotations
  if (lane == 0) draws[0] = d.ra | d.rb << 16;
  if (lane < 2) draws[1 + lane] = d.r / R | d.r % R << 16;       // without a pair only the latter counts
  if (child && kOverGpus) return;
  const WordSource source(a, t, p0, Q > 1);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const Words w = source.block(s.prefix, q, lane);
    uint32_t out;
    if (child) {
      out = words_below(w, a.T_x);
    } else {
      const uint32_t k = outcomes_drawn(w, s.draws[q * kLanes + lane]), redrawn = words_below(w, a.T_mut);
      out = redrawn & (codes_of_draws(s, q * kLanes + lane, k) | kTops);
    }
    words[q * kLanes + lane] = out;
    phase_fence();
  }
}

template <int Q>
__device__ __forceinline__ void load_shared_genes(const uint32_t *genes, uint32_t row, int lane, uint32_t (&c)[Q]) {
  const uint32_t *at = genes + static_cast<size_t>(row) * (Q * kLanes) + lane;
#pragma unroll
  for (int q = 0; q < Q; ++q) c[q] = shared_load(at + q * kLanes);
}

// One item of generation t: composed, repaired and scored, its genomes stored; done(slot, which child of the item, row,
// score) takes note of each candidate.  rows: of the item's children.
template <int Q, Genes kGenes, bool kOverGpus, bool kSameTable, bool kWalk, typename Done>
__device__ __forceinline__ void compose_item(const EvolveArgs &a, uint32_t t, const Smem &s, const Ranking &rk, const Deal &deal, uint32_t i,
                                             bool new_first, uint64_t *coins, const uint32_t *draws, const uint32_t *words,
                                             const uint16_t *rows, int lane, Done done) {
  const uint32_t K = a.K;
  uint32_t c[Q], other[Q], slot, start, row;
  bool both = false;
  if (i < deal.children) {
    slot = deal.first_slot(i);
    both = deal.both(i);
    const uint32_t parents = __builtin_amdgcn_readfirstlane(draws[0]);
    start = __builtin_amdgcn_readfirstlane(draws[both ? 1 : 2]);
    row = __builtin_amdgcn_readfirstlane(rows[0]);
    load_shared_genes<Q>(a.genes, __builtin_amdgcn_readfirstlane(rk.srow[parents & 0xFFFFu]), lane, c);
    if (slot < 3 * K) {
      load_shared_genes<Q>(a.genes, __builtin_amdgcn_readfirstlane(rk.srow[parents >> 16]), lane, other);
      const bool second = !both && ((slot - K) & 1u) != 0;
      if (kOverGpus) {
        if (!kSameTable) { to_new_table<Q>(s, lane, c); to_new_table<Q>(s, lane, other); }
        phase_fence();
        crossover_over_gpus<Q, kSameTable>(a, t, s, coins, slot - ((slot - K) & 1u), lane, c, other);
#pragma unroll
        for (int q = 0; q < Q; ++q) c[q] = second ? other[q] : c[q];
      } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t drawn = words[q * kLanes + lane], swap = second ? ~drawn : drawn, mine = c[q];
          c[q] = pick(swap, other[q], mine);
          other[q] = pick(swap, mine, other[q]);
        }
        if (!kSameTable) { to_new_table<Q>(s, lane, c); to_new_table<Q>(s, lane, other); }
      }
    } else {
      if (!kSameTable) to_new_table<Q>(s, lane, c);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t drawn = words[q * kLanes + lane], redrawn = spread_tops(drawn);
        c[q] = pick(redrawn, drawn & kSevens, c[q]);
      }
    }
  } else {                                           // only after a table change: the survivor of rank i - children
    slot = i - deal.children;
    const uint32_t R = a.Jp / kLanes, r = __builtin_amdgcn_readfirstlane(candidate_draw(a, t, slot).r);
    start = r / R | r % R << 16;
    row = __builtin_amdgcn_readfirstlane(rk.spare[slot]);
    load_shared_genes<Q>(a.genes, __builtin_amdgcn_readfirstlane(rk.srow[slot]), lane, c);
    to_new_table<Q>(s, lane, c);
  }
  for (uint32_t which = 0;; ++which) {
    phase_fence();
    const uint32_t lr = start & 0xFFFFu, ir = start >> 16;
    uint8_t *window = reinterpret_cast<uint8_t *>(coins);
    if (!kSameTable && new_first) repair<Q, kGenes, true>(c, s, a.G, lr, ir, lane, a.Jp, a.time_rank != nullptr, window, kWalk);
    else repair<Q, kGenes, false>(c, s, a.G, lr, ir, lane, a.Jp, false, window, kWalk);
    phase_fence();
    const double f = score<Q>(c, s, a.term_lds, lane);
    uint32_t *at = a.genes + static_cast<size_t>(row) * (Q * kLanes) + lane;
#pragma unroll
    for (int q = 0; q < Q; ++q) shared_store(at + q * kLanes, c[q]);
    done(slot + which, which, row, f);
    if (!both || which == 1) break;
    start = __builtin_amdgcn_readfirstlane(draws[2]);
    row = __builtin_amdgcn_readfirstlane(rows[1]);
#pragma unroll
    for (int q = 0; q < Q; ++q) c[q] = other[q];
  }
}

// ----------------------------------------------------------------- exchange --------
// Waits until the workgroups' flags show generation number `want`: a thread per workgroup polls, and takes the count that
// came with the flag.  False when the polls ran out.
__device__ __forceinline__ bool wait_for_all(const uint64_t *flags, uint32_t n, uint32_t want, uint32_t spin_limit, uint32_t &count) {
  count = 0;
  if (threadIdx.x / kLanes * kLanes >= n) return true;           // whole waves without a flag to look at
  const uint64_t *mine = flags + min(threadIdx.x, n - 1);
  for (uint32_t spins = 0; spins < spin_limit; ++spins) {
    const uint64_t v = shared_load(mine);
    if (__ballot(static_cast<uint32_t>(v >> 32) != want) == 0) {
      if (threadIdx.x < n) count = static_cast<uint32_t>(v);
      return true;
    }
  }
  return false;
}

// x, y: before the call this thread's counts, after it those of the threads before it; and the totals.  With one barrier.
__device__ __forceinline__ void sums_before(const Ranking &rk, uint32_t &x, uint32_t &y, uint32_t &total_x, uint32_t &total_y) {
  static_assert(2 * kResWaves <= kLanes, "a lane per count");
  const uint32_t lane = threadIdx.x % kLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const uint32_t ix = wave_inclusive_scan(x), iy = wave_inclusive_scan(y);
  if (lane == kLanes - 1) { rk.wcount[wave] = ix; rk.wcount[kResWaves + wave] = iy; }
  __syncthreads();
  const uint32_t n = lane < 2 * kResWaves ? rk.wcount[lane] : 0u, upto = wave_inclusive_scan(n);
  total_x = __builtin_amdgcn_readlane(upto, kResWaves - 1);
  total_y = __builtin_amdgcn_readlane(upto, 2 * kResWaves - 1) - total_x;
  x = __builtin_amdgcn_readlane(upto - n, wave) + ix - x;
  y = __builtin_amdgcn_readlane(upto - n, kResWaves + wave) - total_x + iy - y;
}

// ----------------------------------------------------------------- rows ------------
// The rows that are not the survivors', in ascending order, as rows of the children and then of the refreshed
// survivors, when no selection has assigned them.  rk.bits is zero before and after.  Whole workgroup; ends with a barrier.
__device__ __forceinline__ void list_free_rows(const Ranking &rk, const Deal &deal, uint32_t P, bool changed, uint32_t *spare) {
  const uint32_t K = P / 4, n_rows = P + K, words = (n_rows + 31) / 32;
  static_assert((kResidentMaxPool + kResidentMaxPool / 4) / 32 <= kResThreads, "a thread per word of the bitmap");
  for (uint32_t g = threadIdx.x; g < K; g += kResThreads) atomicOr(&rk.bits[rk.srow[g] >> 5], 1u << (rk.srow[g] & 31u));
  __syncthreads();
  uint32_t free_bits = threadIdx.x < words ? ~rk.bits[threadIdx.x] : 0u;
  if (threadIdx.x + 1 == words && n_rows % 32 != 0) free_bits &= (1u << (n_rows % 32)) - 1u;
  uint32_t at = __popc(free_bits), unused = 0, total, total_unused;
  sums_before(rk, at, unused, total, total_unused);
  while (free_bits) {
    const uint32_t row = threadIdx.x * 32 + (__ffs(static_cast<int>(free_bits)) - 1);
    if (at < 3 * K) {
      const uint32_t own = deal.own(K + at);
      if (own != ~0u) rk.rows[own] = static_cast<uint16_t>(row);
    } else if (at < P) {
      if (changed) rk.spare[at - 3 * K] = static_cast<uint16_t>(row);
      else if (deal.me == 0) shared_store(spare + (at - 3 * K), row);
    }
    free_bits &= free_bits - 1;
    ++at;
  }
  if (threadIdx.x < words) rk.bits[threadIdx.x] = 0;
  __syncthreads();
}

// The scores and rows that go with a ranking of the whole pool.  entry[k]: slot and, above it, row of the new survivor of
// rank threadIdx.x + k * kResThreads.  The new survivors keep their rows, and the slots of the surviving children
// take the rows of the survivors that dropped out, the i-th the i-th (both counted in the same order by every
// workgroup).  changed: the pool's first K slots are refreshed survivors in the spare rows, and the rows they came from are
// spare from now on.  score(slot): the score of the pool's slot.  rk.bits is zero before and after.  Ends with a barrier.
template <bool kScores, typename Score>
__device__ __forceinline__ void settle(const Ranking &rk, const Deal &deal, uint32_t K, const uint32_t (&entry)[kResElites], bool changed,
                                       int32_t *sel, uint32_t *spare, Score score) {
  const uint32_t tid = opaque(threadIdx.x), lane = tid % kLanes, wave = tid / kLanes;
  uint64_t key[kResElites];
  uint32_t mine[kResElites], was[kResElites];
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads, slot = entry[k] & 0xFFFFu;
    if (e >= K) continue;
    if (kScores) key[k] = score(slot);
    was[k] = rk.srow[e];
    mine[k] = changed ? static_cast<uint32_t>(rk.spare[e]) : was[k];
    if (slot < K) atomicOr(&rk.bits[slot / 32], 1u << (slot % 32));
    if (sel) shared_store(sel + e, static_cast<int32_t>(slot));
  }
  __syncthreads();
  uint64_t children[kResElites], gone[kResElites];
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads;
    children[k] = __ballot(e < K && (entry[k] & 0xFFFFu) >= K);
    gone[k] = __ballot(e < K && ((rk.bits[min(e, K - 1) / 32] >> (e % 32)) & 1u) == 0);
    if (lane == 0) rk.wcount[k * kResWaves + wave] = static_cast<uint32_t>(__popcll(children[k])) | static_cast<uint32_t>(__popcll(gone[k])) << 16;
    if (e < K) {
      if (kScores) rk.ckey[e] = key[k];
      rk.srow[e] = static_cast<uint16_t>(entry[k] >> 16);
    }
  }
  __syncthreads();
  static_assert(kResElites * kResWaves <= kLanes, "a lane per count");
  const uint32_t count = lane < kResElites * kResWaves ? rk.wcount[lane] : 0u, upto = wave_inclusive_scan(count) - count;
  uint32_t nth[kResElites];
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads, before = __builtin_amdgcn_readlane(upto, __builtin_amdgcn_readfirstlane(k * kResWaves + wave));
    const uint64_t lower = (1ull << lane) - 1ull;
    nth[k] = (before & 0xFFFFu) + static_cast<uint32_t>(__popcll(children[k] & lower));
    if ((gone[k] >> lane) & 1ull) rk.drow[(before >> 16) + static_cast<uint32_t>(__popcll(gone[k] & lower))] = static_cast<uint16_t>(mine[k]);
    if (e / 32 < (K + 31) / 32 && e % 32 == 0) rk.bits[e / 32] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads, slot = entry[k] & 0xFFFFu;
    if (e >= K) continue;
    const uint32_t own = slot >= K ? deal.own(slot) : ~0u;
    if (own != ~0u) rk.rows[own] = rk.drow[nth[k]];
    if (changed && deal.me == 0) shared_store(spare + e, was[k]);
  }
  __syncthreads();
}

// Adds to place[i] how many records are below record i, in (score, slot) order, for all i < n; there are others behind
// those n, the last `more` of the kResInside.  A lane holds kOf records and compares them with the wave's share of all:
// one LDS read serves 64 * kOf comparisons (with a record per lane the reads, the same for all lanes, were what it
// took).  Scores are integers below 2^63 here.
template <int kOf>
__device__ __forceinline__ void count_below(const Ranking &rk, uint32_t n, uint32_t more, uint32_t first) {
  const uint32_t lane = threadIdx.x % kLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const uint32_t all = n + more, per = (all + kResWaves - 1) / kResWaves, from = wave * per, to = min(from + per, all);
  int64_t minus[kOf];
  uint32_t slot[kOf], count[kOf];
#pragma unroll
  for (int k = 0; k < kOf; ++k) {
    const uint4 v = rk.records[min(first + lane + k * kLanes, n - 1)];
    minus[k] = -static_cast<int64_t>(static_cast<uint64_t>(v.y) << 32 | v.x);
    slot[k] = v.z;
    count[k] = 0;
  }
#pragma unroll 2
  for (uint32_t q = from; q < to; ++q) {
    const uint4 v = rk.records[q < n ? q : q + (kResInside - all)];
    const int64_t key = static_cast<int64_t>(static_cast<uint64_t>(v.y) << 32 | v.x);
#pragma unroll
    for (int k = 0; k < kOf; ++k) {
      const int64_t less = key + minus[k] + (static_cast<int32_t>(v.z - slot[k]) >> 31);     // below 0 if it is
      count[k] += static_cast<uint32_t>(static_cast<uint64_t>(less) >> 63);
    }
  }
#pragma unroll
  for (int k = 0; k < kOf; ++k)
    if (first + lane + k * kLanes < n && from < to) atomicAdd(&rk.place[first + lane + k * kLanes], count[k]);
}
__device__ __forceinline__ void count_all_below(const Ranking &rk, uint32_t n, uint32_t more) {
  if (n <= kLanes) return count_below<1>(rk, n, more, 0u);
  if (n <= 2 * kLanes) return count_below<2>(rk, n, more, 0u);
  for (uint32_t first = 0; first < n; first += 4 * kLanes) count_below<4>(rk, n, more, first);
}

// (Argument block: ResidentArgs by value, which starts with its EvolveArgs, see kernel_args.)
static_assert(offsetof(ResidentArgs, ev) == 0, "kernel_args() reads the EvolveArgs at the start of the argument block");
// kSampled: the remaining work is drawn anew for every generation (Alg. 1, Eq. 7) and the whole pool, survivors
// included, is scored with the draw; the draws and their term tables have been made ahead (a ring in memory).
template <int Q, Genes kGenes, bool kOverGpus, bool kSampled, bool kWalk>
__global__ __launch_bounds__(kResThreads) void resident_kernel(ResidentArgs ra) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const EvolveArgs &a = ra.ev;
  const uint32_t P = a.P, K = a.K, tid = threadIdx.x, E = a.term_lds;
  const Deal deal{K, gridDim.x, blockIdx.x, ra.paired, (ra.paired ? 2u : 3u) * K};
  const Smem s = carve_table<Q>(smem_raw, E, kWalk);
  const Ranking rk = carve_ranking(smem_raw + ra.table_lds, Q, P, deal.groups, ra.list, ra.child_items);
  const int lane0 = tid & (kLanes - 1);
  const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t child_items = deal.mine(deal.children), all_items = deal.mine(deal.children + K);
  uint64_t *coins = reinterpret_cast<uint64_t *>(s.coins + static_cast<size_t>(wave_in_block) * a.coin_stride);
  auto draw_items = [&](uint32_t t) {                // for this workgroup's children and mutants of generation t
    for (uint32_t m = wave_in_block; m < child_items; m += kResWaves) {
      const uint32_t i = m * deal.groups + deal.me;
      draw_genes<Q, kOverGpus>(a, s, t, deal.first_slot(i), deal.both(i), opaque(lane0), rk.draws + 3 * m, rk.words + m * Q * kLanes);
    }
  };
  auto give_up = [&] { if (tid == 0) shared_store(ra.sync + 1, 1u); };
  auto terms_of = [&](uint32_t t) { return ra.ring_terms + static_cast<size_t>(t % kDrawRing) * ra.ring_stride; };
  auto load_terms = [&](const double *terms, uint32_t tile) {        // of a tile of the term table, see stage_table
    const uint32_t e = tile / (4 * Q), row = tile % (4 * Q);
    return tile < E * 4 * Q && row < a.Jp / kLanes ? terms[(row * E + e) * kLanes + lane0] : 0.0;
  };
  auto each_own_row = [&](auto f) {                  // f(slot, its row) for this workgroup's children
    for (uint32_t m = tid; m < 2 * child_items; m += kResThreads) {
      const uint32_t i = m / 2 * deal.groups + deal.me;
      if (m % 2 == 0 || deal.both(i)) f(deal.first_slot(i) + m % 2, rk.rows[m]);
    }
  };

  stage_table<Q>(a, s, E, ra.first_changed != 0, tid, kResThreads, kWalk);
  // the state the last selection left: the survivors' rows and scores, the rows of the units
  for (uint32_t e = tid; e < K; e += kResThreads) {
    const uint32_t row = checked_row(ra.parent_rows[e], P + K);
    rk.srow[e] = static_cast<uint16_t>(row);
    if (!ra.first_changed) rk.ckey[e] = static_cast<uint64_t>(__double_as_longlong(a.fit_row[row]));
    else if (a.assigned) rk.spare[e] = static_cast<uint16_t>(checked_row(a.spare[e], P + K));
  }
  for (uint32_t e = tid; e < max(K, kResInside); e += kResThreads) rk.place[e] = 0;
  if (tid < (P + K + 31) / 32) rk.bits[tid] = 0;
  if (tid < 4) rk.misc[tid] = 0;
  if (a.assigned) each_own_row([&](uint32_t slot, uint16_t &row) { row = static_cast<uint16_t>(checked_row(a.row_of[slot], P + K)); });
  __syncthreads();
  draw_items(a.t + 1);
  if (!a.assigned) list_free_rows(rk, deal, P, ra.first_changed != 0, a.spare);
  __syncthreads();

  for (uint32_t g = 0; g < ra.n_generations; ++g) {
    const uint32_t t = a.t + g + 1;
    const bool changed = g == 0 && ra.first_changed != 0;
    const bool new_first = changed && a.new_first != 0;
    const bool last = g + 1 == ra.n_generations;
    const bool all_new = changed || kSampled;                   // every candidate of the pool gets a new score
    const uint32_t items = all_new ? all_items : child_items;
    const uint32_t use = ra.generations_before + g;             // how often the exchange buffers have been used
    uint64_t *xk = ra.xkeys + static_cast<size_t>(use & 1u) * P;         // scores by pool slot
    uint32_t *xr = ra.xrow + static_cast<size_t>(use & 1u) * P;          // rows by pool slot
    uint64_t *flags = ra.flags + static_cast<size_t>(use & 1u) * kResidentMaxGroups;
    uint64_t *lists = ra.lists + static_cast<size_t>(use & 1u) * (P + 2 * kResidentMaxGroups) * 2;
    // ---- compose, repair, score and store this workgroup's candidates, one item after the other
    const uint64_t thresh = all_new ? 0ull : rk.ckey[K - 1];
    for (uint32_t m = wave_in_block < ra.unit_waves ? wave_in_block : items; m < items;) {
      const int lane = opaque(lane0);
      const uint32_t i = m * deal.groups + deal.me;
      auto done = [&](uint32_t slot, uint32_t which, uint32_t row, double f) {
        // (the butterfly leaves the same sum in every lane)
        const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(f));
        // A child that beats the K-th survivor (an equal score loses to the survivor's smaller slot) goes to the list with
        // its place, the survivors with a score at or below its own: here that takes a wave two reads, of every
        // stride-th survivor and of those between two of them; a search by each of its readers took them 1 to 4 us.
        const bool beats = bits < thresh;
        uint32_t place = 0;
        if (__ballot(beats) != 0) {
          const uint32_t stride = (K + kLanes - 1) / kLanes;
          place = stride * static_cast<uint32_t>(__popcll(__ballot((lane + 1) * stride <= K && rk.ckey[min((lane + 1) * stride, K) - 1] <= bits)));
          place += static_cast<uint32_t>(__popcll(__ballot(lane < static_cast<int>(stride) && place + lane < K && rk.ckey[min(place + lane, K - 1)] <= bits)));
        }
        if (lane != 0) return;
        shared_store(xk + slot, bits);
        shared_store(xr + slot, row);
        if (beats) {
          uint64_t *at = lists + (static_cast<size_t>(deal.me) * ra.segment + atomicAdd(&rk.misc[3], 1u)) * 2;
          shared_store(at, bits);
          shared_store(at + 1, slot | static_cast<uint64_t>(row) << 16 | static_cast<uint64_t>(place) << 32 | static_cast<uint64_t>(2 * m + which) << 48);
        }
        // the scores kept with the rows are only looked at after the call (to the point of coherence
        // like the rest: a plain store could linger in one XCD's cache)
        if (last) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + row, bits);
      };
      if (kSampled && !changed && i >= deal.children) {
        // the survivor of this rank keeps genome and row; only its score changes with the draw
        const uint32_t e = i - deal.children, row = __builtin_amdgcn_readfirstlane(rk.srow[e]);
        uint32_t c[Q];
        load_shared_genes<Q>(a.genes, row, lane, c);
        done(e, 0u, row, score<Q>(c, s, E, lane));
      } else if (changed) {
        compose_item<Q, kGenes, kOverGpus, false, kWalk>(a, t, s, rk, deal, i, new_first, coins, rk.draws + 3 * m, rk.words + m * Q * kLanes,
                                                  rk.rows + 2 * m, lane, done);
      } else {
        compose_item<Q, kGenes, kOverGpus, true, kWalk>(a, t, s, rk, deal, i, false, coins, rk.draws + 3 * m, rk.words + m * Q * kLanes,
                                                 rk.rows + 2 * m, lane, done);
      }
      uint32_t taken = 0;
      if (lane == 0) taken = atomicAdd(&rk.misc[2], 1u);
      m = ra.unit_waves + __builtin_amdgcn_readfirstlane(taken);
    }
    // genomes and scores of the whole workgroup have arrived before its flag says so
    phase_fence();
    __builtin_amdgcn_s_waitcnt(0);
    phase_fence();
    __syncthreads();
    if (tid == 0) {
      shared_store(flags + deal.me, static_cast<uint64_t>(use + 1) << 32 | rk.misc[3]);
      rk.misc[1] = rk.misc[2] = rk.misc[3] = 0;
    }
    // while the others' scores are on their way
    if (!last) draw_items(t + 1);
    constexpr int kTermsAhead = 4;                   // tiles of the next term table a wave loads ahead
    double term[kTermsAhead];
    if (kSampled && !last) {
#pragma unroll
      for (int v = 0; v < kTermsAhead; ++v) term[v] = load_terms(terms_of(t + 1), wave_in_block + v * kResWaves);
    }

    uint32_t listed_here, failed = 0, M, any_failed;            // children that this thread's workgroup lists; that all do
    if (!wait_for_all(flags, deal.groups, use + 1, ra.spin_limit, listed_here)) failed = 1;
    uint32_t before_me = listed_here;
    sums_before(rk, before_me, failed, M, any_failed);
    if (any_failed) return give_up();
    if (tid < deal.groups) {
      rk.from[tid] = before_me;
      if (M <= ra.list) for (uint32_t i = 0; i < listed_here; ++i) rk.order[before_me + i] = static_cast<uint16_t>(tid);
    }

    // every wave of this workgroup is done with the term table of this generation: the next one's
    if (kSampled && !last) {
      const double *terms = terms_of(t + 1);
#pragma unroll
      for (int v = 0; v < kTermsAhead; ++v) {
        const uint32_t tile = wave_in_block + v * kResWaves;
        if (tile < E * 4 * Q) s.terms[tile * kLanes + lane0] = term[v];
      }
      for (uint32_t tile = wave_in_block + kTermsAhead * kResWaves; tile < E * 4 * Q; tile += kResWaves)
        s.terms[tile * kLanes + lane0] = load_terms(terms, tile);
    }

    // what the state after the call says of this pool's survivors, before a ranking moves them: their rows and,
    // unless every score is new, the scores, which the generation that made them did not store with the rows
    if (last && deal.me == 0)
      for (uint32_t e = tid; e < K; e += kResThreads) {
        shared_store(a.row_of + e, static_cast<uint32_t>(rk.srow[e]));
        if (!all_new) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + rk.srow[e], rk.ckey[e]);
      }

    // ---- rank the pool
    bool crowded = !all_new && M > ra.list;          // so many children that the whole pool is ranked
    if (!all_new && M == 0) {
      // no child beats the K-th survivor: same survivors, same order, same rows
      if (last && deal.me == 0) for (uint32_t e = tid; e < K; e += kResThreads) shared_store(ra.sel + e, static_cast<int32_t>(e));
    } else if (!all_new && !crowded) {
      const uint32_t id = opaque(tid);
      __syncthreads();
      uint64_t key[kResListed], about[kResListed];   // of listed child id + k * kResThreads: slot, row, place, its row's among the workgroup's
      uint32_t own[kResListed];
#pragma unroll
      for (int k = 0; k < kResListed; ++k) {
        if (k * static_cast<uint32_t>(kResThreads) + wave_in_block * kLanes >= M) break;       // whole wave
        const uint32_t i = min(id + k * kResThreads, M - 1);
        own[k] = rk.order[i];
        const uint64_t *at = lists + (static_cast<size_t>(own[k]) * ra.segment + (i - rk.from[own[k]])) * 2;
        key[k] = shared_load(at);
        about[k] = shared_load(at + 1);
      }
      uint32_t place[kResListed];                    // its place and, above it, how many children came to that place before
#pragma unroll
      for (int k = 0; k < kResListed; ++k) {
        const uint32_t i = id + k * kResThreads;
        if (k * static_cast<uint32_t>(kResThreads) + wave_in_block * kLanes >= M) break;
        own[k] = own[k] == deal.me ? static_cast<uint32_t>(about[k] >> 48) : ~0u;
        const uint32_t lo = static_cast<uint32_t>(about[k] >> 32) & 0xFFFFu;
        if (i >= M) continue;
        place[k] = lo | atomicAdd(&rk.place[lo], 1u) << 16;
        rk.lkey[i] = key[k];
        rk.lslot[i] = static_cast<uint16_t>(about[k]);
      }
      __syncthreads();
      {                                              // running sum over the places
        const uint32_t per = (K + kResThreads - 1) / kResThreads, e0 = id * per;
        uint32_t n[kResElites], sum = 0, unused = 0, total, total_unused;
#pragma unroll
        for (int i = 0; i < kResElites; ++i) {
          n[i] = static_cast<uint32_t>(i) < per && e0 + i < K ? rk.place[e0 + i] : 0u;
          if (n[i] > kResPlace) rk.misc[1] = 1;
          sum += n[i];
        }
        sums_before(rk, sum, unused, total, total_unused);
#pragma unroll
        for (int i = 0; i < kResElites; ++i) {
          sum += n[i];
          if (static_cast<uint32_t>(i) < per && e0 + i < K) rk.place[e0 + i] = sum;
        }
      }
      __syncthreads();
      crowded = rk.misc[1] != 0;
      if (!crowded) {
        // the children in the order of their places, ...
        auto before = [&](uint32_t pos) { return pos ? rk.place[pos - 1] : 0u; };
#pragma unroll
        for (int k = 0; k < kResListed; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i < M) rk.order[before(place[k] & 0xFFFFu) + (place[k] >> 16)] = static_cast<uint16_t>(i);
        }
        __syncthreads();
        // ... those of one place ranked among themselves.  A child that comes b-th takes rank b + its place, and
        // if that is below K its slot the row of the last survivor but b, which drops out.
        uint32_t next_row[kResListed];
#pragma unroll
        for (int k = 0; k < kResListed; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i >= M) continue;
          const uint32_t pos = place[k] & 0xFFFFu, first = before(pos), end = rk.place[pos], slot = static_cast<uint32_t>(about[k]) & 0xFFFFu;
          uint32_t b = first;
          if (end - first > 1) {
            for (uint32_t q = first; q < end; q += 4) {          // (reads side by side: one after the other a place of eight took 2 us)
              uint32_t o[4], other[4];
              uint64_t score[4];
#pragma unroll
              for (int v = 0; v < 4; ++v) o[v] = rk.order[min(q + v, end - 1)];
#pragma unroll
              for (int v = 0; v < 4; ++v) { score[v] = rk.lkey[o[v]]; other[v] = rk.lslot[o[v]]; }
#pragma unroll
              for (int v = 0; v < 4; ++v) b += q + v < end && key_less(score[v], other[v], key[k], slot) ? 1u : 0u;
            }
          }
          place[k] = pos + b;                        // its rank
          next_row[k] = rk.srow[b < K ? K - 1 - b : 0u];
        }
        uint64_t elite_key[kResElites];
        uint32_t elite_row[kResElites], elite_rank[kResElites];
#pragma unroll
        for (int k = 0; k < kResElites; ++k) {
          const uint32_t e = id + k * kResThreads;
          elite_rank[k] = K;
          if (e < K) {
            elite_key[k] = rk.ckey[e];
            elite_row[k] = rk.srow[e];
            elite_rank[k] = e + rk.place[e];         // the children before it: those at its place or an earlier one
          }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kResListed; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i >= M || place[k] >= K) continue;
          rk.ckey[place[k]] = key[k];
          rk.srow[place[k]] = static_cast<uint16_t>(about[k] >> 16);
          if (own[k] != ~0u) rk.rows[own[k]] = static_cast<uint16_t>(next_row[k]);
          if (last && deal.me == 0) shared_store(ra.sel + place[k], static_cast<int32_t>(about[k] & 0xFFFFu));
        }
#pragma unroll
        for (int k = 0; k < kResElites; ++k) {
          const uint32_t e = id + k * kResThreads;
          if (e < K) rk.place[e] = 0;
          if (elite_rank[k] >= K) continue;
          rk.ckey[elite_rank[k]] = elite_key[k];
          rk.srow[elite_rank[k]] = static_cast<uint16_t>(elite_row[k]);
          if (last && deal.me == 0) shared_store(ra.sel + elite_rank[k], static_cast<int32_t>(e));
        }
        __syncthreads();
      }
    }
    if (all_new || crowded) {
      const uint32_t id = opaque(tid);
      // Every candidate's slot and row go to its rank.  In a pool of more than kResLocal each workgroup ranks a
      // range of the order, between two points of a sample of the pool, (score, slot) pairs, or every n-th slot of those of
      // a range: it counts the candidates below, ranks its own among those inside, and the workgroups exchange the order.
      // The ranges only divide what can survive, below a bound that a part of the sample gives, and each is shared by
      // several workgroups: with 256 ranges of the whole pool, one each, three quarters of them had nothing to do and the
      // others waited for the one with the largest range (16384 candidates: 30 us, now 19).
      const bool local = P <= kResLocal;
      auto score_at = [&](uint32_t slot) { return !all_new && slot < K ? rk.ckey[slot] : shared_load(xk + slot); };
      auto slot_of_point = [&](uint32_t q) { return q * P / kResSample; };
      auto record = [&](uint64_t key, uint32_t slot) { return make_uint4(static_cast<uint32_t>(key), static_cast<uint32_t>(key >> 32), slot, 0u); };
      uint64_t score_of[kResPool];
      uint64_t point = 0;
      if (!local && id < kResSample) point = score_at(slot_of_point(id));
#pragma unroll
      for (int k = 0; k < kResPool; ++k)
        if (k * static_cast<uint32_t>(kResThreads) < P) score_of[k] = score_at(min(id + k * kResThreads, P - 1));
      if (local && id < P) rk.records[id] = record(score_of[0], id);
      if (!local && id < kResSample) rk.sample[id] = point;
      if (id < 4) rk.range[id] = 0;
      if (!all_new) for (uint32_t e = id; e < K; e += kResThreads) rk.place[e] = 0;
      __syncthreads();
      uint32_t n_below = 0, n_inside = P, n_others = 0, share = 1, lo_slot = 0, hi_slot = 0;
      uint32_t inside = 0, mine = 0;                 // a bit for each of this thread's candidates inside, in this workgroup's share
      uint32_t front = 0, back = 0;                  // candidates in this workgroup's share, and the others, before this thread's
      uint64_t lo_key = 0ull, hi_key = ~0ull;        // the range: (score, slot) from lo on, below hi
      auto below = [&](uint64_t key, uint32_t slot) { return key < lo_key + (slot < lo_slot ? 1u : 0u); };
      auto beyond = [&](uint64_t key, uint32_t slot) { return key >= hi_key + (slot < hi_slot ? 1u : 0u); };
      if (!local) {
        {
          // the bound: a part of the sample ranked by counting
          // (counted in vector registers: one wave's ballot after the other, added up by the scalar unit that the
          // waves share, took twice as long)
          constexpr uint32_t kParts = kResThreads / kResFirst, kPer = kResFirst / kParts;
          const uint32_t every = kResSample / kResFirst, i = id % kResFirst, part = id / kResFirst;     // the part is the wave's
          const uint64_t key = rk.sample[i * every];
          uint32_t n = 0;
#pragma unroll
          for (uint32_t v = 0; v < kPer; ++v) {
            const uint32_t q = part * kPer + v;
            n += rk.sample[q * every] < key + (q < i ? 1u : 0u) ? 1u : 0u;
          }
          if (n) atomicAdd(&rk.place[i], n);
          __syncthreads();
          if (id < kResFirst) {
            if (rk.place[id] == kResBound) rk.range[0] = id * every;
            rk.place[id] = 0;
          }
          __syncthreads();
        }
        // the points of the sample below it, ranked by counting
        {
          const uint32_t q = rk.range[0], bound_slot = slot_of_point(q), slot = slot_of_point(id);
          const bool taken = id < kResSample && point < rk.sample[q] + (slot < bound_slot ? 1u : 0u);
          const uint64_t mask = __ballot(taken);
          uint32_t at = 0;
          if (lane0 == 0 && mask != 0) at = atomicAdd(&rk.range[1], static_cast<uint32_t>(__popcll(mask)));
          at = __builtin_amdgcn_readfirstlane(at) + static_cast<uint32_t>(__popcll(mask & ((1ull << lane0) - 1ull)));
          if (taken) rk.records[at] = record(point, slot);
        }
        __syncthreads();
        const uint32_t points = rk.range[1];         // at least kResBound
        {
          const uint4 v = rk.records[min(id, points - 1)];
          count_all_below(rk, points, 0u);
          __syncthreads();
          if (id < points) {
            const uint32_t r = rk.place[id];
            rk.sample[r] = static_cast<uint64_t>(v.y) << 32 | v.x;
            rk.order[r] = static_cast<uint16_t>(v.z);
            rk.place[id] = 0;
          }
        }
        __syncthreads();
        // this workgroup's range: one of the gaps before, between and behind those points, or, where there are fewer
        // workgroups, several; the last one has no end, so that the K best lie in the ranges whatever the sample was like
        const uint32_t gaps = points + 1;
        uint32_t lo = deal.me * gaps / deal.groups, hi = (deal.me + 1) * gaps / deal.groups;
        if (deal.groups >= gaps) {
          share = deal.groups / gaps;
          lo = deal.me / share;
          hi = lo + 1;
          if (lo >= gaps) lo = hi = 0;               // one of the workgroups left over
        }
        const uint32_t part = deal.me % share;
        if (lo != 0) { lo_key = rk.sample[lo - 1]; lo_slot = rk.order[lo - 1]; }
        if (hi != gaps) {
          if (hi == 0) hi_key = 0ull;                // (no gap)
          else { hi_key = rk.sample[hi - 1]; hi_slot = rk.order[hi - 1]; }
        }
#pragma unroll
        for (int k = 0; k < kResPool; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= P) continue;
          const uint32_t slot = id + k * kResThreads;
          const bool low = below(score_of[k], slot), real = slot < P;
          n_below += real && low ? 1u : 0u;
          inside |= real && !low && !beyond(score_of[k], slot) ? 1u << k : 0u;
        }
        if (share == 1) {
          mine = inside;
        } else {
          for (uint32_t left = inside; left != 0; left &= left - 1) {
            const uint32_t k = __ffs(static_cast<int>(left)) - 1;
            mine |= (id + k * kResThreads) % share == part ? 1u << k : 0u;
          }
        }
        if (__ballot(inside != 0) != 0) {
          // this workgroup's from the front, the others from the back
          const uint32_t n = __popc(mine) | __popc(inside & ~mine) << 16, upto = wave_inclusive_scan(n);
          uint32_t at = 0;
          if (lane0 == kLanes - 1) at = atomicAdd(&rk.range[3], upto);
          at = __builtin_amdgcn_readlane(at, kLanes - 1) + upto - n;
          front = at & 0xFFFFu;
          back = at >> 16;
          uint32_t f = front, b = back;
#pragma unroll
          for (int k = 0; k < kResPool; ++k) {
            if (k * static_cast<uint32_t>(kResThreads) >= P) continue;
            if (((inside >> k) & 1u) == 0) continue;
            const uint32_t to = (mine >> k) & 1u ? f++ : kResInside - 1 - b++;
            if (to < kResInside) rk.records[to] = record(score_of[k], id + k * kResThreads);
          }
        }
        n_below = wave_sum(n_below);
        if (lane0 == 0 && n_below != 0) atomicAdd(&rk.range[2], n_below);
        __syncthreads();
        n_below = rk.range[2];
        n_inside = n_below < K ? rk.range[3] & 0xFFFFu : 0u;     // otherwise nothing of this range survives
        n_others = rk.range[3] >> 16;
      }
      const uint64_t stamp = static_cast<uint64_t>(use + 1u) << 32;     // no generation has number 0
      auto row_at = [&](uint32_t slot) {
        return slot < K ? static_cast<uint32_t>(changed ? rk.spare[slot] : rk.srow[slot]) : shared_load(xr + slot);
      };
      auto put = [&](uint32_t rank, uint32_t slot, uint32_t row) {
        if (rank >= K) return;
        if (local) rk.nsel[rank] = slot | row << 16;
        else shared_store(ra.xrank + rank, stamp | row << 16 | slot);
      };
      if (n_inside + n_others <= kResInside) {
        uint32_t slot = 0, row = 0;
        if (id < n_inside) {
          slot = rk.records[id].z;
          row = row_at(slot);
        }
        if (n_inside != 0) count_all_below(rk, n_inside, n_others);
        __syncthreads();
        if (id < n_inside) {
          put(n_below + rk.place[id], slot, row);
          rk.place[id] = 0;
        }
      } else if (n_inside != 0) {
        // one of each thread's candidates after the other, against all of the range, kResInside at a time
        const uint32_t all = n_inside + n_others;
        for (uint32_t left = mine; __syncthreads_or(left != 0 ? 1 : 0); left &= left - 1) {
          const uint32_t own = left != 0 ? __ffs(static_cast<int>(left)) - 1 : 0u, slot = id + own * kResThreads;
          const uint64_t key = left != 0 ? score_at(slot) : 0ull;         // (read again: there is no room for them in registers)
          uint32_t n = 0;
          for (uint32_t from = 0; from < all; from += kResInside) {
            uint32_t f = front, b = n_inside + back;
#pragma unroll 1
            for (uint32_t bits = inside; bits != 0; bits &= bits - 1) {
              const uint32_t k = __ffs(static_cast<int>(bits)) - 1, to = ((mine >> k) & 1u ? f++ : b++) - from;
              if (to < kResInside) rk.records[to] = record(score_at(id + k * kResThreads), id + k * kResThreads);
            }
            __syncthreads();
            for (uint32_t q = 0; left != 0 && q < min(all - from, kResInside); ++q) {
              const uint4 v = rk.records[q];
              n += (static_cast<uint64_t>(v.y) << 32 | v.x) < key + (v.z < slot ? 1u : 0u) ? 1u : 0u;
            }
            __syncthreads();
          }
          if (left != 0) put(n_below + n, slot, row_at(slot));
        }
      }
      __syncthreads();
      uint32_t entry[kResElites];                    // slot and row of the new survivors id, id + kResThreads, ...
      bool ranked = local;
      if (local) {
        entry[0] = rk.nsel[min(id, K - 1)];
      } else {
        for (uint32_t spins = 0; spins < ra.spin_limit && !ranked; ++spins) {
          bool all = true;
#pragma unroll
          for (int k = 0; k < kResElites; ++k) {
            if (k * static_cast<uint32_t>(kResThreads) >= K) break;
            const uint64_t v = shared_load(ra.xrank + min(id + k * kResThreads, K - 1));
            entry[k] = static_cast<uint32_t>(v);
            all = all && (v >> 32) == (stamp >> 32);
          }
          ranked = __ballot(!all) == 0;
        }
      }
      if (__syncthreads_or(ranked ? 0 : 1)) return give_up();
      settle<!kSampled>(rk, deal, K, entry, changed, last && deal.me == 0 ? ra.sel : nullptr, a.spare, score_at);
    }
    if (last) {
      // the state the next call (of either kind) starts from
      if (deal.me == 0) for (uint32_t e = tid; e < K; e += kResThreads) shared_store(ra.parent_rows + e, static_cast<uint32_t>(rk.srow[e]));
      each_own_row([&](uint32_t slot, uint16_t row) { shared_store(a.row_of + slot, static_cast<uint32_t>(row)); });
      // and, if that is one of the launched kernels, the splitters of its buckets, as a selection of theirs would have left them
      // (without them its first one ranks the pool in full: a selection of 24 us in place of 6.4, 16384 candidates)
      // (their addresses are read from the argument block here, see kernel_args, not carried through the generations)
      const auto *late = (const __attribute__((address_space(4))) ResidentArgs *)kernel_args();
      if (!kSampled && deal.me + 1 == deal.groups && late->n_buckets != 0) {
        const uint32_t nb = late->n_buckets;
        for (uint32_t c = tid; c < static_cast<uint32_t>(kBucketCounters); c += kResThreads) {
          shared_store(late->count[0] + c, 0u);
          shared_store(late->count[1] + c, 0u);
          if (c < static_cast<uint32_t>(kMaxBuckets)) shared_store(late->split + c, c + 1 < nb ? rk.ckey[bucket_bound(c + 1, K, nb)] : static_cast<uint64_t>(kNoSplitter));
          if (c == 0) shared_store(late->thresh, rk.ckey[K - 1]);
        }
      }
      if (deal.me == 0) {
        const uint32_t row = rk.srow[0];
        publish_winner(late->winner, a.genes, Q * kLanes, row, a.tab.info, kSampled ? shared_load(reinterpret_cast<const uint64_t *>(a.fit_row) + row) : rk.ckey[0]);
      }
      // The last workgroup tells the host.  Nothing of the workspace is written any more then: what the launch stores there goes
      // to the point of coherence, and is there before the workgroup counts as arrived.
      all_arrived();
      if (tid != 0) return;
      if (deal.me == 0) __threadfence_system();      // the winner
      if (last_to_arrive(late->winner.done.arrived)) signal_call_done(late->winner, late->sync + 1);
      return;
    }
  }
}

template <int Q, Genes kGenes, bool kOverGpus, bool kSampled>
const void *kernel_of(const ResidentPlan &plan) {
  return plan.walk ? reinterpret_cast<const void *>(resident_kernel<Q, kGenes, kOverGpus, kSampled, true>)
                   : reinterpret_cast<const void *>(resident_kernel<Q, kGenes, kOverGpus, kSampled, false>);
}

template <int Q, Genes kGenes>
hipError_t launch_genes(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t stream) {
  const bool over = args.ev.per_gpu != 0, sampled = args.sampled != 0;
  const void *fn = over ? (sampled ? kernel_of<Q, kGenes, true, true>(plan) : kernel_of<Q, kGenes, true, false>(plan))
                        : (sampled ? kernel_of<Q, kGenes, false, true>(plan) : kernel_of<Q, kGenes, false, false>(plan));
  const hipError_t rc = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(plan.lds));
  if (rc != hipSuccess) return rc;
  ResidentArgs ra = args;
  void *params[] = {&ra};
  static const bool plain = getenv("ONES_FUSED_PLAIN_LAUNCH") != nullptr;        // for profilers, see launch_fused
  if (plain) return hipLaunchKernel(fn, dim3(plan.groups), dim3(kResThreads), params, plan.lds, stream);
  return hipLaunchCooperativeKernel(fn, dim3(plan.groups), dim3(kResThreads), params, static_cast<unsigned int>(plan.lds), stream);
}

}  // namespace

#if ONES_RESIDENT_WORDS == 1
size_t resident_exchange_bytes(uint32_t P) {          // zeroed once
  return (static_cast<size_t>(4) * (P + 2 * kResidentMaxGroups) + 2 * P + P / 4 + 2 * kResidentMaxGroups) * 8 + static_cast<size_t>(2) * P * 4;
}

void resident_exchange(uint64_t *base, uint32_t P, ResidentArgs &ra) {
  ra.lists = base;
  ra.xkeys = ra.lists + static_cast<size_t>(4) * (P + 2 * kResidentMaxGroups);
  ra.xrank = ra.xkeys + static_cast<size_t>(2) * P;
  ra.flags = ra.xrank + P / 4;
  ra.xrow = reinterpret_cast<uint32_t *>(ra.flags + 2 * kResidentMaxGroups);
}

bool resident_plan(const EvolveArgs &ev, bool sampled, int n_cus, ResidentPlan &plan) {
  const uint32_t Q = static_cast<uint32_t>(words_of(static_cast<int>(ev.Jp / kLanes))), K = ev.P / 4;
  if (Q > static_cast<uint32_t>(kResidentMaxWords) || ev.P > static_cast<uint32_t>(kResidentMaxPool) || ev.P < 4) return false;
  // A wave of every SIMD computes; where there are more items than those of the whole chip, more do, all for
  // the same number of rounds.
  const uint32_t n_groups = std::min<uint32_t>(static_cast<uint32_t>(n_cus), kResidentMaxGroups);
  plan.paired = 3 * K > n_groups * kResWaves ? 1u : 0u;
  const uint32_t children = (plan.paired ? 2 : 3) * K, items = children + (sampled ? K : 0);
  plan.groups = std::min<uint32_t>(n_groups, (items + 3) / 4);
  const uint32_t per_group = (items + plan.groups - 1) / plan.groups, rounds = (per_group + kResWaves - 1) / kResWaves;
  plan.unit_waves = std::min<uint32_t>(kResWaves, ((per_group + rounds - 1) / rounds + 3) / 4 * 4);
  plan.groups = std::min<uint32_t>(plan.groups, (items + plan.unit_waves - 1) / plan.unit_waves);
  plan.child_items = (children + plan.groups - 1) / plan.groups;
  plan.segment = (plan.paired ? 2 : 1) * plan.child_items;
  plan.list = kResLeastList;
  size_t least = 0;
  for (plan.walk = ev.walk;; plan.walk = 0) {  // the repair walks where there is room for it
    plan.coin_stride = plan.walk ? std::max<uint32_t>(coin_stride(ev), window_bytes(Q)) : coin_stride(ev);
    plan.table_lds = static_cast<uint32_t>((table_bytes(Q, ev.tab.term_E, plan.coin_stride, plan.walk != 0) + 15) & ~size_t(15));
    least = plan.table_lds + ranking_bytes(Q, ev.P, plan);
    if (least <= kResLds) break;
    if (plan.walk == 0) return false;
  }
  // the list of the children takes what is left
  plan.list = std::min<uint32_t>({std::max(ev.P, kResLeastList), kResList, static_cast<uint32_t>(plan.list + (kResLds - least) / 12)});
  plan.lds = plan.table_lds + ranking_bytes(Q, ev.P, plan);
  return plan.lds <= kResLds;
}
#endif

#define ONES_CONCAT2(x, y) x##y
#define ONES_CONCAT(x, y) ONES_CONCAT2(x, y)
hipError_t ONES_CONCAT(launch_resident_words, ONES_RESIDENT_WORDS)(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t s) {
  constexpr int Q = ONES_RESIDENT_WORDS;
  const uint32_t largest = args.ev.tab.term_E - 1;   // largest code under this table
  if (largest <= kNarrowCodes) return launch_genes<Q, kNarrow>(args, plan, s);
  return largest <= kMiddleCodes ? launch_genes<Q, kMiddle>(args, plan, s) : launch_genes<Q, kWide>(args, plan, s);
}

}  // namespace ones
