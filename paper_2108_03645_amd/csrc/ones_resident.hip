// All generations of one ones_generation call in a single launch (ONES, arXiv 2108.03645, Section 3.2.2), for
// pools of a few thousand candidates beyond those of ones_fused.hip: up to kResidentMaxPool candidates of up to
// 64 * 4 * kResidentMaxWords job slots, as far as a workgroup's LDS holds the job table and the ranking.
//
// The protocol is that of ones_fused.hip: a co-resident grid, one workgroup to a compute unit, stays on the chip
// for the whole call; every wave composes, repairs and scores its share of the 3K children (4K candidates when
// every score is new), publishes genome and score, and every workgroup ranks the pool by itself in its LDS from
// the scores of all, so that one exchange separates two generations.  (Two launches a generation, the other way
// to do this, spend more on their boundaries, on staging the job table and on looking rows and scores up through
// memory than on the candidates: a pool of 8192 on 200 slots 15 us a generation, of which 2.5 compute.)
// What differs is the size: hundreds to thousands of children beat the K-th survivor of such a pool in every
// generation, too many to count against each other.  The survivors are in order, so such a child finds its place
// among them by binary search; the children of each place are counted, the counts summed up, and the few
// children that share a place ranked among themselves.  Only where many share one (a pool full of copies of one
// genome), or where every score is new, do the workgroups rank a share of the pool each, by counting, and
// exchange the order in a second step.
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
constexpr uint32_t kResPlace = 128;          // children that share a place among the survivors, at most
constexpr uint32_t kResSample = 128;         // sample points of a pool that is ranked as a whole
constexpr uint32_t kResLocal = 256;          // ... unless it is so small that every workgroup ranks it by itself
constexpr uint32_t kResInside = kResThreads / 2;       // candidates of a range whose scores are copied together
constexpr uint32_t kResPlaces = 2 * kResInside + kResInside;    // counters at least: room for those scores and a count each
static_assert(kResLocal <= kResInside, "ranked like a range");
constexpr int kResKids = 3 * kResidentMaxPool / 4 / kResThreads;         // children a thread handles, at most
constexpr int kResElites = kResidentMaxPool / 4 / kResThreads;           // survivors ...
constexpr int kResPool = kResidentMaxPool / kResThreads;
static_assert(kResidentMaxPool % (4 * kResThreads) == 0, "whole numbers of children and survivors per thread");

// ----------------------------------------------------------------- LDS -------------
struct Ranking {
  uint64_t *ckey;    // [P] score bits: of the survivors, best first, then of the children that beat the last of
                     // them, in any order; in a ranking of the whole pool of all candidates, by slot
  uint32_t *place;   // [K, at least kResPlaces] children at each place, then their running sum; zero between uses
  uint32_t *range;   // [4] slots of the sample points that bound this workgroup's range, candidates below and inside it
  uint32_t *bits;    // bitmap: over the P + K rows when rows are listed, over the survivors of the generation before
  uint32_t *wcount;  // [2][kResWaves] counts of the waves, for prefix sums
  uint32_t *misc;    // [0] children that beat the K-th survivor, [1] whether a place is crowded
  uint32_t *draws;   // [unit waves][child units][2] per child: ranks of its parents, start of its repair (drawn ahead)
  uint32_t *words;   // [unit waves][child units][Q * 64] what it draws per gene (see draw_genes)
  uint16_t *lslot;   // [3K] slots of the children in ckey + K
  uint16_t *order;   // [3K] those children in the order of their places
  uint16_t *all;     // [P] in their place, when the whole pool is ranked: slots of the candidates of this workgroup's range
  uint16_t *nsel;    // [K] ... and behind it pool slots of the new survivors
  uint16_t *drow;    // [K] ... and rows of survivors that dropped out
  uint16_t *srow;    // [K] genome rows of the survivors
  uint16_t *frow;    // [P] the row unit u of a generation writes; the last K are spare between table changes
};

[[maybe_unused]] inline size_t ranking_bytes(uint32_t Q, uint32_t P, uint32_t unit_waves, uint32_t child_units) {
  const size_t K = P / 4, words = (P + K + 31) / 32;
  return 8 * static_cast<size_t>(P) +
         4 * (std::max<size_t>(K, kResPlaces) + 4 + words + 2 * kResWaves + 4 + static_cast<size_t>(unit_waves) * child_units * (2 + Q * kLanes)) +
         2 * (2 * 3 * K + K + P) + 16;
}

__device__ __forceinline__ Ranking carve_ranking(unsigned char *base, uint32_t Q, uint32_t P, uint32_t unit_waves, uint32_t child_units) {
  const uint32_t K = P / 4, words = (P + K + 31) / 32;
  Ranking r;
  r.ckey = reinterpret_cast<uint64_t *>(base);
  r.place = reinterpret_cast<uint32_t *>(r.ckey + P);
  r.range = r.place + max(K, kResPlaces);
  r.bits = r.range + 4;
  r.wcount = r.bits + words;
  r.misc = r.wcount + 2 * kResWaves;
  r.draws = r.misc + 4;
  r.words = r.draws + unit_waves * child_units * 2;
  r.lslot = reinterpret_cast<uint16_t *>(r.words + static_cast<size_t>(unit_waves) * child_units * Q * kLanes);
  r.all = r.lslot;
  r.nsel = r.all + P;
  r.drow = r.nsel + K;
  r.order = r.lslot + 3 * K;
  r.srow = r.order + 3 * K;
  r.frow = r.srow + K;
  return r;
}

// The job table in LDS without what only the kernels of one generation need.
[[maybe_unused]] inline size_t table_bytes(uint32_t Q, uint32_t E, uint32_t unit_waves, uint32_t stride) {
  const size_t words = static_cast<size_t>(Q) * kLanes;
  return words * (4 * 8 * static_cast<size_t>(E) + 8 + 8 + 7 * 4) + static_cast<size_t>(unit_waves) * stride;
}
template <int Q>
__device__ __forceinline__ Smem carve_table(unsigned char *at, uint32_t E) {
  constexpr uint32_t kWords = Q * kLanes;
  Smem s{};
  s.terms = reinterpret_cast<double *>(at);
  s.rank = reinterpret_cast<uint2 *>(s.terms + static_cast<size_t>(4 * kWords) * E);
  s.prefix = s.rank + kWords;
  s.start = reinterpret_cast<uint32_t *>(s.prefix + kWords);
  s.most = s.start + kWords;
  s.draws = s.most + kWords;
  s.base = s.draws + kWords;
  s.shift = s.base + kWords;
  s.fresh = s.shift + kWords;
  s.bl = s.fresh + kWords;
  s.coins = reinterpret_cast<uint8_t *>(s.bl + kWords);
  return s;
}

// ----------------------------------------------------------------- exchange --------
// Waits until the flags of all workgroups have come to `want` (flags only ever count up, modulo 2^32): a thread per
// workgroup polls.  False when the polls ran out.
__device__ __forceinline__ bool wait_for_all(const uint32_t *flags, uint32_t n, uint32_t want, uint32_t spin_limit) {
  const uint32_t *mine = flags + min(threadIdx.x, n - 1);
  if (threadIdx.x / kLanes * kLanes >= n) return true;           // whole waves without a flag to look at
  for (uint32_t spins = 0; spins < spin_limit; ++spins)
    if (__ballot(static_cast<int32_t>(shared_load(mine) - want) < 0) == 0) return true;
  return false;
}

// ----------------------------------------------------------------- candidates ------
// What a child or mutant draws before it needs anything of its parents depends on (seed, generation, slot)
// only, so a wave draws for the coming generation while the scores of the current one are still arriving.
// A word per four genes: for a child of a pair 0xFF where the pair's genes are swapped; for a mutant 0x80 and the
// new code where a gene is redrawn.
template <int Q, bool kOverGpus>
__device__ __forceinline__ void draw_genes(const EvolveArgs &a, const Smem &s, uint32_t t, uint32_t u, int lane, uint32_t *draws,
                                           uint32_t *words) {
  const uint32_t K = a.K, R = a.Jp / kLanes;
  const bool child = u < 2 * K;
  const uint32_t p = K + u, p0 = child ? p - (u & 1u) : p;       // a pair shares what is drawn for its first slot,
  const Draw d = candidate_draw(a, t, lane == 0 ? p0 : p);       // but for the rotation: lane 0 the former, lane 1 the latter
  if (lane == 0) draws[0] = d.ra | d.rb << 16;
  if (lane == 1) draws[1] = d.r / R | d.r % R << 16;
  if (child && kOverGpus) return;
  const WordSource source(a, t, p0);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const Words w = source.block(s.prefix, q, lane);
    uint32_t out;
    if (child) {
      out = words_below(w, a.T_x);
    } else {
      const uint32_t outcomes = s.draws[q * kLanes + lane], redrawn = words_below(w, a.T_mut);
      uint32_t k = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) k |= (((w.w[v] & 0xFFFFu) * ((outcomes >> (8 * v)) & 0xFFu)) >> 16) << (8 * v);
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

// One candidate of generation t: unit u < 2K is a child of pair u / 2, u < 3K a mutant, u >= 3K (only after a
// table change) the survivor of rank u - 3K to refresh.  Returns the score; the repaired genes are left in c.
template <int Q, Genes kGenes, bool kOverGpus, bool kSameTable>
__device__ __forceinline__ double compose_unit(const EvolveArgs &a, uint32_t t, const Smem &s, const uint16_t *srow, uint32_t u,
                                               bool new_first, uint64_t *coins, const uint32_t *draws, const uint32_t *words, int lane,
                                               uint32_t (&c)[Q]) {
  const uint32_t K = a.K;
  uint32_t start;
  if (u < 3 * K) {
    const uint32_t parents = __builtin_amdgcn_readfirstlane(draws[0]);
    start = __builtin_amdgcn_readfirstlane(draws[1]);
    load_shared_genes<Q>(a.genes, srow[parents & 0xFFFFu], lane, c);
    if (u < 2 * K) {
      const bool second = (u & 1u) != 0;
      uint32_t other[Q];
      load_shared_genes<Q>(a.genes, srow[parents >> 16], lane, other);
      if (kOverGpus) {
        if (!kSameTable) { to_new_table<Q>(s, lane, c); to_new_table<Q>(s, lane, other); }
        phase_fence();
        crossover_over_gpus<Q, kSameTable>(a, t, s, coins, K + (u & ~1u), lane, c, other);
#pragma unroll
        for (int q = 0; q < Q; ++q) c[q] = second ? other[q] : c[q];
      } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t drawn = words[q * kLanes + lane];
          c[q] = pick(second ? ~drawn : drawn, other[q], c[q]);
        }
        if (!kSameTable) to_new_table<Q>(s, lane, c);
      }
    } else {
      if (!kSameTable) to_new_table<Q>(s, lane, c);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t drawn = words[q * kLanes + lane], redrawn = spread_tops(drawn);
        c[q] = pick(redrawn, drawn & kSevens, c[q]);
      }
    }
  } else {
    const uint32_t p = u - 3 * K, R = a.Jp / kLanes, r = __builtin_amdgcn_readfirstlane(candidate_draw(a, t, p).r);
    start = r / R | r % R << 16;
    load_shared_genes<Q>(a.genes, srow[p], lane, c);
    to_new_table<Q>(s, lane, c);
  }
  phase_fence();
  const uint32_t lr = start & 0xFFFFu, ir = start >> 16;
  if (!kSameTable && new_first) repair<Q, kGenes, true>(c, s, a.G, lr, ir, lane, a.Jp, a.time_rank != nullptr);
  else repair<Q, kGenes, false>(c, s, a.G, lr, ir, lane, a.Jp, false);
  phase_fence();
  return score<Q>(c, s, a.term_lds, lane);
}

// ----------------------------------------------------------------- rows ------------
// Running sum of two counts over the threads of the workgroup; with one barrier.
__device__ __forceinline__ void sums_before(const Ranking &rk, uint32_t &x, uint32_t &y) {
  const uint32_t lane = threadIdx.x % kLanes, wave = threadIdx.x / kLanes;
  const uint32_t ix = wave_inclusive_scan(x), iy = wave_inclusive_scan(y);
  if (lane == kLanes - 1) { rk.wcount[wave] = ix; rk.wcount[kResWaves + wave] = iy; }
  __syncthreads();
  // the waves before this one, summed up by each wave for itself
  const bool earlier = lane < wave;
  const uint32_t wx = wave_sum(earlier ? rk.wcount[lane] : 0u), wy = wave_sum(earlier ? rk.wcount[kResWaves + lane] : 0u);
  x = wx + ix - x;
  y = wy + iy - y;
}

// The rows that are not the survivors', in ascending order, as rows of the units, when no selection has
// assigned them.  rk.bits is zero before and after.  Whole workgroup; ends with a barrier.
__device__ __forceinline__ void list_free_rows(const Ranking &rk, uint32_t P) {
  const uint32_t K = P / 4, n_rows = P + K, words = (n_rows + 31) / 32;
  static_assert((kResidentMaxPool + kResidentMaxPool / 4) / 32 <= kResThreads, "a thread per word of the bitmap");
  for (uint32_t g = threadIdx.x; g < K; g += kResThreads) atomicOr(&rk.bits[rk.srow[g] >> 5], 1u << (rk.srow[g] & 31u));
  __syncthreads();
  uint32_t free_bits = threadIdx.x < words ? ~rk.bits[threadIdx.x] : 0u;
  if (threadIdx.x + 1 == words && n_rows % 32 != 0) free_bits &= (1u << (n_rows % 32)) - 1u;
  uint32_t at = __popc(free_bits), unused = 0;
  sums_before(rk, at, unused);
  while (free_bits) {
    if (at < P) rk.frow[at] = static_cast<uint16_t>(threadIdx.x * 32 + (__ffs(static_cast<int>(free_bits)) - 1));
    free_bits &= free_bits - 1;
    ++at;
  }
  if (threadIdx.x < words) rk.bits[threadIdx.x] = 0;
  __syncthreads();
}

// The scores and rows that go with a ranking of the whole pool, whose new survivors' slots are in nsel: the new survivors
// keep theirs, and the slots of the surviving children take the rows of the survivors that dropped out, the i-th the
// i-th (both counted in the same order by every workgroup).  changed: the pool's first K slots are refreshed survivors in the
// spare rows, and the rows they came from are spare from now on.  rk.bits is zero before and after.  Ends with a barrier.
__device__ __forceinline__ void settle(const Ranking &rk, uint32_t P, bool changed, int32_t *sel) {
  const uint32_t K = P / 4, tid = opaque(threadIdx.x), lane = tid % kLanes, wave = tid / kLanes;
  uint64_t key[kResElites];
  uint32_t slot[kResElites], kept[kResElites], mine[kResElites], was[kResElites];
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads;
    if (e >= K) continue;
    auto row_of_elite = [&](uint32_t i) { return static_cast<uint32_t>(changed ? rk.frow[3 * K + i] : rk.srow[i]); };
    slot[k] = rk.nsel[e];
    key[k] = rk.ckey[slot[k]];
    mine[k] = row_of_elite(e);
    was[k] = rk.srow[e];
    kept[k] = slot[k] < K ? row_of_elite(slot[k]) : rk.frow[slot[k] - K];
    if (slot[k] < K) atomicOr(&rk.bits[slot[k] / 32], 1u << (slot[k] % 32));
    if (sel) sel[e] = static_cast<int32_t>(slot[k]);
  }
  __syncthreads();
  uint64_t children[kResElites], gone[kResElites];
#pragma unroll
  for (int k = 0; k < kResElites; ++k) {
    const uint32_t e = tid + k * kResThreads;
    children[k] = __ballot(e < K && slot[k] >= K);
    gone[k] = __ballot(e < K && ((rk.bits[min(e, K - 1) / 32] >> (e % 32)) & 1u) == 0);
    if (lane == 0) rk.wcount[k * kResWaves + wave] = static_cast<uint32_t>(__popcll(children[k])) | static_cast<uint32_t>(__popcll(gone[k])) << 16;
    if (e < K) {
      rk.ckey[e] = key[k];
      rk.srow[e] = static_cast<uint16_t>(kept[k]);
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
    const uint32_t e = tid + k * kResThreads;
    if (e >= K) continue;
    if (slot[k] >= K) rk.frow[slot[k] - K] = rk.drow[nth[k]];
    if (changed) rk.frow[3 * K + e] = static_cast<uint16_t>(was[k]);
  }
  __syncthreads();
}

// (Argument block: ResidentArgs by value, which starts with its EvolveArgs, see kernel_args.)
static_assert(offsetof(ResidentArgs, ev) == 0, "kernel_args() reads the EvolveArgs at the start of the argument block");
// kSampled: the remaining work is drawn anew for every generation (Alg. 1, Eq. 7) and the whole pool, survivors
// included, is scored with the draw; the draws and their term tables have been made ahead (a ring in memory).
template <int Q, Genes kGenes, bool kOverGpus, bool kSampled>
__global__ __launch_bounds__(kResThreads) void resident_kernel(ResidentArgs ra) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const EvolveArgs &a = ra.ev;
  const uint32_t P = a.P, K = a.K, tid = threadIdx.x, E = a.term_lds;
  const Smem s = carve_table<Q>(smem_raw, E);
  const Ranking rk = carve_ranking(smem_raw + ra.table_lds, Q, P, ra.unit_waves, ra.child_units);
  const int lane0 = tid & (kLanes - 1);
  const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t n_groups = gridDim.x, n_waves = n_groups * ra.unit_waves;
  // the first unit_waves waves of every workgroup compute candidates; all of them rank
  const uint32_t wave = wave_in_block < ra.unit_waves ? blockIdx.x * ra.unit_waves + wave_in_block : 4 * K;
  uint64_t *coins = reinterpret_cast<uint64_t *>(s.coins + static_cast<size_t>(wave_in_block) * a.coin_stride);
  uint32_t *my_draws = rk.draws + wave_in_block * ra.child_units * 2;
  uint32_t *my_words = rk.words + wave_in_block * ra.child_units * Q * kLanes;
  auto draw_units = [&](uint32_t t) {                // for this wave's children and mutants of generation t
    for (uint32_t k = 0, u = wave; u < 3 * K; ++k, u += n_waves)
      draw_genes<Q, kOverGpus>(a, s, t, u, opaque(lane0), my_draws + 2 * k, my_words + k * Q * kLanes);
  };
  auto give_up = [&] { if (tid == 0) shared_store(ra.sync + 1, 1u); };
  auto terms_of = [&](uint32_t t) { return ra.ring_terms + static_cast<size_t>(t % kDrawRing) * ra.ring_stride; };
  auto load_terms = [&](const double *terms, uint32_t tile) {        // of a tile of the term table, see stage_table
    const uint32_t e = tile / (4 * Q), row = tile % (4 * Q);
    return tile < E * 4 * Q && row < a.Jp / kLanes ? terms[(row * E + e) * kLanes + lane0] : 0.0;
  };

  stage_table<Q>(a, s, E, ra.first_changed != 0, tid, kResThreads);
  // the state the last selection left: the survivors' rows and scores, the rows of the units
  for (uint32_t e = tid; e < K; e += kResThreads) {
    const uint32_t row = checked_row(ra.parent_rows[e], P + K);
    rk.srow[e] = static_cast<uint16_t>(row);
    rk.ckey[e] = static_cast<uint64_t>(__double_as_longlong(a.fit_row[row]));
    if (a.assigned) rk.frow[3 * K + e] = static_cast<uint16_t>(checked_row(a.spare[e], P + K));
  }
  for (uint32_t e = tid; e < max(K, kResPlaces); e += kResThreads) rk.place[e] = 0;
  if (tid < (P + K + 31) / 32) rk.bits[tid] = 0;
  if (a.assigned)
    for (uint32_t u = tid; u < 3 * K; u += kResThreads) rk.frow[u] = static_cast<uint16_t>(checked_row(a.row_of[K + u], P + K));
  __syncthreads();
  draw_units(a.t + 1);
  if (!a.assigned) list_free_rows(rk, P);

  for (uint32_t g = 0; g < ra.n_generations; ++g) {
    const uint32_t t = a.t + g + 1;
    const bool changed = g == 0 && ra.first_changed != 0;
    const bool new_first = changed && a.new_first != 0;
    const bool last = g + 1 == ra.n_generations;
    const bool all_new = changed || kSampled;                   // every candidate of the pool gets a new score
    const uint32_t units = all_new ? 4 * K : 3 * K;
    const uint32_t use = ra.generations_before + g;             // how often the exchange buffers have been used
    uint64_t *xk = ra.xkeys + static_cast<size_t>(use & 1u) * P;         // scores by pool slot
    // ---- compose, repair, score and store this wave's candidates
    for (uint32_t k = 0, u = wave; u < units; ++k, u += n_waves) {
      const int lane = opaque(lane0);
      uint32_t c[Q], row;
      double f;
      if (kSampled && !changed && u >= 3 * K) {
        // the survivor of rank u - 3K keeps genome and row; only its score changes with the draw
        row = rk.srow[u - 3 * K];
        load_shared_genes<Q>(a.genes, row, lane, c);
        f = score<Q>(c, s, E, lane);
      } else {
        f = changed ? compose_unit<Q, kGenes, kOverGpus, false>(a, t, s, rk.srow, u, new_first, coins, my_draws + 2 * k,
                                                                my_words + k * Q * kLanes, lane, c)
                    : compose_unit<Q, kGenes, kOverGpus, true>(a, t, s, rk.srow, u, false, coins, my_draws + 2 * k,
                                                               my_words + k * Q * kLanes, lane, c);
        row = rk.frow[u];
        uint32_t *at = a.genes + static_cast<size_t>(row) * (Q * kLanes) + lane;
#pragma unroll
        for (int q = 0; q < Q; ++q) shared_store(at + q * kLanes, c[q]);
      }
      if (lane == 0) {
        const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(f));
        shared_store(u < 3 * K ? xk + K + u : xk + (u - 3 * K), bits);
        // the scores kept with the rows are only looked at after the call (to the point of coherence
        // like the rest: a plain store could linger in one XCD's cache)
        if (last) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + row, bits);
      }
    }
    // genomes and scores of the whole workgroup have arrived before its flag says so
    phase_fence();
    __builtin_amdgcn_s_waitcnt(0);
    phase_fence();
    __syncthreads();
    if (tid == 0) {
      shared_store(ra.flags + blockIdx.x, use + 1);
      rk.misc[0] = rk.misc[1] = 0;
    }
    // while the others' scores are on their way
    if (!last) draw_units(t + 1);
    constexpr int kTermsAhead = 4;                   // tiles of the next term table a wave loads ahead
    double term[kTermsAhead];
    if (kSampled && !last) {
#pragma unroll
      for (int v = 0; v < kTermsAhead; ++v) term[v] = load_terms(terms_of(t + 1), wave_in_block + v * kResWaves);
    }

    // ---- collect the scores: children and mutants i < 3K, then, when every score is new, the survivors.  The
    // children that beat the K-th survivor are listed behind the survivors' scores (an equal score loses to the
    // survivor's smaller slot); when every score is new all of them go to their slots.
    if (__syncthreads_or(wait_for_all(ra.flags, n_groups, use + 1, ra.spin_limit) ? 0 : 1)) return give_up();
    uint64_t score_of[kResPool];                     // of the candidates slot_of_entry(tid + k * kResThreads)
    auto slot_of_entry = [&](uint32_t i) { return i < 3 * K ? K + i : i - 3 * K; };
    {
      const uint32_t id = opaque(tid), n = all_new ? P : 3 * K;
      const uint64_t thresh = all_new ? 0ull : rk.ckey[K - 1];
#pragma unroll
      for (int k = 0; k < kResPool; ++k)
        if (k * static_cast<uint32_t>(kResThreads) < n)
          score_of[k] = shared_load(xk + slot_of_entry(min(id + k * kResThreads, n - 1)));
#pragma unroll
      for (int k = 0; k < kResPool; ++k) {
        const uint32_t i = id + k * kResThreads;
        if (k * static_cast<uint32_t>(kResThreads) >= n) continue;
        if (all_new) {
          if (i < n) rk.ckey[slot_of_entry(i)] = score_of[k];
        } else {
          const bool beats = i < n && score_of[k] < thresh;
          const uint64_t mask = __ballot(beats);
          if (mask == 0) continue;
          uint32_t at = 0;
          if (lane0 == 0) at = atomicAdd(&rk.misc[0], static_cast<uint32_t>(__popcll(mask)));
          at = __builtin_amdgcn_readfirstlane(at) + static_cast<uint32_t>(__popcll(mask & ((1ull << lane0) - 1ull)));
          if (beats) { rk.ckey[K + at] = score_of[k]; rk.lslot[at] = static_cast<uint16_t>(K + i); }
        }
      }
    }
    __syncthreads();

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
    if (last && blockIdx.x == 0)
      for (uint32_t e = tid; e < K; e += kResThreads) {
        a.row_of[e] = rk.srow[e];
        if (!all_new) shared_store(reinterpret_cast<uint64_t *>(a.fit_row) + rk.srow[e], rk.ckey[e]);
      }

    // ---- rank the pool
    const uint32_t M = all_new ? 0u : rk.misc[0];
    bool crowded = false;                            // so many children share a place that the whole pool is ranked
    if (!all_new && M == 0) {
      // no child beats the K-th survivor: same survivors, same order, same rows
      if (last && blockIdx.x != 0) return;
      if (last) for (uint32_t e = tid; e < K; e += kResThreads) ra.sel[e] = static_cast<int32_t>(e);
    } else if (!all_new) {
      const uint32_t id = opaque(tid);
      // A child's place: the survivors with a score at or below its own.
      uint32_t place[kResKids];                      // and, above it, how many children came to that place before
#pragma unroll
      for (int k = 0; k < kResKids; ++k) {
        const uint32_t i = id + k * kResThreads;
        if (k * static_cast<uint32_t>(kResThreads) >= M) break;      // whole workgroup
        if (i >= M) continue;
        const uint64_t key = rk.ckey[K + i];
        uint32_t lo = 0, hi = K - 1;                 // it beats the K-th
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (rk.ckey[mid] <= key) lo = mid + 1; else hi = mid;
        }
        place[k] = lo | atomicAdd(&rk.place[lo], 1u) << 16;
      }
      __syncthreads();
      {                                              // running sum over the places
        const uint32_t per = (K + kResThreads - 1) / kResThreads, e0 = id * per;
        uint32_t n[kResElites], sum = 0, unused = 0;
#pragma unroll
        for (int i = 0; i < kResElites; ++i) {
          n[i] = static_cast<uint32_t>(i) < per && e0 + i < K ? rk.place[e0 + i] : 0u;
          if (n[i] > kResPlace) rk.misc[1] = 1;
          sum += n[i];
        }
        sums_before(rk, sum, unused);
#pragma unroll
        for (int i = 0; i < kResElites; ++i) {
          sum += n[i];
          if (static_cast<uint32_t>(i) < per && e0 + i < K) rk.place[e0 + i] = sum;
        }
      }
      __syncthreads();
      crowded = rk.misc[1] != 0;
      // in the last generation only the first workgroup needs the ranking (it writes the state the call
      // leaves); the others stay for their share of a ranking by counting, if there is one
      if (last && blockIdx.x != 0 && !crowded) return;
      if (!crowded) {
        // the children in the order of their places, ...
        auto before = [&](uint32_t pos) { return pos ? rk.place[pos - 1] : 0u; };
#pragma unroll
        for (int k = 0; k < kResKids; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i < M) rk.order[before(place[k] & 0xFFFFu) + (place[k] >> 16)] = static_cast<uint16_t>(i);
        }
        __syncthreads();
        // ... those of one place ranked among themselves.  A child that comes b-th takes rank b + its place, and
        // if that is below K its slot the row of the last survivor but b, which drops out.
        uint32_t rows[kResKids];                     // its row and, above it, the slot's next one
#pragma unroll
        for (int k = 0; k < kResKids; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i >= M) continue;
          const uint32_t pos = place[k] & 0xFFFFu, first = before(pos), end = rk.place[pos], slot = rk.lslot[i];
          uint32_t b = first;
          if (end - first > 1) {
            const uint64_t key = rk.ckey[K + i];
            for (uint32_t q = first; q < end; ++q) {
              const uint32_t o = rk.order[q];
              b += key_less(rk.ckey[K + o], rk.lslot[o], key, slot) ? 1u : 0u;
            }
          }
          place[k] = pos + b;                        // its rank
          rows[k] = rk.frow[slot - K] | static_cast<uint32_t>(rk.srow[b < K ? K - 1 - b : 0u]) << 16;
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
        for (int k = 0; k < kResKids; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= M) break;
          const uint32_t i = id + k * kResThreads;
          if (i >= M || place[k] >= K) continue;
          const uint32_t slot = rk.lslot[i];
          rk.ckey[place[k]] = rk.ckey[K + i];
          rk.srow[place[k]] = static_cast<uint16_t>(rows[k]);
          rk.frow[slot - K] = static_cast<uint16_t>(rows[k] >> 16);
          if (last) ra.sel[place[k]] = static_cast<int32_t>(slot);
        }
#pragma unroll
        for (int k = 0; k < kResElites; ++k) {
          const uint32_t e = id + k * kResThreads;
          if (e < K) rk.place[e] = 0;
          if (elite_rank[k] >= K) continue;
          rk.ckey[elite_rank[k]] = elite_key[k];
          rk.srow[elite_rank[k]] = static_cast<uint16_t>(elite_row[k]);
          if (last) ra.sel[elite_rank[k]] = static_cast<int32_t>(e);
        }
        __syncthreads();
      }
    }
    if (all_new || crowded) {
      const uint32_t id = opaque(tid);
      if (!all_new) {
        // the children's scores by slot, from where they were published, with the survivors' in front of them
#pragma unroll
        for (int k = 0; k < kResPool; ++k) {
          const uint32_t i = id + k * kResThreads;
          if (i < 3 * K) rk.ckey[K + i] = score_of[k] = shared_load(xk + K + i);
          else if (i < P) score_of[k] = rk.ckey[i - 3 * K];
        }
        for (uint32_t e = id; e < K; e += kResThreads) rk.place[e] = 0;
        __syncthreads();
      }
      // Every candidate's slot goes to its rank in nsel.  In a pool of more than kResLocal each workgroup ranks a
      // range of the order, between two quantiles of a sample of the pool, (score, slot) pairs: it counts the
      // candidates below, ranks those inside against each other, and the workgroups exchange the slots by rank.
      const bool local = P <= kResLocal;
      uint32_t n_below = 0, n_inside = P;
      if (!local) {
        auto sampled_slot = [&](uint32_t q) { return q * P / kResSample; };
        {
          // (counted in vector registers: one wave's ballot after the other, added up by the scalar unit that the
          // waves share, took twice as long)
          constexpr uint32_t kParts = kResThreads / kResSample, kPer = kResSample / kParts;
          const uint32_t i = id % kResSample, part = id / kResSample;       // the part is the wave's
          const uint64_t key = rk.ckey[sampled_slot(i)];
          uint32_t n = 0;
#pragma unroll
          for (uint32_t v = 0; v < kPer; ++v) {
            const uint32_t q = part * kPer + v;
            n += rk.ckey[sampled_slot(q)] < key + (q < i ? 1u : 0u) ? 1u : 0u;      // (scores are integers below 2^63 here)
          }
          if (n) atomicAdd(&rk.place[i], n);
        }
        __syncthreads();
        // this workgroup's range: from the sample point of rank b S / n on, up to that of rank (b + 1) S / n
        const uint32_t lo = blockIdx.x * kResSample / n_groups, hi = (blockIdx.x + 1) * kResSample / n_groups;
        if (id < kResSample) {
          const uint32_t r = rk.place[id];
          if (r == lo) rk.range[0] = sampled_slot(id);
          if (r == hi) rk.range[1] = sampled_slot(id);
        }
        if (id == kResThreads - 1) rk.range[2] = rk.range[3] = 0;
        __syncthreads();
        if (id < kResSample) rk.place[id] = 0;
        const uint32_t lo_slot = rk.range[0], hi_slot = rk.range[1];
        const uint64_t lo_key = lo == 0 ? 0ull : rk.ckey[lo_slot], hi_key = hi == kResSample ? ~0ull : rk.ckey[hi_slot];
#pragma unroll
        for (int k = 0; k < kResPool; ++k) {
          if (k * static_cast<uint32_t>(kResThreads) >= P) continue;
          const uint32_t i = id + k * kResThreads, slot = slot_of_entry(i);
          const bool real = i < P;
          const bool below = real && lo != 0 && score_of[k] < lo_key + (slot < lo_slot ? 1u : 0u);
          const bool inside = real && !below && (hi == kResSample || score_of[k] < hi_key + (slot < hi_slot ? 1u : 0u));
          n_below += below ? 1u : 0u;
          const uint64_t mask = __ballot(inside);
          if (mask == 0) continue;
          uint32_t at = 0;
          if (lane0 == 0) at = atomicAdd(&rk.range[3], static_cast<uint32_t>(__popcll(mask)));
          at = __builtin_amdgcn_readfirstlane(at) + static_cast<uint32_t>(__popcll(mask & ((1ull << lane0) - 1ull)));
          if (inside) rk.all[at] = static_cast<uint16_t>(slot);
        }
        n_below = wave_sum(n_below);
        if (lane0 == 0 && n_below != 0) atomicAdd(&rk.range[2], n_below);
        __syncthreads();
        n_below = rk.range[2];
        n_inside = n_below < K ? rk.range[3] : 0u;   // otherwise nothing of this range survives
      }
      const uint64_t stamp = static_cast<uint64_t>(use + 1u) << 32;     // no generation has number 0
      auto listed = [&](uint32_t q) { return local ? q : static_cast<uint32_t>(rk.all[q]); };
      auto put = [&](uint32_t rank, uint32_t slot) {
        if (rank >= K) return;
        if (local) rk.nsel[rank] = static_cast<uint16_t>(slot);
        else shared_store(ra.xrank + rank, stamp | slot);
      };
      uint32_t *below = rk.place + 2 * kResInside;
      if (n_inside <= kResInside) {
        // thread (i, part): candidate i against candidates part, part + parts, ..., whose scores lie together
        uint64_t *inside = reinterpret_cast<uint64_t *>(rk.place);
        if (!local) {
          if (id < n_inside) inside[id] = rk.ckey[rk.all[id]];
          __syncthreads();
        }
        const uint64_t *keys = local ? rk.ckey : inside;
        const uint32_t width = pow2_at_least(n_inside), parts = kResThreads / width, i = id % width, part = id / width;
        const uint32_t slot = i < n_inside ? listed(i) : 0u;
        if (i < n_inside) {
          const uint64_t key = keys[i];
          uint32_t n = 0;
#pragma unroll 4
          for (uint32_t q = part; q < n_inside; q += parts) n += keys[q] < key + (listed(q) < slot ? 1u : 0u) ? 1u : 0u;
          if (n) atomicAdd(&below[i], n);
        }
        __syncthreads();
        if (id < n_inside) {                         // part 0
          put(n_below + below[i], slot);
          below[i] = 0;
          if (!local) inside[id] = 0;
        }
      } else {
        for (uint32_t i = id; i < n_inside; i += kResThreads) {
          const uint32_t slot = rk.all[i];
          const uint64_t key = rk.ckey[slot];
          uint32_t n = 0;
#pragma unroll 8
          for (uint32_t q = 0; q < n_inside; ++q) {
            const uint32_t other = rk.all[q];
            n += rk.ckey[other] < key + (other < slot ? 1u : 0u) ? 1u : 0u;
          }
          put(n_below + n, slot);
        }
      }
      __syncthreads();
      if (last && blockIdx.x != 0) return;
      if (!local) {
        static_assert(kResElites == 2, "entries per thread");
        auto entry = [&](uint32_t e) { return ra.xrank + e; };
        auto ready = [&](uint32_t, uint64_t v) { return (v >> 32) == (stamp >> 32); };
        auto take = [&](uint32_t e, uint64_t v, bool now) { if (now) rk.nsel[e] = static_cast<uint16_t>(v); };
        const bool ranked = K <= static_cast<uint32_t>(kResThreads) ? gather_per<1, kResThreads>(K, ra.spin_limit, entry, ready, take)
                                                                    : gather_per<2, kResThreads>(K, ra.spin_limit, entry, ready, take);
        if (__syncthreads_or(ranked ? 0 : 1)) return give_up();
      }
      settle(rk, P, changed, last ? ra.sel : nullptr);
    }
    if (last) {
      // the state the next call (of either kind) starts from
      for (uint32_t e = tid; e < K; e += kResThreads) {
        ra.parent_rows[e] = rk.srow[e];
        a.spare[e] = rk.frow[3 * K + e];
      }
      for (uint32_t u = tid; u < 3 * K; u += kResThreads) a.row_of[K + u] = rk.frow[u];
      return;
    }
  }
}

template <int Q, Genes kGenes>
hipError_t launch_genes(const ResidentArgs &args, const ResidentPlan &plan, hipStream_t stream) {
  const bool over = args.ev.per_gpu != 0, sampled = args.sampled != 0;
  const void *fn = over ? (sampled ? reinterpret_cast<const void *>(resident_kernel<Q, kGenes, true, true>)
                                   : reinterpret_cast<const void *>(resident_kernel<Q, kGenes, true, false>))
                        : (sampled ? reinterpret_cast<const void *>(resident_kernel<Q, kGenes, false, true>)
                                   : reinterpret_cast<const void *>(resident_kernel<Q, kGenes, false, false>));
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
bool resident_plan(const EvolveArgs &ev, bool sampled, int n_cus, ResidentPlan &plan) {
  const uint32_t Q = static_cast<uint32_t>(words_of(static_cast<int>(ev.Jp / kLanes))), K = ev.P / 4;
  if (Q > static_cast<uint32_t>(kResidentMaxWords) || ev.P > static_cast<uint32_t>(kResidentMaxPool) || ev.P < 4) return false;
  // A wave of every SIMD computes; where the pool has more candidates than those of the whole chip, more do, all for
  // the same number of rounds.
  const uint32_t units = (sampled ? 4 : 3) * K;
  plan.groups = std::min<uint32_t>({static_cast<uint32_t>(n_cus), kResidentMaxGroups, (units + 3) / 4});
  const uint32_t per_group = (units + plan.groups - 1) / plan.groups, rounds = (per_group + kResWaves - 1) / kResWaves;
  plan.unit_waves = std::min<uint32_t>(kResWaves, ((per_group + rounds - 1) / rounds + 3) / 4 * 4);
  plan.groups = std::min<uint32_t>(plan.groups, (units + plan.unit_waves - 1) / plan.unit_waves);
  const uint32_t n_waves = plan.groups * plan.unit_waves;
  plan.child_units = (3 * K + n_waves - 1) / n_waves;
  plan.coin_stride = coin_stride(ev);
  plan.table_lds = static_cast<uint32_t>((table_bytes(Q, ev.tab.term_E, plan.unit_waves, plan.coin_stride) + 15) & ~size_t(15));
  plan.lds = plan.table_lds + ranking_bytes(Q, ev.P, plan.unit_waves, plan.child_units);
  return plan.lds <= kLdsBudget;
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
