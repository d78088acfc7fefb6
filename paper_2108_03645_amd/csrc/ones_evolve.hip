// Evolve kernel of the ONES search (arXiv 2108.03645, Section 3.2.2) for gfx950.
//
// One wave64 owns one pool slot (a crossover wave owns the two children of a pair): the
// job columns lie across the 64 lanes, the rows of a column in a lane's registers.  The
// wave composes the candidate from the survivors of the previous generation (refresh copy,
// uniform crossover, uniform mutation), repairs it to the cluster capacity (refresh + fill
// under Eq. 4), scores it (Eq. 3 with T = Y/X, Eq. 5) and writes genome and score.
//
// Workgroups are persistent: each owns a contiguous share of the work and stages the job table, the
// draws and the rows of the slots it will fill in LDS; then its waves take the share's items one by
// one from an LDS counter and never wait for each other.
#include "ones_candidate.h"

#ifndef ONES_ROW_GROUP
#error "compile with -DONES_ROW_GROUP=0..3"
#endif

namespace ones {
namespace {

constexpr int kGroupFirst = 2 * ONES_ROW_GROUP + 1;   // words per lane kGroupFirst, kGroupFirst + 1

// ----------------------------------------------------------------- kernels ---------
template <int Q> struct Shape { static constexpr int kWaves = Q > 4 ? 16 : 8; };

template <int Q, Genes kGenes, bool kArrivals, bool kWalk>
__device__ __forceinline__ double finish(const EvolveArgs &a, const Smem &s, uint32_t dst_row, uint32_t lr, uint32_t ir,
                                         uint32_t (&c)[Q], int lane, uint8_t *window) {
  repair<Q, kGenes, kArrivals>(c, s, a.G, lr, ir, lane, a.Jp, kArrivals && a.time_rank != nullptr, window, kWalk && a.walk != 0);
  phase_fence();
  const double f = score<Q>(c, s, a.term_lds, lane);
  phase_fence();
  uint32_t *row = a.genes + static_cast<size_t>(dst_row) * (Q * kLanes);
#pragma unroll
  for (int q = 0; q < Q; ++q) row[q * kLanes + lane] = c[q];
  if (lane == 0) a.fit_row[dst_row] = f;
  return f;
}

// Initial population G_0: every gene uniform over {waiting, bmin..bmax}.
// (Argument block: one EvolveArgs by value, see kernel_args.)
template <int Q, Genes kGenes, bool kWalk>
__global__ __launch_bounds__(Shape<Q>::kWaves *kLanes) void init_kernel(EvolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const Smem s = carve<Q>(smem_raw, a.term_lds, Shape<Q>::kWaves, a.coin_stride, kWalk && a.walk != 0);
  stage_table<Q>(a, s, a.term_lds, false, threadIdx.x, blockDim.x, kWalk && a.walk != 0);
  uint8_t *window = s.coins + static_cast<size_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * a.coin_stride;
  if (threadIdx.x == 0) *s.next_item = 0;
  __syncthreads();
  const int lane0 = threadIdx.x & (kLanes - 1);
  const uint32_t R = a.Jp / kLanes;
  // The workgroup owns a contiguous share of the slots; its waves take them one by one from an
  // LDS counter (random genomes differ widely in the fill rounds their repair needs).
  const uint32_t first = static_cast<uint32_t>(static_cast<uint64_t>(a.P) * blockIdx.x / gridDim.x);
  const uint32_t last = static_cast<uint32_t>(static_cast<uint64_t>(a.P) * (blockIdx.x + 1) / gridDim.x);
  for (;;) {
    const int lane = opaque(lane0);
    uint32_t taken = 0;
    if (lane == 0) taken = atomicAdd(s.next_item, 1u);
    const uint32_t p = first + static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(taken));
    if (p >= last) break;
    const uint32_t r = __builtin_amdgcn_readfirstlane(candidate_draw(a, a.t, p).r);
    const WordSource words(a, a.t, p, Q > 1);
    uint32_t c[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const Words w = words.block(s.prefix, q, lane);
      const uint32_t n = s.draws[q * kLanes + lane];
      uint32_t k = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) k |= bounded(w.w[u], (n >> (8 * u)) & 0xFFu) << (8 * u);
      c[q] = codes_of_draws(s, q * kLanes + lane, k);
    }
    phase_fence();
    const double f = finish<Q, kGenes, false, kWalk>(a, s, p, r / R, r % R, c, lane, window);   // slot p starts in row p
    note_slot_score(p, f, lane);
    if (lane == 0) a.row_of[p] = p;
  }
}

// One generation.  Work items: K crossover pairs, K mutants and, after a table change, the K
// survivors to refresh (or, when only the remaining work changed, to score again).  kSame: the
// job table has not changed since the previous generation was repaired and scored, so a survivor is
// a fixed point of the repair with the same score: it stays in its row untouched, and stored genes
// hold as they are.  kChanged: the first generation under a new table; kArrivals: the same, and the
// jobs that arrived with it are served first.  kOverGpus: the uniform crossover scans the GPUs instead of the jobs.
// (Argument block: one EvolveArgs by value, see kernel_args.)
enum Table { kSame, kChanged, kArrivals };
template <int Q, Table kTable, bool kOverGpus, Genes kGenes, bool kWalk>
__global__ __launch_bounds__(Shape<Q>::kWaves *kLanes) void evolve_kernel(EvolveArgs a) {
  constexpr bool kSameTable = kTable == kSame;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const Smem s = carve<Q>(smem_raw, a.term_lds, Shape<Q>::kWaves, a.coin_stride, kWalk && a.walk != 0);
  const int lane0 = threadIdx.x & (kLanes - 1);
  const bool assigned = a.assigned != 0;
  if (!assigned) {
    const IndexLoads index_loads = index_free_rows_begin(a, lane0);
    index_free_rows_end(a, s, index_loads, lane0);
  }
  const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t K = a.K;
  uint8_t *window = s.coins + static_cast<size_t>(wave_in_block) * a.coin_stride;     // this wave's scratch
  uint64_t *coins = reinterpret_cast<uint64_t *>(window);
  // This workgroup's share of the ranks 0..K-1: for each rank a pair, a mutant and, after a
  // table change, a survivor, a round of kRound ranks at a time.  The rows the round fills are read
  // where the selection has assigned them; otherwise the slots K + 2 ra .., 3K + ra .. and the ranks
  // ra .. take three runs of consecutive free rows, which one wave each lists into LDS while the
  // others stage the job table and make the slots' draws, a lane per slot (a wave that drew for its
  // own item spent a tenth of its time on a Philox block per slot with the same numbers in all lanes).
  const uint32_t first = static_cast<uint32_t>(static_cast<uint64_t>(K) * blockIdx.x / gridDim.x);
  const uint32_t last = static_cast<uint32_t>(static_cast<uint64_t>(K) * (blockIdx.x + 1) / gridDim.x);
  const uint32_t listing = assigned ? 0u : 3u * kLanes;          // threads that only list
  constexpr uint32_t kDrawn = kSameTable ? 3 : 4;                // slots per rank that are drawn for
  auto slot_at = [&](uint32_t ra, uint32_t n, uint32_t i) {      // the i-th slot of a round
    return i < 2 * n ? K + 2 * ra + i : i < 3 * n ? 3 * K + ra + (i - 2 * n) : ra + (i - 3 * n);
  };
  auto prepare_round = [&](uint32_t ra, uint32_t n) {
    if (threadIdx.x < listing) {
      if (wave_in_block == 0) list_free_rows(a, s, 2 * ra, 2 * n, s.rows, lane0);
      if (wave_in_block == 1) list_free_rows(a, s, 2 * K + ra, n, s.rows + 2 * n, lane0);
      if (wave_in_block == 2) list_free_rows(a, s, 3 * K + ra, n, s.rows + 3 * n, lane0);
      return;
    }
    const uint32_t R = a.Jp / kLanes;
    for (uint32_t i = threadIdx.x - listing; i < 4 * n; i += blockDim.x - listing) {
      const uint32_t p = slot_at(ra, n, i);
      uint32_t row = 0;
      if (assigned) row = i < 3 * n ? a.row_of[p] : a.spare[p];
      if (i < kDrawn * n) {
        Draw d = candidate_draw(a, a.t, p);
        if (p < K) d.ra = d.rb = p;                              // a survivor is its own parent
        s.drawn[i] = pack_draw(min(a.parent_row[d.ra], a.P + K - 1), min(a.parent_row[d.rb], a.P + K - 1), d.r, R);
      }
      if (assigned) s.rows[i] = checked_row(row, a.P + K);
    }
  };
  if (first < last) prepare_round(first, min(kRound, last - first));
  if (threadIdx.x >= listing) stage_table<Q>(a, s, a.term_lds, !kSameTable, threadIdx.x - listing, blockDim.x - listing, kWalk && a.walk != 0);
  if (kSameTable && threadIdx.x < static_cast<uint32_t>(kTieClasses)) tie_counts(s, a.term_lds)[threadIdx.x] = 0;
  if (a.occupied_other != nullptr)
    for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < (a.P + K + 31) / 32; w += gridDim.x * blockDim.x)
      a.occupied_other[w] = 0;
  for (uint32_t ra = first; ra < last; ra += kRound) {
  const uint32_t n = min(kRound, last - ra);
  if (ra != first) {
    __syncthreads();                                 // the previous round's rows have been used
    prepare_round(ra, n);
  }
  if (threadIdx.x == blockDim.x - 1) *s.next_item = 0;
  __syncthreads();
  // record what the slots and ranks got
  for (uint32_t i = threadIdx.x; i < 4 * n; i += blockDim.x) {
    const uint32_t p = slot_at(ra, n, i);
    if (i < 3 * n) {
      if (!assigned) a.row_of[p] = checked_row(s.rows[i], a.P + K);
    } else {
      const uint32_t row = checked_row(s.rows[i], a.P + K), old = a.parent_row[p];
      a.row_of[p] = kSameTable ? old : row;
      if (!kSameTable) a.spare[p] = old;
      else if (!assigned) a.spare[p] = row;
    }
  }
  const uint32_t kinds = (!kSameTable || a.rescore) ? 3u : 2u;
  // The waves take the items one by one (the pairs first: they take twice as long), so that a
  // wave whose items needed many fill rounds does not hold the others up at the end.
  for (;;) {
    const int lane = opaque(lane0);
    uint32_t taken = 0;
    if (lane == 0) taken = atomicAdd(s.next_item, 1u);
    const uint32_t idx = __builtin_amdgcn_readfirstlane(taken);
    if (idx >= kinds * n) break;
    // pairs first, then mutants, then survivors
    if (kSameTable && idx >= 2 * n) {
      // the remaining work was drawn anew: the survivor of this rank keeps its genome and row
      // and only gets its score under the new draw
      const uint32_t rank = ra + (idx - 2 * n), row = a.parent_row[rank];
      uint32_t c[Q];
      load_genes<Q>(a.genes, row, lane, c);
      const double f = score<Q>(c, s, a.term_lds, lane);
      if (lane == 0) a.fit_row[row] = f;
      note_slot_score(rank, f, lane);
      continue;
    }
    uint32_t i = idx < n ? 2 * idx : idx + n;                    // the item's (first) slot in the round
    uint32_t children = 1;
    PackedDraw d = draw_at(s.drawn, i);
    uint32_t c[Q], other[Q];
    load_genes<Q>(a.genes, d.row_a(), lane, c);
    if (idx < n) {
      // uniform crossover: per gene the children swap their parents' genes with rate chi
      children = 2;
      const uint32_t p0 = slot_at(ra, n, i);
      load_genes<Q>(a.genes, d.row_b(), lane, other);
      if (kOverGpus) {
        if (!kSameTable) { to_new_table<Q>(s, lane, c); to_new_table<Q>(s, lane, other); }
        phase_fence();
        crossover_over_gpus<Q, kSameTable>(a, a.t, s, coins, p0, lane, c, other);
      } else {
        const WordSource words(a, a.t, p0, Q > 1);
        uint32_t swap[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          swap[q] = words_below(words.block(s.prefix, q, lane), a.T_x);
          if (q % 2 == 1) { pin(swap[q]); phase_fence(); }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t mine = c[q];
          c[q] = pick(swap[q], other[q], mine);
          other[q] = pick(swap[q], mine, other[q]);
        }
        if (!kSameTable) { to_new_table<Q>(s, lane, c); to_new_table<Q>(s, lane, other); }
      }
    } else {
      if (!kSameTable) to_new_table<Q>(s, lane, c);
      if (idx < 2 * n) {
        // uniform mutation: each job redrawn with rate theta (k = 0 pre-empts it)
        const WordSource words(a, a.t, slot_at(ra, n, i), Q > 1);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const Words w = words.block(s.prefix, q, lane);
          const uint32_t k = outcomes_drawn(w, s.draws[q * kLanes + lane]);
          c[q] = pick(words_below(w, a.T_mut), codes_of_draws(s, q * kLanes + lane, k), c[q]);
          if (q % 2 == 1) { pin(c[q]); phase_fence(); }
        }
      }
      // (else the survivor of this rank, projected onto the new job table; it goes to one of the last
      // K free rows: its old row is still being read as a parent by other waves)
    }
    phase_fence();
    for (;;) {
      const uint32_t p = slot_at(ra, n, i);
      const double f = finish<Q, kGenes, kTable == kArrivals, kWalk>(a, s, row_at(s, i, a), d.lane(), d.row(), c, lane, window);
      if (kSameTable && a.bk.nb != 0) drop_in_bucket(s, p, f, lane); else note_slot_score(p, f, lane);
      if (--children == 0) break;
      phase_fence();
#pragma unroll
      for (int q = 0; q < Q; ++q) c[q] = other[q];
      d = draw_at(s.drawn, ++i);
    }
  }
  }
  if (kSameTable && a.bk.nb != 0) {                  // one count a workgroup and class of copies, not one a child
    __syncthreads();
    uint32_t *counts = tie_counts(s, a.term_lds);
    const uint32_t copies = threadIdx.x < static_cast<uint32_t>(kTieClasses) ? counts[threadIdx.x] : 0u;
    if (copies != 0) {
      atomicAdd(&a.bk.count[kTieCount + threadIdx.x], copies);
      a.bk.count[kTieBucket + threadIdx.x] = tie_buckets(counts)[threadIdx.x];
      a.bk.count[kTieFlag] = 1;
    }
  }
}

template <typename Kernel>
hipError_t launch_persistent(Kernel k, EvolveArgs a, int words, int waves, uint32_t items, uint32_t max_blocks, int n_cus,
                             hipStream_t s) {
  // the term table goes to LDS when it fits beside the rest
  const uint32_t rows = a.P + a.K;
  a.coin_stride = coin_stride(a);
  a.term_lds = (a.tab.term_E != 0 && smem_bytes(words, waves, a.tab.term_E, rows, a.coin_stride) <= kLdsBudget)
                   ? a.tab.term_E : 0u;
  size_t lds = smem_bytes(words, waves, a.term_lds, rows, a.coin_stride);
  if (lds > kLdsBudget) return hipErrorInvalidValue;
  // as many workgroups as can be resident (limited by LDS and registers), at most one wave per item.  Of eight waves
  // three, though a fourth has room: what it costs to stage its tables is more than its waves hide
  // (epochs of 10 sampled generations, 130 slots, pool 16384: 526 us with four, 485 with three, 492 with
  // two; pool 65536: 845, 799, 841; unsampled 512 slots, 16384: 19 us a generation's launch with four, 16.5 with three).
  // Of sixteen, whose waves take 71 to 128 registers, one: a second would come after it and stage the tables again (six generations of
  // 32768 candidates, jobs of one GPU at most: 1260 slots 227 us with two workgroups to a compute unit, 200 with one; 2028 299
  // and 259; crossover over 3072 GPUs 311 and 259, 433 and 360).
  const size_t resident = waves == 8 ? 3 : 1;
  auto places = [&](size_t bytes) { return std::max<size_t>(1, std::min<size_t>(kLdsBudget / lds_taken(bytes), resident)); };
  // The repair walks where it fits beside that, with two workgroups in place of three if need be (six generations of 32768
  // candidates: 492 slots, jobs of up to 32 GPUs, crossover over 2816: 225 us walking, 237 with three workgroups; 748 slots, 8 GPUs, over
  // 768: 231 and 287), but not with one in place of two (492 slots, 4096 GPUs, over 2304: 325 and 275; 748, 64, over 5376: 338 and 306),
  // unless the items need no two.
  const uint32_t scratch = std::max<uint32_t>(a.coin_stride, window_bytes(words));
  const size_t walking = smem_bytes(words, waves, a.term_lds, rows, scratch, true);
  const uint32_t groups = std::max<uint32_t>(1u, std::min<uint32_t>((items + waves - 1) / waves, max_blocks));
  const size_t needed = std::min<size_t>({places(lds), (groups + n_cus - 1) / n_cus, 2});
  a.walk = a.walk != 0 && walking <= kLdsBudget && places(walking) >= needed ? 1u : 0u;
  if (a.walk) { a.coin_stride = scratch; lds = walking; }
  const uint32_t blocks = std::min<uint32_t>(groups, static_cast<uint32_t>(n_cus * places(lds)));
  hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      static_cast<int>(lds));
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(waves * kLanes), lds, s, a);
  return hipGetLastError();
}

template <int Q, Genes kGenes, bool kWalk>
hipError_t launch_words_of(const EvolveArgs &a, bool same_table, int n_cus, hipStream_t s) {
  constexpr int kWaves = Shape<Q>::kWaves;
  if (a.t == 0) return launch_persistent(init_kernel<Q, kGenes, kWalk>, a, Q, kWaves, a.P, a.P, n_cus, s);
  const uint32_t items = (!same_table || a.rescore ? 3 : 2) * a.K;       // a share of the ranks each
  const Table table = same_table ? kSame : a.new_first ? kArrivals : kChanged;
  auto launch = [&](auto kernel) { return launch_persistent(kernel, a, Q, kWaves, items, a.K, n_cus, s); };
  switch (table) {
    case kSame: return a.per_gpu ? launch(evolve_kernel<Q, kSame, true, kGenes, kWalk>) : launch(evolve_kernel<Q, kSame, false, kGenes, kWalk>);
    case kChanged: return a.per_gpu ? launch(evolve_kernel<Q, kChanged, true, kGenes, kWalk>) : launch(evolve_kernel<Q, kChanged, false, kGenes, kWalk>);
    default: return a.per_gpu ? launch(evolve_kernel<Q, kArrivals, true, kGenes, kWalk>) : launch(evolve_kernel<Q, kArrivals, false, kGenes, kWalk>);
  }
}

template <int Q, Genes kGenes>
hipError_t launch_words(const EvolveArgs &a, bool same_table, int n_cus, hipStream_t s) {
  if constexpr (Q <= 4) {
    if (a.walk == 0) return launch_words_of<Q, kGenes, false>(a, same_table, n_cus, s);
  }
  return launch_words_of<Q, kGenes, true>(a, same_table, n_cus, s);
}

template <int Q>
hipError_t launch_width(const EvolveArgs &a, bool same_table, int n_cus, hipStream_t s) {
  const uint32_t largest = a.tab.term_E - 1;         // largest code under this table
  if (largest <= kNarrowCodes) return launch_words<Q, kNarrow>(a, same_table, n_cus, s);
  return largest <= kMiddleCodes ? launch_words<Q, kMiddle>(a, same_table, n_cus, s) : launch_words<Q, kWide>(a, same_table, n_cus, s);
}

}  // namespace

// This file is compiled once per group of two word counts (-DONES_ROW_GROUP=0..3) so that the
// instantiations build in parallel.
#define ONES_CONCAT2(x, y) x##y
#define ONES_CONCAT(x, y) ONES_CONCAT2(x, y)
hipError_t ONES_CONCAT(launch_evolve_group, ONES_ROW_GROUP)(const EvolveArgs &a, int words, bool same_table,
                                                            int n_cus, hipStream_t s) {
  if (words == kGroupFirst) return launch_width<kGroupFirst>(a, same_table, n_cus, s);
  if (words == kGroupFirst + 1) return launch_width<kGroupFirst + 1>(a, same_table, n_cus, s);
  return hipErrorInvalidValue;
}

}  // namespace ones
