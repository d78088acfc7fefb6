// Selection of the best K candidates (arXiv 2108.03645, Section 3.2.2 "Selection"; Alg. 1:
// the smallest score wins), plus the small table / readout kernels of libones.
//
// Order: ascending (score, pool slot).  A score is a non-negative fp64, so its bit pattern
// read as an unsigned 64-bit integer orders the same way; ties fall to the smaller slot.
#include "ones_device.h"
#include "ones_exchange.h"
#include "ones_sort.h"

#pragma clang fp contract(off)

namespace ones {
namespace {

constexpr int kSortThreads = kSortChunk / 2 > 1024 ? 1024 : kSortChunk / 2;

// Value of lane + n within the lane's row of 16 (DPP row_shl:n), or fallback where that row ends.
template <int N>
__device__ __forceinline__ uint32_t from_lane_above(uint32_t fallback, uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int>(fallback), static_cast<int>(v), 0x100 + N,
                                                           0xF, 0xF, false));
}

// The candidate in genome row `row` takes rank g < K (lanes with valid set): it survives in its
// row, which the bitmap of the general selection notes.  Called by whole
// waves.  Neighbouring lanes whose rows share a word of the bitmap hand their bits to the first
// lane of their run (within a row of 16 lanes), which issues one atomic for all of them: the
// rows of a pool that has stopped changing are neighbours, and one atomic per row would queue
// up on the same few words.  Lanes that share a word without being neighbours simply issue
// their own atomics.
__device__ __forceinline__ void keep_and_mark(const RowPlan &rp, bool valid, uint32_t g, uint32_t row) {
  if (valid) rp.parent_next[g] = row;
  const uint32_t word = valid ? row / 32 : 0xFFFFFFFFu;        // no bitmap has that many words
  uint32_t bits = valid ? 1u << (row % 32) : 0u;
  // after the steps 1, 2, 4, 8 a lane holds the bits of the lanes above it up to the end of its run
  { const uint32_t w = from_lane_above<1>(~word, word), b = from_lane_above<1>(0u, bits); bits |= w == word ? b : 0u; }
  { const uint32_t w = from_lane_above<2>(~word, word), b = from_lane_above<2>(0u, bits); bits |= w == word ? b : 0u; }
  { const uint32_t w = from_lane_above<4>(~word, word), b = from_lane_above<4>(0u, bits); bits |= w == word ? b : 0u; }
  { const uint32_t w = from_lane_above<8>(~word, word), b = from_lane_above<8>(0u, bits); bits |= w == word ? b : 0u; }
  // the lane below (DPP row_shr:1) has another word, or there is none: this lane starts a run
  const uint32_t below = static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(static_cast<int>(~word), static_cast<int>(word), 0x111, 0xF, 0xF, false));
  if (valid && below != word) atomicOr(&rp.occupied[word], bits);
}

// The same for the i-th best child or mutant of a bucketed selection, in pool slot p: the slot is
// handed the row of the last survivor of the selection before but i, which has dropped out (survivors
// keep their order, so as many as there are surviving children drop out, and at the end).
__device__ __forceinline__ void keep_child(const RowPlan &rp, uint32_t g, uint32_t row, uint32_t p, uint32_t i, uint32_t K) {
  rp.parent_next[g] = row;
  rp.row_of[p] = rp.parents[K - 1 - i];
}

// ---------------------------------------------------------------- general path -----
// Pools of at most kRankPoolMax slots: the rank of a candidate is the number of candidates below
// it in (score, slot) order.  Every workgroup loads all scores into LDS and ranks 64 of them:
// lane l of every wave works on element l, each wave over its own sixteenth of the pool (so a
// wave reads one LDS address at a time, a broadcast); ranks below K are survivors.  One launch,
// where the sample sort below takes three; but the comparisons per thread grow with the pool
// (P / 16), and at P = 16384 this takes 75 us where the three launches take 21.
#ifndef ONES_RANK_POOL_MAX
#define ONES_RANK_POOL_MAX 4096
#endif
constexpr uint32_t kRankPoolMax = ONES_RANK_POOL_MAX;
constexpr int kRankPoolPer = 64;
__global__ __launch_bounds__(kSortThreads) void rank_pool_kernel(const double *fit_row, const double *slot_score,
                                                                RowPlan rp, uint32_t P, uint32_t K, int32_t *sel) {
  const uint32_t *row_of = rp.row_of;
  extern __shared__ __align__(16) uint64_t sk[];       // [padded] scores, then [kRankPoolPer] counters
  constexpr uint32_t kTeam = kSortThreads / kRankPoolPer;
  const uint32_t t = threadIdx.x;
  const uint32_t padded = (P + 8 * kTeam - 1) / (8 * kTeam) * (8 * kTeam);     // eight comparisons per step
  uint32_t *below = reinterpret_cast<uint32_t *>(sk + padded);
  constexpr int kAhead = 4;                            // loads in flight per thread
  for (uint32_t base = 0; base < padded; base += kAhead * kSortThreads) {
    uint64_t loaded[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {                 // all loads first
      const uint32_t e = base + t + u * kSortThreads;
      loaded[u] = e < P ? static_cast<uint64_t>(__double_as_longlong(slot_score ? slot_score[e] : fit_row[row_of[e]])) : ~0ull;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (base + t + u * kSortThreads < padded) sk[base + t + u * kSortThreads] = loaded[u];
  }
  if (t < kRankPoolPer) below[t] = 0;
  __syncthreads();
  const uint32_t mine = blockIdx.x * kRankPoolPer + t % kRankPoolPer;
  const uint32_t part = padded / kTeam, from = (t / kRankPoolPer) * part;
  if (mine < P) {
    const uint64_t key = sk[mine];
    uint32_t n = 0;
    for (uint32_t q = from; q < from + part; q += 8) {
#pragma unroll
      for (int u = 0; u < 8; ++u) n += key_less(sk[q + u], q + u, key, mine) ? 1u : 0u;   // padding is never below
    }
    if (n != 0) atomicAdd(&below[t % kRankPoolPer], n);
  }
  __syncthreads();
  if (t < kRankPoolPer) {                              // one whole wave
    const bool in = mine < P && below[t] < K;
    if (in) sel[below[t]] = static_cast<int32_t>(mine);
    keep_and_mark(rp, in, below[t], in ? row_of[mine] : 0u);
  }
}

// ----------------------------------------------------------- quantile buckets ------
// While the job table stays the same, the K survivors reappear in the next pool with the same
// scores, already in rank order (slots 0..K-1).  Their scores at ranks r_c = c*K/nb therefore
// split the next pool into nb buckets that each hold K/nb survivors; the evolve kernel drops
// every child or mutant that beats the K-th survivor into its bucket, and one workgroup per
// bucket sorts those few and merges them with its survivors.  Buckets concatenate to the
// global order.

// Records the next generation's splitters when an element lands on a boundary rank.
__device__ __forceinline__ void note_rank(uint32_t g, uint64_t bits, uint32_t K, uint32_t nb, uint64_t *split,
                                          uint64_t *thresh) {
  if (g == K - 1) *thresh = bits;
  const uint32_t c = (g * nb) / K;                   // g < 2^20, nb <= 1024
  if (c >= 1 && bucket_bound(c, K, nb) == g) split[c - 1] = bits;
  if (c + 1 < nb && bucket_bound(c + 1, K, nb) == g) split[c] = bits;
}

constexpr int kBucketThreads = 256;
constexpr int kBucketLds = 2048;      // offspring of one bucket that are sorted in LDS
constexpr int kBucketCount = kManyInBucket;   // up to here offspring are ranked by counting, not sorted
constexpr int kBucketElites = 1025;   // survivors of one bucket: at most ceil(2^18 / 256) + 1

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, kLanes);
  return v;
}

// A bucket's copies of a class of survivors (see kTieRun): n children with the score of the bucket's first survivor, ranked
// behind the survivors with that score and before all other offspring of the bucket.
struct Copies {
  uint32_t n = 0;
  uint64_t key = 0;
  __device__ __forceinline__ uint32_t before(uint64_t survivor) const { return survivor > key ? n : 0u; }
};

// Ranks one bucket: offspring in (sk, si)[0..n) (padded with never-smaller keys up to npad, a
// multiple of 8), survivors' score bits in ek[0..ne).  Writes the survivor list entries that
// fall below K and notes the next generation's splitters.
template <bool kElites, int kThreads>
__device__ __forceinline__ void rank_bucket(const uint64_t *sk, const uint32_t *si, const uint64_t *ek, uint32_t n, uint32_t npad,
                                            uint32_t ne, uint32_t e0, uint32_t off, bool sorted, uint32_t K,
                                            const BucketArgs &bk, const RowPlan &rp, const Copies &copies, int32_t *sel) {
  const uint32_t tid = threadIdx.x, nb = bk.nb;
  // offspring i: rank = offspring before it + survivors with score <= its score (a survivor
  // wins a tie: smaller slot)
  for (uint32_t base = 0; base < n; base += kThreads) {   // whole waves go round together
    const uint32_t i = base + tid;
    uint32_t g = K, row = 0;
    if (i < n) {
      const uint64_t key = sk[i];
      const uint32_t id = si[i];
      row = rp.row_of[id];
      uint32_t below = i;
      if (!sorted) {
        // scores alone decide nearly every comparison: count the smaller and the equal ones, and
        // only an element that shares its score looks at the slots
        uint32_t equal = 0;
        below = 0;                                   // padding keys are never below a real one
        for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const uint64_t other = sk[q + u];
            below += other < key ? 1u : 0u;
            equal += other == key ? 1u : 0u;
          }
        }
        if (equal > 1)
          for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
            for (int u = 0; u < 8; ++u) below += (sk[q + u] == key && si[q + u] < id) ? 1u : 0u;
          }
      }
      uint32_t lo = 0, hi = ne;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ek[mid] <= key) lo = mid + 1; else hi = mid;
      }
      g = off + copies.n + below + lo;
      if (g < K) {
        sel[g] = static_cast<int32_t>(id);
        if (kElites) {
          note_rank(g, key, K, nb, bk.split_next, bk.thresh_next);
          keep_child(rp, g, row, id, off + copies.n - e0 + below, K);
        }
      }
    }
    if (!kElites) keep_and_mark(rp, g < K, g, row);
  }
  if (!kElites) return;
  // survivor e: rank = e + offspring with a strictly smaller score.  The threads are taken from
  // the top, so that in a small bucket the survivors' waves are not the offspring's.
  for (uint32_t base = 0; base < ne; base += kThreads) {
    const uint32_t e = base + (kThreads - 1 - tid);
    if (e < ne) {
      const uint64_t key = ek[e];
      uint32_t lo = 0;
      if (!sorted) {
        for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
          for (int u = 0; u < 8; ++u) lo += sk[q + u] < key ? 1u : 0u;
        }
      } else {
        uint32_t hi = n;
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (sk[mid] < key) lo = mid + 1; else hi = mid;
        }
      }
      const uint32_t g = off + e + lo + copies.before(key);
      if (g < K) {
        sel[g] = static_cast<int32_t>(e0 + e);
        note_rank(g, key, K, nb, bk.split_next, bk.thresh_next);
        rp.parent_next[g] = rp.parents[e0 + e];
      }
    }
  }
}

// Gathers the bucket's offspring (own storage, then its share of the spill list) into
// (dk, di)[0..n) and pads up to npad.
__device__ __forceinline__ void gather_bucket(uint64_t *dk, uint32_t *di, const BucketArgs &bk, uint32_t b, uint32_t n,
                                              uint32_t npad, uint32_t *lds_counter) {
  const uint32_t tid = threadIdx.x;
  const uint32_t n_main = n < bk.seg ? n : bk.seg;
  const uint64_t *gk = bk.keys + static_cast<size_t>(b) * bk.seg;
  const uint32_t *gi = bk.idx + static_cast<size_t>(b) * bk.seg;
  for (uint32_t e = tid; e < n_main; e += blockDim.x) { dk[e] = gk[e]; di[e] = gi[e]; }
  for (uint32_t e = n + tid; e < npad; e += blockDim.x) { dk[e] = ~0ull; di[e] = 0xFFFFFFFFu; }
  if (n > n_main) {
    const uint32_t spilled = bk.count[kSpillCounter];
    for (uint32_t q = tid; q < spilled; q += blockDim.x) {
      if (bk.spill_bucket[q] == b) {
        const uint32_t at = n_main + atomicAdd(lds_counter, 1u);
        dk[at] = bk.spill_keys[q];
        di[at] = bk.spill_idx[q];
      }
    }
  }
  __syncthreads();
}

constexpr uint32_t kFewCrowded = 8;   // so few crowded buckets may be ranked by counting (see Crowd)

// What the threads of a workgroup that handles buckets share.
template <int kThreads>
struct BucketShared {
  uint64_t sk[kBucketLds];
  uint32_t si[kBucketLds];
  uint64_t ek[kBucketElites];
  uint32_t red[kThreads / kLanes];
  uint32_t below[kThreads];
  uint32_t spill_cursor;
  uint32_t n_many, n_teams;            // buckets above kBucketCount; crowded ones that are dealt to teams
  uint32_t counted[kFewCrowded], n_counted;   // ... that all workgroups rank by counting
  uint32_t helps, member, team;        // the crowded bucket this workgroup helps to rank, as number `member` of `team`
  uint32_t valid, smaller, inside;     // of that bucket: sample points; records below and inside a range
  uint32_t tie_count[kTieClasses], tie_bucket[kTieClasses];   // see BucketArgs
};

// Children in the buckets before o, this thread's share of them: to be added up over the workgroup.
template <int kThreads>
__device__ __forceinline__ uint32_t children_before(const BucketShared<kThreads> &sh, const BucketArgs &bk, bool any_copies, uint32_t o) {
  uint32_t before = 0;
  for (uint32_t c = threadIdx.x; c < o; c += kThreads) before += bk.count[c];
  if (any_copies && threadIdx.x < static_cast<uint32_t>(kTieClasses) && sh.tie_bucket[threadIdx.x] < o) before += sh.tie_count[threadIdx.x];
  return before;
}
// Copies in bucket o.  Called by whole waves.
template <int kThreads>
__device__ __forceinline__ uint32_t copies_in(const BucketShared<kThreads> &sh, uint32_t o) {
  const uint32_t lane = threadIdx.x % kLanes, one = sh.tie_bucket[lane] == o ? sh.tie_count[lane] : 0u;
  const uint32_t n = one + (sh.tie_bucket[kLanes + lane] == o ? sh.tie_count[kLanes + lane] : 0u);     // one of them at most
  const uint64_t found = __ballot(n != 0);
  return found ? __builtin_amdgcn_readlane(n, __ffsll(static_cast<long long>(found)) - 1) : 0u;
}

// Which buckets are crowded, and how they are ranked.  A bucket is crowded when it holds more than a
// workgroup sorts in LDS, or more than it ranks by counting while at most kFewCrowded buckets do (the
// LDS sort of 2048 takes one workgroup 20 us; with many such buckets the workgroups are all busy anyway).
// A few crowded buckets are ranked by counting, by all workgroups together, one after the other, as long
// as that takes a thread no more than kCountedMost comparisons per bucket; the others are dealt to teams.
// (An epoch of 10 generations, pool of 65536 with crowded buckets of up to 40000: 1744 us when all are
// counted, 1531 with a limit of 2048, 1424 with 512; a pool of 4096 with buckets of up to 1500: 280 us with any
// of these limits, 345 when all are dealt to teams.)
constexpr uint64_t kCountedMost = 512;
struct Crowd {
  uint32_t many;       // most offspring of a bucket that is not crowded
  uint64_t counted;    // most comparisons of a bucket ranked by counting
  uint32_t spilled;    // records in the spill list
  // places where the records of a bucket of n are: its own storage, and all of the spill list if that is full
  __device__ __forceinline__ uint32_t places(const BucketArgs &bk, uint32_t n) const { return n > bk.seg ? bk.seg + spilled : n; }
  __device__ __forceinline__ bool by_counting(const BucketArgs &bk, uint32_t n) const {
    const uint64_t p = places(bk, n);
    return n > many && p * p <= counted;
  }
  __device__ __forceinline__ bool by_team(const BucketArgs &bk, uint32_t n) const { return n > many && !by_counting(bk, n); }
};

// Deals the workgroups to the n_teams crowded buckets that are ranked by teams: one each, the others by
// the number of records; a team's workgroups are consecutive.  Every workgroup computes the same shares
// and notes its own in sh (team 0: left over).  Whole workgroup; ends with a barrier.
template <int kThreads>
__device__ __forceinline__ void join_team(BucketShared<kThreads> &sh, const BucketArgs &bk, const Crowd &crowd, uint32_t n_teams) {
  const uint32_t tid = threadIdx.x, nb = bk.nb;
  auto weight_of = [&](uint32_t c) {
    const uint32_t n = c < nb ? bk.count[c] : 0u;
    return crowd.by_team(bk, n) ? n : 0u;
  };
  if (tid == 0) sh.inside = sh.team = 0;
  __syncthreads();
  uint32_t w = 0;
  for (uint32_t c = tid; c < nb; c += kThreads) w += weight_of(c);
  if (w != 0) atomicAdd(&sh.inside, w);              // at most a pool, 2^20
  __syncthreads();
  const uint32_t all = sh.inside;
  uint32_t before = 0;                               // workgroups dealt to the buckets before c0
  for (uint32_t c0 = 0; c0 < nb; c0 += kThreads) {
    w = weight_of(c0 + tid);
    const uint32_t size = w != 0 ? 1u + (nb - n_teams) * w / all : 0u;            // 1024 * 2^20 fits 32 bits
    uint32_t incl = size;
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) {
      const uint32_t up = __shfl_up(incl, d, kLanes);
      if (tid % kLanes >= static_cast<uint32_t>(d)) incl += up;
    }
    if (tid % kLanes == kLanes - 1) sh.red[tid / kLanes] = incl;
    __syncthreads();
    uint32_t first = before + incl - size;
    for (uint32_t v = 0; v < kThreads / kLanes; ++v) {
      if (v < tid / kLanes) first += sh.red[v];
      before += sh.red[v];
    }
    if (blockIdx.x - first < size) { sh.helps = c0 + tid; sh.member = blockIdx.x - first; sh.team = size; }
    __syncthreads();
  }
}

// A crowded bucket o, ranked by counting by all workgroups of the launch together: each takes an equal
// share of the bucket's records (places of its storage, then of the spill list, whose records of other
// buckets count for nothing) and ranks it against all of them, a tile at a time; the
// bucket's own workgroup ranks its survivors too.
template <bool kElites, int kThreads>
__device__ __forceinline__ void rank_counted(BucketShared<kThreads> &sh, const double *fit_row, const BucketArgs &bk,
                                             const RowPlan &rp, uint32_t K, uint32_t o, bool any_copies, int32_t *sel) {
  const uint32_t tid = threadIdx.x, nb = bk.nb, b = blockIdx.x;
  const uint32_t before = wave_sum_u32(children_before(sh, bk, any_copies, o));
  __syncthreads();                                   // the shared arrays are free
  if ((tid & (kLanes - 1)) == 0) sh.red[tid / kLanes] = before;
  const uint32_t e0 = kElites ? bucket_bound(o, K, nb) : 0u, ne = kElites ? bucket_bound(o + 1, K, nb) - e0 : 0u;
  for (uint32_t e = tid; e < ne; e += kThreads)
    sh.ek[e] = static_cast<uint64_t>(__double_as_longlong(fit_row[rp.parents[e0 + e]]));
  __syncthreads();
  uint32_t off = e0;
#pragma unroll
  for (int w = 0; w < kThreads / kLanes; ++w) off += sh.red[w];
  if (off >= K) return;                              // nothing of this bucket survives
  Copies copies;
  if (any_copies) { copies.n = copies_in(sh, o); copies.key = sh.ek[0]; }
  const uint32_t n = bk.count[o], n_main = min(n, bk.seg);
  const uint32_t places = n_main + (n > n_main ? bk.count[kSpillCounter] : 0u);
  auto record = [&](uint32_t at, uint64_t &key, uint32_t &id) {      // a place of the bucket; id ~0: no record of it
    key = ~0ull;
    id = 0xFFFFFFFFu;
    if (at < n_main) {
      key = bk.keys[static_cast<size_t>(o) * bk.seg + at];
      id = bk.idx[static_cast<size_t>(o) * bk.seg + at];
    } else if (at < places && bk.spill_bucket[at - n_main] == o) {
      key = bk.spill_keys[at - n_main];
      id = bk.spill_idx[at - n_main];
    }
  };
  const uint32_t first = static_cast<uint32_t>(static_cast<uint64_t>(places) * b / nb);
  const uint32_t last = static_cast<uint32_t>(static_cast<uint64_t>(places) * (b + 1) / nb);
  const uint32_t total = (last - first) + (b == o ? ne : 0u);
  for (uint32_t base = 0; base < total; base += kThreads) {
    // thread (i, part): element base + i against every parts-th record of a tile
    const uint32_t m = min(total - base, static_cast<uint32_t>(kThreads)), width = pow2_at_least(m);
    const uint32_t parts = kThreads / width, i = tid % width, part = tid / width;
    const uint32_t mine = base + i;
    uint64_t key = ~0ull;
    uint32_t id = 0xFFFFFFFFu, e = 0;
    bool offspring = false, survivor = false;
    if (i < m) {
      if (mine < last - first) {
        record(first + mine, key, id);
        offspring = id != 0xFFFFFFFFu;
      } else {                                       // wins every tie, like slot 0
        e = mine - (last - first);
        key = sh.ek[e];
        id = 0;
        survivor = true;
      }
    }
    uint32_t n_below = 0;
    for (uint32_t tile = 0; tile < places; tile += kBucketLds) {
      __syncthreads();
      // (loads first, then the stores; the comparisons in steps of eight: one at a time, each waited for
      // its LDS read, and a bucket of 20000 took 300 us)
      constexpr int kPer = kBucketLds / kThreads;
      uint64_t loaded[kPer];
      uint32_t ids[kPer];
#pragma unroll
      for (int v = 0; v < kPer; ++v) record(tile + tid + v * kThreads, loaded[v], ids[v]);
#pragma unroll
      for (int v = 0; v < kPer; ++v) { sh.sk[tid + v * kThreads] = loaded[v]; sh.si[tid + v * kThreads] = ids[v]; }
      __syncthreads();
      const uint32_t count = min(places - tile, static_cast<uint32_t>(kBucketLds));   // what lies beyond is never below
      if (offspring || survivor)
        for (uint32_t q = part; q < count; q += 8 * parts) {
#pragma unroll
          for (uint32_t v = 0; v < 8; ++v) {
            const uint32_t at = min(q + v * parts, static_cast<uint32_t>(kBucketLds) - 1);
            n_below += q + v * parts < static_cast<uint32_t>(kBucketLds) && key_less(sh.sk[at], sh.si[at], key, id) ? 1u : 0u;
          }
        }
    }
    sh.below[tid] = 0;
    __syncthreads();
    if (n_below) atomicAdd(&sh.below[i], n_below);
    __syncthreads();
    uint32_t g = K, row = 0;
    if (part == 0 && (offspring || survivor)) {
      const uint32_t below = sh.below[i];
      g = off + below;
      if (survivor) {
        g += e + copies.before(key);
      } else {                                       // survivors with a score at or below its own come before it
        g += copies.n;
        uint32_t lo = 0, hi = ne;
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (sh.ek[mid] <= key) lo = mid + 1; else hi = mid;
        }
        g += lo;
      }
      if (g < K) {
        sel[g] = static_cast<int32_t>(survivor ? e0 + e : id);
        if (kElites) note_rank(g, key, K, nb, bk.split_next, bk.thresh_next);
        if (survivor) {
          rp.parent_next[g] = rp.parents[e0 + e];
        } else {
          row = rp.row_of[id];
          if (kElites) keep_child(rp, g, row, id, off + copies.n - e0 + below, K);
        }
      }
    }
    if (!kElites) keep_and_mark(rp, g < K, g, row);
  }
}

// A crowded bucket, ranked by a team of workgroups that do not wait for each other: every member sorts
// the same sample of the bucket's records, whose quantiles, (score, slot) pairs, cut the bucket into a
// range per member; then it reads all records, counts those below its range, collects those inside
// and ranks them and the survivors among them like a bucket of its own.
// Where children crowd, be it because a pool is full of copies of one genome or because nearly all
// children beat its best members, a bucket of about 800000 (pool of 2^20) took one workgroup alone 21 ms
// (sorting network in global memory) and all of them by counting 93 ms; a team takes 2.3.  Without such
// children the general selection of a pool of 2^20 leaves about a hundred buckets above 2048: 192 us when a
// workgroup each sorted them in global memory, 545 by counting, one after the other, 98 in teams.
constexpr uint32_t kPerMember = 256;    // records to a member, if the team is large enough
constexpr uint32_t kSamplePoints = 8;   // ... and sample points
template <bool kElites, int kThreads>
__device__ __forceinline__ void rank_in_team(BucketShared<kThreads> &sh, const double *fit_row, const BucketArgs &bk,
                                             const RowPlan &rp, uint32_t K, bool any_copies, int32_t *sel) {
  const uint32_t tid = threadIdx.x, nb = bk.nb, o = sh.helps, member = sh.member;
  const uint32_t n = bk.count[o], n_main = min(n, bk.seg);
  const uint32_t places = n_main + (n > n_main ? bk.count[kSpillCounter] : 0u);
  const uint32_t parts = min(sh.team, (n + kPerMember - 1) / kPerMember);
  if (member >= parts) return;
  auto record = [&](uint32_t at, uint64_t &key, uint32_t &id) {      // a place of the bucket; (~0, ~0): no record of it
    key = ~0ull;
    id = 0xFFFFFFFFu;
    if (at < n_main) {
      key = bk.keys[static_cast<size_t>(o) * bk.seg + at];
      id = bk.idx[static_cast<size_t>(o) * bk.seg + at];
    } else if (at < places) {
      const uint32_t owner = bk.spill_bucket[at - n_main];
      key = bk.spill_keys[at - n_main];
      id = bk.spill_idx[at - n_main];
      if (owner != o) { key = ~0ull; id = 0xFFFFFFFFu; }
    }
  };
  const uint32_t before = wave_sum_u32(children_before(sh, bk, any_copies, o));
  __syncthreads();                                   // the shared arrays are free
  if ((tid & (kLanes - 1)) == 0) sh.red[tid / kLanes] = before;
  const uint32_t e0 = kElites ? bucket_bound(o, K, nb) : 0u, ne = kElites ? bucket_bound(o + 1, K, nb) - e0 : 0u;
  for (uint32_t e = tid; e < ne; e += kThreads)
    sh.ek[e] = static_cast<uint64_t>(__double_as_longlong(fit_row[rp.parents[e0 + e]]));
  // the sample, taken at a fixed stride; places without a record of the bucket sort behind the others
  const uint32_t sample = min(pow2_at_least(kSamplePoints * parts), static_cast<uint32_t>(kBucketLds));
  if (tid == 0) sh.valid = 0;
  __syncthreads();
  uint32_t off = e0;
#pragma unroll
  for (int w = 0; w < kThreads / kLanes; ++w) off += sh.red[w];
  if (off >= K) return;                              // nothing of this bucket survives
  Copies copies;
  if (any_copies) { copies.n = copies_in(sh, o); copies.key = sh.ek[0]; }
  uint64_t lo_key = 0, end_key = ~0ull;              // this member's range [lo, end)
  uint32_t lo_slot = 0, end_slot = 0xFFFFFFFFu;
  if (parts > 1) {
    uint32_t valid = 0;
    for (uint32_t q = tid; q < sample; q += kThreads) {
      uint64_t key;
      uint32_t id;
      record(static_cast<uint32_t>(static_cast<uint64_t>(q) * places / sample), key, id);
      sh.sk[q] = key;
      sh.si[q] = id;
      valid += id != 0xFFFFFFFFu ? 1u : 0u;
    }
    if (valid) atomicAdd(&sh.valid, valid);
    __syncthreads();
    bitonic_sort(sh.sk, sh.si, sample);
    valid = sh.valid;
    if (valid == 0 && member != 0) return;           // no record in the sample: the first member takes the whole bucket
    if (valid != 0) {
      const uint32_t at = member * valid / parts, to = (member + 1) * valid / parts;
      if (member != 0) { lo_key = sh.sk[at]; lo_slot = sh.si[at]; }
      if (member + 1 != parts) { end_key = sh.sk[to]; end_slot = sh.si[to]; }
    }
  }
  auto survivors_below = [&](uint64_t key, uint32_t slot) {          // a survivor comes before an equal score
    uint32_t lo = 0, hi = ne;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (sh.ek[mid] < key || (sh.ek[mid] == key && slot != 0)) lo = mid + 1; else hi = mid;
    }
    return lo;
  };
  // the range is ranked in one piece, or, if more records lie in it than fit LDS, in several
  while (key_less(lo_key, lo_slot, end_key, end_slot)) {
    uint64_t hi_key = end_key;
    uint32_t hi_slot = end_slot, inside;
    for (;;) {
      __syncthreads();
      if (tid == 0) sh.smaller = sh.inside = 0;
      __syncthreads();
      uint32_t below = 0;
      constexpr int kPer = 8;                        // loads in flight per thread
      for (uint32_t base = 0; base < places; base += kPer * kThreads) {
        uint64_t key[kPer];
        uint32_t id[kPer];
#pragma unroll
        for (int v = 0; v < kPer; ++v) record(base + tid + v * kThreads, key[v], id[v]);
#pragma unroll
        for (int v = 0; v < kPer; ++v) {
          if (key_less(key[v], id[v], lo_key, lo_slot)) {
            ++below;
          } else if (key_less(key[v], id[v], hi_key, hi_slot)) {
            const uint32_t at = atomicAdd(&sh.inside, 1u);
            if (at < static_cast<uint32_t>(kBucketLds)) { sh.sk[at] = key[v]; sh.si[at] = id[v]; }
          }
        }
      }
      if (below) atomicAdd(&sh.smaller, below);
      __syncthreads();
      inside = sh.inside;
      if (inside <= static_cast<uint32_t>(kBucketLds)) break;
      // the kBucketLds records that were collected say where about half as many end; at least the last of
      // them falls out, so this comes to an end
      bitonic_sort(sh.sk, sh.si, kBucketLds);
      const uint32_t at = max(1u, static_cast<uint32_t>(static_cast<uint64_t>(kBucketLds) * (kBucketLds / 2) / inside));
      hi_key = sh.sk[at];
      hi_slot = sh.si[at];
    }
    const uint32_t below = sh.smaller, e_lo = survivors_below(lo_key, lo_slot), e_hi = survivors_below(hi_key, hi_slot);
    const bool sorted = inside > static_cast<uint32_t>(kBucketCount);
    const uint32_t npad = sorted ? pow2_at_least(inside) : (inside + 7) & ~7u;
    for (uint32_t q = inside + tid; q < npad; q += kThreads) { sh.sk[q] = ~0ull; sh.si[q] = 0xFFFFFFFFu; }
    __syncthreads();
    if (off + below + e_lo < K) {
      if (sorted) bitonic_sort(sh.sk, sh.si, npad);
      rank_bucket<kElites, kThreads>(sh.sk, sh.si, sh.ek + e_lo, inside, npad, e_hi - e_lo, e0 + e_lo, off + below + e_lo, sorted,
                                     K, bk, rp, copies, sel);
    }
    lo_key = hi_key;
    lo_slot = hi_slot;
  }
}

// The copies: the workgroups are dealt to the classes that have any, in turn, and a class's words to its workgroups.  A
// child's place is the number of marks before its own.
template <int kThreads>
__device__ __forceinline__ void rank_copies(BucketShared<kThreads> &sh, const double *fit_row, const BucketArgs &bk, const RowPlan &rp,
                                            uint32_t K, uint64_t lower, uint64_t upper, int32_t *sel) {
  const uint32_t tid = threadIdx.x, lane = tid % kLanes, wave = tid / kLanes, nb = bk.nb, b = blockIdx.x;
  const uint32_t n_lower = static_cast<uint32_t>(__popcll(lower)), n_classes = n_lower + static_cast<uint32_t>(__popcll(upper));
  const uint32_t member = b / n_classes, turn = b % n_classes, team = (nb - turn + n_classes - 1) / n_classes;
  uint64_t half = turn < n_lower ? lower : upper;
  for (uint32_t k = turn < n_lower ? 0u : n_lower; k < turn; ++k) half &= half - 1;
  const uint32_t c = (turn < n_lower ? 0u : kLanes) + __ffsll(static_cast<long long>(half)) - 1, o = sh.tie_bucket[c], words = tie_words(K);
  const uint32_t *marks = bk.ties + static_cast<size_t>(c) * words;
  const uint32_t first = words * member / team, last = words * (member + 1) / team;     // 24576 * 1024 fits 32 bits
  const uint32_t e0 = bucket_bound(o, K, nb), ne = bucket_bound(o + 1, K, nb) - e0;
  const uint64_t key = static_cast<uint64_t>(__double_as_longlong(fit_row[rp.parents[e0]]));
  // children before the bucket; survivors of the bucket with the same score; marks before this workgroup's words
  uint32_t before = children_before(sh, bk, true, o), equal = 0, marked = 0;
  for (uint32_t e = tid; e < ne; e += kThreads) equal += static_cast<uint64_t>(__double_as_longlong(fit_row[rp.parents[e0 + e]])) == key ? 1u : 0u;
  for (uint32_t w = tid; w < first; w += kThreads) marked += __popc(marks[w]);
  before = wave_sum_u32(before);
  equal = wave_sum_u32(equal);
  marked = wave_sum_u32(marked);
  constexpr uint32_t kWaves = kThreads / kLanes;
  static_assert(3 * kWaves <= kThreads, "room for the sums");
  __syncthreads();                                   // the shared arrays are free
  if (lane == 0) { sh.below[wave] = before; sh.below[kWaves + wave] = equal; sh.below[2 * kWaves + wave] = marked; }
  __syncthreads();
  before = equal = marked = 0;
#pragma unroll
  for (uint32_t w = 0; w < kWaves; ++w) { before += sh.below[w]; equal += sh.below[kWaves + w]; marked += sh.below[2 * kWaves + w]; }
  const uint32_t base = e0 + before + equal;         // rank of the first copy
  for (uint32_t at = first; at < last && base + marked < K; at += kThreads) {
    const uint32_t n = min(last - at, static_cast<uint32_t>(kThreads)), word = tid < n ? marks[at + tid] : 0u;
    uint32_t incl = __popc(word);
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) {
      const uint32_t up = __shfl_up(incl, d, kLanes);
      if (lane >= static_cast<uint32_t>(d)) incl += up;
    }
    __syncthreads();
    if (lane == kLanes - 1) sh.red[wave] = incl;
    sh.si[tid] = word;
    __syncthreads();
    uint32_t upto = marked + incl - __popc(word);
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      if (w < wave) upto += sh.red[w];
      marked += sh.red[w];
    }
    sh.below[tid] = upto;
    __syncthreads();
    for (uint32_t q = tid; q < n * 32; q += kThreads) {
      const uint32_t bits = sh.si[q / 32], i = sh.below[q / 32] + __popc(bits & ((1u << (q % 32)) - 1u)), g = base + i;
      if (((bits >> (q % 32)) & 1u) == 0 || g >= K) continue;
      const uint32_t p = K + at * 32 + q, row = rp.row_of[p];
      sel[g] = static_cast<int32_t>(p);
      note_rank(g, key, K, nb, bk.split_next, bk.thresh_next);
      keep_child(rp, g, row, p, before + i, K);
    }
  }
}

// kElites: the quantile buckets above, each with its share of the survivors.  Without: the last
// step of the sample sort of the general path below, a bucket holds candidates only (fit_row,
// rp.parents, count_next unused) and its first rank is the number of candidates before it.
// kThreads: a bucket of at most that many offspring (nearly all) is ranked straight from registers.
template <bool kElites, int kThreads>
__global__ __launch_bounds__(kThreads) void bucket_select_kernel(const double *fit_row, BucketArgs bk, RowPlan rp,
                                                                 uint32_t K, uint32_t *count_next, uint32_t *ties_next, int32_t *sel) {
  __shared__ BucketShared<kThreads> sh;
  const uint32_t b = blockIdx.x, nb = bk.nb, tid = threadIdx.x;
  // offset of this bucket = its first survivor rank + all offspring of the buckets before it
  uint32_t before = 0;
  for (uint32_t c = tid; c < b; c += kThreads) before += bk.count[c];
  before = wave_sum_u32(before);
  if ((tid & (kLanes - 1)) == 0) sh.red[tid / kLanes] = before;
  const bool any_many = bk.count[kManyFlag] != 0;    // a bucket holds more than kBucketCount
  const bool any_copies = kElites && bk.count[kTieFlag] != 0;
  const uint32_t e0 = kElites ? bucket_bound(b, K, nb) : 0u, ne = kElites ? bucket_bound(b + 1, K, nb) - e0 : 0u;
  const uint32_t n = bk.count[b];
  // Every global load a small bucket needs is issued here, before anything waits for one: an
  // offspring per thread counted from thread 0 (read before the bucket's count is known: the
  // places beyond it hold whatever an earlier generation left, which is only used as an index
  // when it is one), a survivor per thread counted from the last one, and the rows of both.
  const uint32_t seg = bk.seg;
  uint64_t my_key = ~0ull, elite_key = 0;
  uint32_t my_idx = 0xFFFFFFFFu, my_row = 0, elite_row = 0;
  if (tid < seg) {
    my_key = bk.keys[static_cast<size_t>(b) * seg + tid];
    my_idx = bk.idx[static_cast<size_t>(b) * seg + tid];
  }
  const uint32_t se = kThreads - 1 - tid;
  if (se < ne) elite_row = rp.parents[e0 + se];
  if (se < ne) elite_key = static_cast<uint64_t>(__double_as_longlong(fit_row[elite_row]));   // survivors stayed in their rows
  if (my_idx < 4 * K) my_row = rp.row_of[my_idx];
  if (any_copies && tid < static_cast<uint32_t>(kTieClasses)) {
    const uint32_t n_copies = bk.count[kTieCount + tid], in = bk.count[kTieBucket + tid];
    sh.tie_count[tid] = n_copies;
    sh.tie_bucket[tid] = in;
    const uint32_t more = wave_sum_u32(in < b ? n_copies : 0u);
    if (tid % kLanes == 0) sh.red[tid / kLanes] += more;
  }
  static_assert(kThreads <= kBucketCount, "a small bucket is ranked by counting");
  const bool small = n <= static_cast<uint32_t>(kThreads) && n <= seg && ne <= static_cast<uint32_t>(kThreads);
  // counting loops run in steps of 8 over padding; the sorting network needs a power of two
  const bool sorted = n > static_cast<uint32_t>(kBucketCount);
  const bool in_lds = n <= static_cast<uint32_t>(kBucketLds);
  const uint32_t npad = !in_lds ? 0u : sorted ? pow2_at_least(n) : (n < 8 ? 8u : (n + 7) & ~7u);
  if (small) {
    if (tid < npad) {                                // never sorted: npad <= the threads
      sh.sk[tid] = tid < n ? my_key : ~0ull;
      sh.si[tid] = tid < n ? my_idx : 0xFFFFFFFFu;
    }
    if (se < ne) sh.ek[se] = elite_key;
  } else {
    for (uint32_t e = tid; e < ne; e += kThreads)
      sh.ek[e] = static_cast<uint64_t>(__double_as_longlong(fit_row[rp.parents[e0 + e]]));
  }
  if (tid == 0) sh.spill_cursor = sh.n_many = sh.n_teams = sh.n_counted = 0;
  __syncthreads();
  uint32_t off = e0;
#pragma unroll
  for (int w = 0; w < kThreads / kLanes; ++w) off += sh.red[w];
  Copies copies;
  if (any_copies) { copies.n = copies_in(sh, b); copies.key = sh.ek[0]; }
  Crowd crowd{};
  uint32_t n_teams = 0;
  bool crowded = false;                              // this workgroup's own bucket
  if (any_many) {
    constexpr int kPer = kMaxBuckets / kThreads;     // buckets this thread looks at
    uint32_t counts[kPer], many = 0, teams = 0;
#pragma unroll
    for (int v = 0; v < kPer; ++v) counts[v] = bk.count[min(tid + v * kThreads, static_cast<uint32_t>(kMaxBuckets) - 1)];
#pragma unroll
    for (int v = 0; v < kPer; ++v) {
      if (tid + v * kThreads >= nb) counts[v] = 0;
      many += counts[v] > static_cast<uint32_t>(kBucketCount) ? 1u : 0u;
    }
    if (many) atomicAdd(&sh.n_many, many);
    crowd.spilled = bk.count[kSpillCounter];
    __syncthreads();
    const bool few = sh.n_many <= kFewCrowded;
    crowd.many = few ? kBucketCount : kBucketLds;
    crowd.counted = few ? kCountedMost * kThreads * nb : 0;
#pragma unroll
    for (int v = 0; v < kPer; ++v) {
      if (crowd.by_counting(bk, counts[v])) sh.counted[atomicAdd(&sh.n_counted, 1u)] = tid + v * kThreads;
      teams += crowd.by_team(bk, counts[v]) ? 1u : 0u;
    }
    if (teams) atomicAdd(&sh.n_teams, teams);
    __syncthreads();
    n_teams = sh.n_teams;
    if (n_teams != 0) join_team(sh, bk, crowd, n_teams);
    crowded = n > crowd.many;
  }
  if (!crowded && off < K && n + ne != 0) {          // otherwise nothing of this bucket survives
    if (small) {
      // offspring tid: rank = offspring below it + survivors with score <= its score (a survivor
      // wins a tie: smaller slot)
      {
        uint32_t g = K;
        if (tid < n) {
          uint32_t below = 0, equal = 0;             // padding keys are never below a real one
          for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
            for (int v = 0; v < 8; ++v) {
              const uint64_t other = sh.sk[q + v];
              below += other < my_key ? 1u : 0u;
              equal += other == my_key ? 1u : 0u;
            }
          }
          if (equal > 1)                             // shares its score: the slots decide
            for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
              for (int v = 0; v < 8; ++v) below += (sh.sk[q + v] == my_key && sh.si[q + v] < my_idx) ? 1u : 0u;
            }
          uint32_t lo = 0, hi = ne;
          while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (sh.ek[mid] <= my_key) lo = mid + 1; else hi = mid;
          }
          g = off + copies.n + below + lo;
          if (g < K) {
            sel[g] = static_cast<int32_t>(my_idx);
            if (kElites) {
              note_rank(g, my_key, K, nb, bk.split_next, bk.thresh_next);
              keep_child(rp, g, my_row, my_idx, off + copies.n - e0 + below, K);
            }
          }
        }
        if (!kElites) keep_and_mark(rp, g < K, g, my_row);
      }
      // survivor se: rank = se + offspring with a strictly smaller score
      if (kElites) {
        if (se < ne) {
          uint32_t lo = 0;
          for (uint32_t q = 0; q < npad; q += 8) {
#pragma unroll
            for (int v = 0; v < 8; ++v) lo += sh.sk[q + v] < elite_key ? 1u : 0u;
          }
          const uint32_t g = off + se + lo + copies.before(elite_key);
          if (g < K) {
            sel[g] = static_cast<int32_t>(e0 + se);
            note_rank(g, elite_key, K, nb, bk.split_next, bk.thresh_next);
            rp.parent_next[g] = elite_row;
          }
        }
      }
    } else {
      gather_bucket(sh.sk, sh.si, bk, b, n, npad, &sh.spill_cursor);
      if (sorted) bitonic_sort(sh.sk, sh.si, npad);
      rank_bucket<kElites, kThreads>(sh.sk, sh.si, sh.ek, n, npad, ne, e0, off, sorted, K, bk, rp, copies, sel);
    }
  }
  if (any_many)
    for (uint32_t k = 0; k < sh.n_counted; ++k) rank_counted<kElites, kThreads>(sh, fit_row, bk, rp, K, sh.counted[k], any_copies, sel);
  if (n_teams != 0 && sh.team != 0) rank_in_team<kElites, kThreads>(sh, fit_row, bk, rp, K, any_copies, sel);
  if (kElites) {
    uint64_t classes[2] = {0, 0};
    if (any_copies) {
      classes[0] = __ballot(sh.tie_count[tid % kLanes] != 0);
      classes[1] = __ballot(sh.tie_count[kLanes + tid % kLanes] != 0);
      rank_copies(sh, fit_row, bk, rp, K, classes[0], classes[1], sel);
    }
    // the other counter set and bitmaps, for the next generation
    if (tid == 0) count_next[b] = 0;
    for (uint32_t c = kMaxBuckets + tid; b == 0 && c < static_cast<uint32_t>(kBucketCounters); c += kThreads) count_next[c] = 0;
    // (only the classes that it was used for: clearing all of them took 0.8 of the kernel's 6 us on the stress workload)
    const uint32_t words = tie_words(K), from = words * b / nb, to = words * (b + 1) / nb;        // 24576 * 1024 fits 32 bits
    const uint32_t *mask = ties_next + kTieClasses * words;
#pragma unroll
    for (uint32_t k = 0; k < kTieMask; ++k)
      for (uint32_t used = mask[k]; used != 0; used &= used - 1) {
        uint32_t *marks = ties_next + (32 * k + __ffs(static_cast<int>(used)) - 1) * words;
        for (uint32_t w = from + tid; w < to; w += kThreads) marks[w] = 0;
      }
    if (b == 0 && tid < kTieMask) bk.ties[kTieClasses * words + tid] = static_cast<uint32_t>(classes[tid / 2] >> (32 * (tid % 2)));
  }
}

// ------------------------------------------------- general path, larger pools -----
// Sample sort over the same bucket storage: a ranked sample of the pool's scores gives the
// splitters, every candidate is dropped into its bucket, and one workgroup per bucket ranks its
// share (bucket_select_kernel<false, .>); buckets concatenate to the global (score, slot) order and
// only those that reach below rank K do any work.  The sample only decides how even the buckets
// are, never the result.

// Splitters: `sample` = per * nb candidates taken at a fixed stride from the pool; those of rank
// per * (c + 1) - 1 among them, in (score, slot) order like everything else, become splitter c (per =
// kOversample sample points per bucket, two where that would take more than kSampleMax; a bucket of
// 64 to 127 candidates on average then hardly ever grows beyond the 512 that are ranked straight from
// registers).  A splitter is a (score, slot) pair, not a score: a pool that has been searched for a
// while is full of copies of one genome, and splitters that only knew the scores put all of them into
// one bucket, which one workgroup then ranked alone (16384 candidates of 512 jobs: 544 us for the
// bucket kernel where a pool of distinct scores takes 9).  Ranks by counting: every workgroup loads the
// whole sample into LDS and each of its waves ranks one element, the lanes striding over the sample.
constexpr int kSampleThreads = 1024;
constexpr int kOversample = 4;
constexpr int kSampleMax = 2048;
constexpr int kSamplePer = kSampleThreads / kLanes;    // elements ranked by one workgroup
__global__ __launch_bounds__(kSampleThreads) void sample_splitters_kernel(const double *fit_row, const double *slot_score,
                                                                         const uint32_t *row_of, uint32_t P,
                                                                         uint32_t sample, uint32_t nb,
                                                                         uint64_t *split, uint32_t *split_slot,
                                                                         uint32_t *count) {
  __shared__ uint64_t sk[kSampleMax];
  const uint32_t per = sample / nb;                   // sample points per bucket: kOversample, or fewer with kMaxBuckets buckets
  const uint32_t t = threadIdx.x;
  const uint32_t sample_log2 = 31 - __clz(static_cast<int>(sample));
  // sample point e: slot floor(e P / sample); sample is a power of two
  auto slot_of = [&](uint32_t e) { return static_cast<uint32_t>((static_cast<uint64_t>(e) * P) >> sample_log2); };
  if (blockIdx.x == 0)
    for (uint32_t c = t; c < static_cast<uint32_t>(kBucketCounters); c += kSampleThreads) count[c] = 0;
  uint64_t mine_of[kSampleMax / kSampleThreads];
#pragma unroll
  for (int u = 0; u < kSampleMax / kSampleThreads; ++u) {          // all loads first, then the stores
    const uint32_t e = t + u * kSampleThreads, p = slot_of(e);
    mine_of[u] = e < sample ? static_cast<uint64_t>(__double_as_longlong(slot_score ? slot_score[p] : fit_row[row_of[p]])) : ~0ull;
  }
#pragma unroll
  for (int u = 0; u < kSampleMax / kSampleThreads; ++u) sk[t + u * kSampleThreads] = mine_of[u];
  __syncthreads();
  const uint32_t lane = t % kLanes;
  const uint32_t mine = blockIdx.x * kSamplePer + t / kLanes;      // sample = kSamplePer * the workgroups
  const uint64_t key = sk[mine];
  uint32_t below = 0;
  for (uint32_t q = lane; q < sample; q += 2 * kLanes) {           // sample is a multiple of 128
    const uint64_t a = sk[q], b = sk[q + kLanes];
    // sample points in ascending order are slots in ascending order
    below += (a < key || (a == key && q < mine) ? 1u : 0u) + (b < key || (b == key && q + kLanes < mine) ? 1u : 0u);
  }
  const uint32_t r = wave_sum_u32(below);
  // rank per * (c + 1) - 1 makes splitter c; the last bucket has none
  if (lane == 0 && r % per == per - 1 && r / per + 1 < nb) {
    split[r / per] = key;
    split_slot[r / per] = slot_of(mine);
  }
}

// Bucket of a candidate = number of splitters at or below it.  A workgroup first counts its
// candidates per bucket in LDS and reserves their places with one global atomic per bucket,
// instead of one per candidate.
constexpr int kDropThreads = 1024;
__global__ __launch_bounds__(kDropThreads) void drop_all_kernel(const double *fit_row, const double *slot_score,
                                                               const uint32_t *row_of, uint32_t P, BucketArgs bk,
                                                               const uint32_t *split_slot) {
  __shared__ uint64_t split[kMaxBuckets];
  __shared__ uint32_t slot_at[kMaxBuckets];
  __shared__ uint32_t here[kMaxBuckets], base[kMaxBuckets];
  const uint32_t t = threadIdx.x, nb = bk.nb;
  for (uint32_t c = t; c < nb; c += kDropThreads) {
    split[c] = c + 1 < nb ? bk.split[c] : ~0ull;
    slot_at[c] = c + 1 < nb ? split_slot[c] : ~0u;
    here[c] = 0;
  }
  const uint32_t p = blockIdx.x * kDropThreads + t;
  uint64_t key = 0;
  if (p < P) key = static_cast<uint64_t>(__double_as_longlong(slot_score ? slot_score[p] : fit_row[row_of[p]]));
  __syncthreads();
  uint32_t b = 0, r = 0;
  if (p < P) {
    uint32_t lo = 0, hi = nb - 1;                    // splitters 0 .. nb-2
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (!key_less(key, p, split[mid], slot_at[mid])) lo = mid + 1; else hi = mid;
    }
    b = lo;
    r = atomicAdd(&here[b], 1u);
  }
  __syncthreads();
  for (uint32_t c = t; c < nb; c += kDropThreads) {
    base[c] = here[c] ? atomicAdd(&bk.count[c], here[c]) : 0u;
    if (base[c] + here[c] > static_cast<uint32_t>(kBucketCount)) bk.count[kManyFlag] = 1;
  }
  __syncthreads();
  if (p < P) {
    const uint32_t slot = base[b] + r;
    if (slot < bk.seg) {
      const size_t at = static_cast<size_t>(b) * bk.seg + slot;
      bk.keys[at] = key;
      bk.idx[at] = p;
    } else {                                         // bucket full: shared spill list (holds a whole pool)
      const uint32_t at = atomicAdd(&bk.count[kSpillCounter], 1u);
      bk.spill_keys[at] = key;
      bk.spill_idx[at] = p;
      bk.spill_bucket[at] = b;
    }
  }
}

__global__ void zero_words_kernel(uint32_t *words, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) words[i] = 0;
}

// Splitters after a selection by the general path.
__global__ void splitters_kernel(const double *fit_row, const uint32_t *row_of, const int32_t *sel, uint32_t K,
                                 uint32_t nb, uint64_t *split, uint64_t *thresh, uint32_t *count0,
                                 uint32_t *count1, uint32_t *ties, uint32_t ties_words) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  for (uint32_t w = c; w < ties_words; w += gridDim.x * blockDim.x) ties[w] = 0;
  if (c < static_cast<uint32_t>(kBucketCounters)) { count0[c] = 0; count1[c] = 0; }
  if (c < static_cast<uint32_t>(kMaxBuckets))
    split[c] = (c + 1 < nb) ? static_cast<uint64_t>(__double_as_longlong(fit_row[row_of[sel[bucket_bound(c + 1, K, nb)]]])) : kNoSplitter;
  if (c == 0) *thresh = static_cast<uint64_t>(__double_as_longlong(fit_row[row_of[sel[K - 1]]]));
}

// The whole workgroup calls it when what it writes for the host, or reads of the host's, is written or read.
__device__ __forceinline__ void signal_host(const HostSignal &done) {
  all_arrived();
  if (threadIdx.x != 0) return;
  __threadfence_system();
  if (last_to_arrive(done.arrived)) __hip_atomic_store(done.flag, done.value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What the kernels need of one job slot, derived from the validated raw table.
struct SlotValues { uint32_t start, most, draws, lift, info; double abl, cc, d, Y; };

__device__ __forceinline__ SlotValues derive_slot(const RawJobs &raw, uint32_t j) {
  const uint32_t w = raw.rawinfo[j];
  const double a = raw.a[j], c = raw.c[j], d = raw.d[j], Y = raw.Y[j];         // (also of an empty slot: nothing waits for w)
  const int lo = w & 31, hi = (w >> 5) & 31, mu = (w >> 10) & 31;
  if (!((w >> 15) & 1u)) return SlotValues{0u, 0u, 0u, 0u, 0u, 0.0, 0.0, 0.0, 0.0};
  const int bl = min(mu, hi);                       // log2 of the local batch of a running job
  const int gstart = max(lo, bl);                   // batch a waiting job resumes with
  SlotValues v;
  v.start = static_cast<uint32_t>(max(0, gstart - mu) + 1);
  v.most = static_cast<uint32_t>(max(0, hi - mu) + 1);
  v.draws = static_cast<uint32_t>(hi - lo + 2);
  v.lift = v.start + static_cast<uint32_t>(mu - lo);     // the batch 2^(lo + k - 1) takes the code lo + k - mu, or, lifted, start (1 .. 31)
  v.info = static_cast<uint32_t>(lo) | (static_cast<uint32_t>(hi - lo + 2) << 5) | (static_cast<uint32_t>(mu) << 11) |
           (static_cast<uint32_t>(bl) << 16) | (1u << 21) | (((w >> 16) & 1u) << 22);
  v.abl = a * static_cast<double>(1u << bl);
  v.cc = c;
  v.d = d;
  v.Y = Y;
  return v;
}

// A new job table in one launch, a thread per slot and a wave per row.  The raw table lies in pinned host memory, so every value
// is read once, and all of a thread's are on their way together.  The thread writes the slot's values and its entries of the
// term table, marks the slot in tab.stored if it changed hands (the genomes,
// stored under another table, hold a gene of its former job: whoever reads one from then on takes
// it as "waiting"; resetting the genes themselves was a scattered store per row and slot, 80 to 240 us
// on the stress cluster) and clears the bytes of the rows beyond the job slots.
__global__ __launch_bounds__(kLanes) void table_change_kernel(RawJobs raw, JobTable tab, double *remaining, uint32_t Jp, HostSignal done) {
  const uint32_t lane = threadIdx.x, row = blockIdx.x, E = tab.term_E, j = row * kLanes + lane;
  const uint32_t flags = raw.rawinfo[j];
  const double raw_Y = raw.Y[j];
  const SlotValues v = derive_slot(raw, j);
  for (uint32_t e = 0; e < E; ++e) tab.terms[(row * E + e) * kLanes + lane] = term_of(v.abl, v.cc, v.d, v.Y, info_blexp(v.info), e);
  remaining[j] = raw_Y;
  uint8_t *arrays[4] = {reinterpret_cast<uint8_t *>(tab.start), reinterpret_cast<uint8_t *>(tab.most),
                        reinterpret_cast<uint8_t *>(tab.draws), reinterpret_cast<uint8_t *>(tab.lift)};
  const uint32_t values[4] = {v.start, v.most, v.draws, v.lift};
  const uint32_t at = gene_byte(j);
#pragma unroll
  for (int k = 0; k < 4; ++k) arrays[k][at] = static_cast<uint8_t>(values[k]);
  if (row == Jp / kLanes - 1)
    for (uint32_t beyond = at % 4 + 1; beyond < 4; ++beyond)
#pragma unroll
      for (int k = 0; k < 4; ++k) arrays[k][at - at % 4 + beyond] = 0;
  tab.info[j] = v.info;
  tab.abl[j] = v.abl; tab.cc[j] = v.cc; tab.d[j] = v.d; tab.Y[j] = v.Y;
  if (tab.stored != tab.info && ((flags >> 17) & 1u)) tab.stored[j] |= kInfoReset;
  signal_host(done);
}

constexpr int kFetchThreads = 256;
__global__ __launch_bounds__(kFetchThreads) void fetch_kernel(const uint4 *from, uint4 *to, uint32_t n, HostSignal done) {
  const uint32_t i = blockIdx.x * kFetchThreads + threadIdx.x;
  if (i < n) to[i] = from[i];
  signal_host(done);
}

// Term table: the score formula evaluated once per (slot, GPU-count code), same operations in
// the same order as the per-gene evaluation, so both give the same bits.
__global__ void build_terms_kernel(JobTable tab, uint32_t Jp) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t E = tab.term_E;
  if (q >= Jp * E) return;
  const uint32_t lane = q % kLanes, e = (q / kLanes) % E, row = q / (kLanes * E);
  const uint32_t j = row * kLanes + lane;
  tab.terms[q] = term_of(tab.abl[j], tab.cc[j], tab.d[j], tab.Y[j], info_blexp(tab.info[j]), e);
}

// Batch size of job slot j in a genome row.
__device__ __forceinline__ uint32_t stored_batch(const uint32_t *row, const uint32_t *stored, uint32_t j) {
  const uint32_t w = stored[j];
  return info_reset(w) ? 0u : batch_of_code(reinterpret_cast<const uint8_t *>(row)[gene_byte(j)], info_blexp(w));
}

__global__ void best_kernel(const uint32_t *genes, const double *fit_row, const uint32_t *best_row, const uint32_t *stored,
                            const uint32_t *info, uint32_t Jn, uint32_t row_words, int32_t *batch_out, int32_t *gpus_out, double *fit_out, const uint32_t *err_in,
                            uint32_t *err_out, HostSignal done) {
  const uint32_t best = *best_row;
  const uint32_t *row = genes + static_cast<size_t>(best) * row_words;
  for (uint32_t j = threadIdx.x; j < Jn; j += blockDim.x) {
    const uint32_t B = stored_batch(row, stored, j);
    batch_out[j] = static_cast<int32_t>(B);
    gpus_out[j] = static_cast<int32_t>(B ? max(1u, B >> info_mu(info[j])) : 0u);
  }
  if (threadIdx.x == 0) {
    *fit_out = fit_row[best];
    err_out[0] = err_in[0];                          // the two error words travel to the host with the winner
    err_out[1] = err_in[1];
  }
  signal_host(done);
}

// The state in slot order.  Two launches each, the second for the survivors (a survivor's slot may have been
// handed another row already, so what the first one wrote for it does not count).
constexpr int kExportThreads = 256;
__device__ __forceinline__ uint32_t exported_row(const ExportArgs &x, uint32_t row) { return min(row, x.P + x.K - 1); }
__device__ __forceinline__ void unpack_row(const ExportArgs &x, uint32_t row, uint32_t at) {
  const uint32_t *genome = x.genes + static_cast<size_t>(row) * (words_of(x.Jp / kLanes) * kLanes);
  int32_t *out = x.genes_out + static_cast<size_t>(at) * x.Jp;
  for (uint32_t j = threadIdx.x; j < x.Jp; j += kExportThreads) out[j] = static_cast<int32_t>(stored_batch(genome, x.stored, j));
}
__device__ __forceinline__ void export_survivor(const ExportArgs &x, uint32_t g, uint32_t row) {
  const uint32_t slot = static_cast<uint32_t>(x.sel[g]);
  x.sel_out[g] = static_cast<int32_t>(slot);
  if (slot < x.P) x.fit_out[slot] = x.fit_row[row];
  if (g == 0) { x.err_out[0] = x.err_in[0]; x.err_out[1] = x.err_in[1]; }
}
// One workgroup per slot, then per survivor.
__global__ __launch_bounds__(kExportThreads) void export_slots_kernel(ExportArgs x, uint32_t first, bool with_scores) {
  const uint32_t row = exported_row(x, x.row_of[first + blockIdx.x]);
  unpack_row(x, row, blockIdx.x);
  if (with_scores && threadIdx.x == 0) x.fit_out[blockIdx.x] = x.fit_row[row];
}
__global__ __launch_bounds__(kExportThreads) void export_survivors_kernel(ExportArgs x, uint32_t first, uint32_t count,
                                                                         bool with_scores) {
  const uint32_t g = blockIdx.x, at = static_cast<uint32_t>(x.sel[g]) - first, row = exported_row(x, x.parents[g]);
  if (at < count) unpack_row(x, row, at);
  if (with_scores && threadIdx.x == 0) export_survivor(x, g, row);
  if (x.done.flag != nullptr) signal_host(x.done);
}
// One thread per slot, then per survivor.
__global__ __launch_bounds__(kExportThreads) void export_slot_scores_kernel(ExportArgs x) {
  const uint32_t p = blockIdx.x * kExportThreads + threadIdx.x;
  if (p < x.P) x.fit_out[p] = x.fit_row[exported_row(x, x.row_of[p])];
}
__global__ __launch_bounds__(kExportThreads) void export_survivor_scores_kernel(ExportArgs x) {
  const uint32_t g = blockIdx.x * kExportThreads + threadIdx.x;
  if (g < x.K) export_survivor(x, g, exported_row(x, x.parents[g]));
}

// The winner unrolled over the GPUs (Eq. 1, reorder): every workgroup scans the jobs' GPU
// counts in LDS (at most 2048 slots), then each thread finds the job of one GPU by binary
// search over the prefix sums.
constexpr int kPlaceThreads = 1024;
__global__ __launch_bounds__(kPlaceThreads) void placement_kernel(const uint32_t *genes, const uint32_t *best_row,
                                                                 const uint32_t *info, uint32_t Jn,
                                                                 uint32_t row_words, uint32_t G, int32_t *slot_of_gpu,
                                                                 int32_t *batch_of_gpu, const uint32_t *err_in,
                                                                 uint32_t *err_out, HostSignal done) {
  __shared__ uint32_t first[2 * kPlaceThreads + 1];    // first GPU of every slot, then the GPUs in use
  __shared__ uint32_t per_gpu[2 * kPlaceThreads];      // local batch of every slot's workers
  __shared__ uint32_t wave_total[kPlaceThreads / kLanes];
  const uint32_t *row = genes + static_cast<size_t>(*best_row) * row_words;
  const uint32_t t = threadIdx.x;
  // thread t owns slots 2t and 2t + 1
  uint32_t c[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint32_t j = 2 * t + u;
    const uint32_t B = j < Jn ? stored_batch(row, info, j) : 0u;
    c[u] = B ? max(1u, B >> info_mu(info[j < Jn ? j : 0])) : 0u;
    per_gpu[j] = B ? B / c[u] : 0u;
  }
  const uint32_t mine = c[0] + c[1];
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < kLanes; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, kLanes);
    if ((t & (kLanes - 1)) >= static_cast<uint32_t>(d)) incl += up;
  }
  if ((t & (kLanes - 1)) == kLanes - 1) wave_total[t / kLanes] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < t / kLanes; ++w) before += wave_total[w];
  const uint32_t excl = before + incl - mine;
  first[2 * t] = excl;
  first[2 * t + 1] = excl + c[0];
  if (t == kPlaceThreads - 1) first[2 * kPlaceThreads] = excl + mine;
  __syncthreads();
  const uint32_t used = first[2 * kPlaceThreads];
  for (uint32_t i = blockIdx.x * kPlaceThreads + t; i < G; i += gridDim.x * kPlaceThreads) {
    int32_t slot = -1, batch = 0;
    if (i < used) {
      uint32_t lo = 0, hi = 2 * kPlaceThreads;       // last slot with first[slot] <= i
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (first[mid] <= i) lo = mid; else hi = mid;
      }
      slot = static_cast<int32_t>(lo);
      batch = static_cast<int32_t>(per_gpu[lo]);
    }
    slot_of_gpu[i] = slot;
    batch_of_gpu[i] = batch;
  }
  if (blockIdx.x == 0 && t < 2) err_out[t] = err_in[t];
  signal_host(done);
}

}  // namespace

hipError_t launch_build_terms(const JobTable &tab, uint32_t Jp, hipStream_t s) {
  const uint32_t n = Jp * tab.term_E;
  hipLaunchKernelGGL(build_terms_kernel, dim3((n + 255) / 256), dim3(256), 0, s, tab, Jp);
  return hipGetLastError();
}

hipError_t launch_table_change(const RawJobs &raw, const JobTable &tab, double *remaining, uint32_t Jp, const HostSignal &done, hipStream_t s) {
  hipLaunchKernelGGL(table_change_kernel, dim3(Jp / kLanes), dim3(kLanes), 0, s, raw, tab, remaining, Jp, done);
  return hipGetLastError();
}

hipError_t launch_fetch(const void *from, void *to, uint32_t n, const HostSignal &done, hipStream_t s) {
  hipLaunchKernelGGL(fetch_kernel, dim3((n + kFetchThreads - 1) / kFetchThreads), dim3(kFetchThreads), 0, s, static_cast<const uint4 *>(from), static_cast<uint4 *>(to),
                     n, done);
  return hipGetLastError();
}

hipError_t launch_export_scores(const ExportArgs &x, hipStream_t s) {
  hipLaunchKernelGGL(export_slot_scores_kernel, dim3((x.P + kExportThreads - 1) / kExportThreads), dim3(kExportThreads), 0, s, x);
  const hipError_t rc = hipGetLastError();
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(export_survivor_scores_kernel, dim3((x.K + kExportThreads - 1) / kExportThreads), dim3(kExportThreads), 0, s, x);
  return hipGetLastError();
}

hipError_t launch_export_genes(const ExportArgs &x, uint32_t first, uint32_t count, bool with_scores, hipStream_t s) {
  hipLaunchKernelGGL(export_slots_kernel, dim3(count), dim3(kExportThreads), 0, s, x, first, with_scores);
  const hipError_t rc = hipGetLastError();
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(export_survivors_kernel, dim3(x.K), dim3(kExportThreads), 0, s, x, first, count, with_scores);
  return hipGetLastError();
}

hipError_t launch_zero_words(uint32_t *words, uint32_t n, hipStream_t s) {
  hipLaunchKernelGGL(zero_words_kernel, dim3((n + 255) / 256), dim3(256), 0, s, words, n);
  return hipGetLastError();
}

hipError_t launch_select(const double *fit, const double *slot_score, const RowPlan &rp, uint32_t P, uint32_t K,
                         const BucketArgs &store, int32_t *sel, hipStream_t s) {
  if (P <= kRankPoolMax) {
    const uint32_t rank_blocks = (P + kRankPoolPer - 1) / kRankPoolPer;
    constexpr uint32_t kStep = 8 * (kSortThreads / kRankPoolPer);
    const size_t lds = static_cast<size_t>((P + kStep - 1) / kStep * kStep) * 8 + kRankPoolPer * 4;
    hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void *>(rank_pool_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL(rank_pool_kernel, dim3(rank_blocks), dim3(kSortThreads), lds, s, fit, slot_score, rp, P, K, sel);
    return hipGetLastError();
  }
  // 64 to 127 candidates per bucket (more in pools beyond 2^17), kOversample sample points per
  // bucket while the sample stays within kSampleMax
  BucketArgs bk = store;
  uint32_t nb = 32;
  while (nb < static_cast<uint32_t>(kMaxBuckets) && nb * 128 <= P) nb <<= 1;
  const uint32_t sample = std::min<uint32_t>(kOversample * nb, kSampleMax);   // a power of two, 256 .. kSampleMax
  bk.seg = static_cast<uint32_t>(static_cast<size_t>(store.nb) * store.seg / nb);   // the same storage, re-divided
  bk.nb = nb;
  hipLaunchKernelGGL(sample_splitters_kernel, dim3(sample / kSamplePer), dim3(kSampleThreads), 0, s, fit, slot_score,
                     rp.row_of, P, sample, nb, const_cast<uint64_t *>(bk.split), bk.split_slot, bk.count);
  hipError_t rc = hipGetLastError();
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL(drop_all_kernel, dim3((P + kDropThreads - 1) / kDropThreads), dim3(kDropThreads), 0, s, fit,
                     slot_score, rp.row_of, P, bk, bk.split_slot);
  rc = hipGetLastError();
  if (rc != hipSuccess) return rc;
  hipLaunchKernelGGL((bucket_select_kernel<false, kBucketCount>), dim3(nb), dim3(kBucketCount), 0, s, nullptr,
                     bk, rp, K, nullptr, nullptr, sel);
  return hipGetLastError();
}

hipError_t launch_bucket_select(const double *fit_row, const BucketArgs &bk, const RowPlan &rp, uint32_t K,
                                uint32_t *count_next, uint32_t *ties_next, int32_t *sel, hipStream_t s) {
  hipLaunchKernelGGL((bucket_select_kernel<true, kBucketThreads>), dim3(bk.nb), dim3(kBucketThreads), 0, s, fit_row, bk,
                     rp, K, count_next, ties_next, sel);
  return hipGetLastError();
}

hipError_t launch_splitters(const double *fit_row, const uint32_t *row_of, const int32_t *sel, uint32_t K,
                            uint32_t nb, uint64_t *split, uint64_t *thresh, uint32_t *count0, uint32_t *count1,
                            uint32_t *ties, uint32_t ties_words, hipStream_t s) {
  const uint32_t blocks = std::max<uint32_t>((kBucketCounters + 255) / 256, std::min<uint32_t>(ties_words / 1024, 1024u));
  hipLaunchKernelGGL(splitters_kernel, dim3(blocks), dim3(256), 0, s, fit_row, row_of, sel, K,
                     nb, split, thresh, count0, count1, ties, ties_words);
  return hipGetLastError();
}

hipError_t launch_placement(const uint32_t *genes, const uint32_t *best, const uint32_t *info, uint32_t Jn, uint32_t Jp,
                            uint32_t G, int32_t *slot_of_gpu, int32_t *batch_of_gpu, const uint32_t *err_in, uint32_t *err_out,
                            const HostSignal &done, hipStream_t s) {
  const uint32_t blocks = std::max<uint32_t>(1u, std::min<uint32_t>((G + kPlaceThreads - 1) / kPlaceThreads, 1024u));
  hipLaunchKernelGGL(placement_kernel, dim3(blocks), dim3(kPlaceThreads), 0, s, genes, best, info, Jn,
                     static_cast<uint32_t>(words_of(Jp / kLanes) * kLanes), G, slot_of_gpu, batch_of_gpu, err_in, err_out, done);
  return hipGetLastError();
}

hipError_t launch_best(const uint32_t *genes, const double *fit_row, const uint32_t *best, const uint32_t *stored,
                       const uint32_t *info, uint32_t Jn, uint32_t Jp, int32_t *batch_out, int32_t *gpus_out,
                       double *fit_out, const uint32_t *err_in, uint32_t *err_out, const HostSignal &done, hipStream_t s) {
  hipLaunchKernelGGL(best_kernel, dim3(1), dim3(256), 0, s, genes, fit_row, best, stored, info, Jn,
                     static_cast<uint32_t>(words_of(Jp / kLanes) * kLanes), batch_out, gpus_out, fit_out, err_in, err_out, done);
  return hipGetLastError();
}

}  // namespace ones
