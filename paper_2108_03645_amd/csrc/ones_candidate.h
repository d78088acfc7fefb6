// Device code that composes, repairs and scores one candidate schedule of the ONES search
// (arXiv 2108.03645, Section 3.2.2) on gfx950: one wave64 per candidate, the job columns across
// the 64 lanes, the rows of a column in the lane's registers, four to a register.  Shared by the
// kernels of ones_evolve.hip (a generation of a large pool) and ones_fused.hip (all generations of
// a small pool in one launch).
//
// A gene is a byte, the code of the job's GPU count: 0 = the job waits, e + 1 = 2^e GPUs (at most
// 2^20).  Compose and repair work on four genes per instruction.  What this is bound by is the issue
// of vector instructions: with one gene per 32-bit register the kernel of a generation issued for
// 80 % of its cycles while it moved its bytes at the rate of a plain copy, so fewer bytes alone would
// have gained little.
#pragma once

#include "ones.h"
#include "ones_device.h"

#include <algorithm>
#include <type_traits>

#pragma clang fp contract(off)   // every fp64 product and sum is rounded on its own

namespace ones {
namespace {

constexpr size_t kLdsBudget = 160 * 1024;             // LDS of one gfx950 compute unit

// Keeps the instruction scheduler from interleaving two phases of a work item, or too many
// rows of one loop, which would keep all their registers live at once.
__device__ __forceinline__ void phase_fence() {
  asm volatile("" ::: "memory");        // loads stay on their side of the fence in the optimiser
  __builtin_amdgcn_sched_barrier(0);    // ... and in the instruction scheduler
}
__device__ __forceinline__ void fence_every(int i, int n) { if (i % n == n - 1) phase_fence(); }
// Forces x to be computed before the following fence (its producers cannot sink below it).
template <typename T> __device__ __forceinline__ void pin(T &x) { asm volatile("" : "+v"(x)); }
// The lane number, re-materialised so that nothing derived from it (LDS addresses, the first
// Philox round) is hoisted out of the work-item loop and kept live, or spilled, across it.
__device__ __forceinline__ int opaque(int v) { asm volatile("" : "+v"(v)); return v; }

// ------------------------------------------------------------------ RNG ------------
__device__ __forceinline__ uint32_t bounded(uint32_t w, uint32_t n) { return __umulhi(w, n); }

// Per-candidate draw: ranks of the two parents among the K survivors and the rotation of
// the repair order.  Counter block 0xFFFFFFFF is reserved for it.
struct Draw { uint32_t ra, rb, r; };

// t: the generation the draw is for.  One draw per lane (p may differ from lane to lane).
__device__ __forceinline__ Draw candidate_draw(const EvolveArgs &a, uint32_t t, uint32_t p) {
  const Words w = philox4x32_10(0xFFFFFFFFu, p, t, 0u, a.key0, a.key1);
  return Draw{bounded(w.w[0], a.K), bounded(w.w[1], a.K), bounded(w.w[2], a.Jp)};
}

// One 32-bit word per gene: the lane's rows 4q..4q+3, which share a register, share Philox block
// q*64 + lane, counter (q*64 + lane, p, t, 0).
// The first two of the ten rounds hardly depend on the candidate: in round 0 the product of the
// block number and, in round 1, the product of what comes of it are the same for every candidate,
// and the other products are the same in all lanes.  The former are kept in LDS (prefix), the latter
// are scalar, so a block costs 16 vector multiplications instead of 20.
constexpr uint32_t kPhiloxA = 0xD2511F53u, kPhiloxB = 0xCD9E8D57u;

// prefix of block number `block`: low and high half of round 1's product
__device__ __forceinline__ uint2 philox_prefix(uint32_t block, uint32_t key1) {
  const uint32_t x2 = __umulhi(block, kPhiloxA) ^ key1;
  return make_uint2(x2 * kPhiloxB, __umulhi(x2, kPhiloxB));
}

struct WordSource {                                  // what the blocks of one candidate share (wave-uniform)
  uint32_t u0, u2, u3, k0, k1;
  // counted: the round keys are counted up by the scalar unit for every block.  Otherwise they are kept, and, where there are no
  // registers for them, reloaded from lanes of a vector register, which takes a vector instruction each: better only for a single
  // block (a generation of the stress workload, eight blocks, 73.2 -> 71.4 us; a call of 50 of 16384 candidates on two words 866 -> 842; of
  // 20 of 8192 on one word 148 -> 150).
  __device__ __forceinline__ WordSource(const EvolveArgs &a, uint32_t t, uint32_t p, bool counted = false) {
    const uint64_t pb = static_cast<uint64_t>(t) * kPhiloxB;
    const uint64_t pa = static_cast<uint64_t>(static_cast<uint32_t>(pb >> 32) ^ p ^ a.key0) * kPhiloxA;
    k0 = a.key0 + 0x9E3779B9u;
    k1 = a.key1 + 0xBB67AE85u;
    if (counted) asm volatile("" : "+s"(k0), "+s"(k1));
    u0 = static_cast<uint32_t>(pb) ^ k0;
    u2 = static_cast<uint32_t>(pa >> 32) ^ k1;
    u3 = static_cast<uint32_t>(pa);
  }
  // the words of the lane's rows 4q .. 4q + 3
  __device__ __forceinline__ Words block(const uint2 *prefix, int q, int lane) const {
    const uint2 e = prefix[q * kLanes + lane];
    uint32_t x0 = e.y ^ u0, x1 = e.x, x2 = (static_cast<uint32_t>(q * kLanes + lane) * kPhiloxA) ^ u2, x3 = u3;
    uint32_t ka = k0, kb = k1;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
      ka += 0x9E3779B9u;
      kb += 0xBB67AE85u;
      const uint64_t pa = static_cast<uint64_t>(x0) * kPhiloxA, pb = static_cast<uint64_t>(x2) * kPhiloxB;
      x0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pb >> 32), x1, ka, 0x96);   // three-input xor
      x2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(pa >> 32), x3, kb, 0x96);
      x1 = static_cast<uint32_t>(pb);
      x3 = static_cast<uint32_t>(pa);
    }
    return Words{{x0, x1, x2, x3}};
  }
};

// --------------------------------------------------------- wave primitives ---------
// DPP controls (gfx9): row_shr:n shifts within a row of 16 lanes, row_bcast:15 / :31 copy the
// last lane of a row / of the lower half-wave into the following row(s).
constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

template <int Ctrl, int RowMask, bool Bound>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), Ctrl, RowMask, 0xF, Bound));
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  v += dpp_or_zero<kRowShr + 1, 0xF, true>(v);
  v += dpp_or_zero<kRowShr + 2, 0xF, true>(v);
  v += dpp_or_zero<kRowShr + 4, 0xF, true>(v);
  v += dpp_or_zero<kRowShr + 8, 0xF, true>(v);
  v += dpp_or_zero<kRowBcast15, 0xA, false>(v);
  v += dpp_or_zero<kRowBcast31, 0xC, false>(v);
  return v;
}

// v of the lane before this one, `first` for lane 0.  (Two shifts: the one across the wave, wave_shr, does not work here.)
__device__ __forceinline__ uint32_t from_lane_before(uint32_t v, uint32_t first) {
  const int rows = __builtin_amdgcn_update_dpp(static_cast<int>(first), static_cast<int>(v), kRowBcast15, 0xE, 0xF, false);
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(rows, static_cast<int>(v), kRowShr + 1, 0xF, 0xF, false));
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return __builtin_amdgcn_readlane(wave_inclusive_scan(v), kLanes - 1);
}

// The sum that a xor butterfly 32, 16, .., 1 over the lanes leaves in every lane (each step adds the
// partner's value, so the order of the additions is that of the butterfly), without LDS: gfx950 swaps
// halves and rows of 16 lanes between two registers; below that, what a lane holds only depends
// on its place among the last 2^k lanes, so a rotation of the row stands for the xor.
__device__ __forceinline__ double butterfly_sum(double v) {
  auto halves = [](double x, auto swap) {             // x of this lane's half (row) of a pair, x of the other's
    const uint64_t bits = static_cast<uint64_t>(__double_as_longlong(x));
    const auto lo = swap(static_cast<uint32_t>(bits)), hi = swap(static_cast<uint32_t>(bits >> 32));
    return __hiloint2double(static_cast<int>(hi[0]), static_cast<int>(lo[0])) +
           __hiloint2double(static_cast<int>(hi[1]), static_cast<int>(lo[1]));
  };
  v = halves(v, [](uint32_t w) { return __builtin_amdgcn_permlane32_swap(w, w, false, false); });
  v = halves(v, [](uint32_t w) { return __builtin_amdgcn_permlane16_swap(w, w, false, false); });
  auto add_from = [](double x, auto ctrl) {
    constexpr int kCtrl = decltype(ctrl)::value;
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), kCtrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), kCtrl, 0xF, 0xF, true);
    return x + __hiloint2double(hi, lo);
  };
  v = add_from(v, std::integral_constant<int, 0x128>{});    // row_ror:8
  v = add_from(v, std::integral_constant<int, 0x124>{});    // row_ror:4
  v = add_from(v, std::integral_constant<int, 0x4E>{});     // quad_perm 2,3,0,1
  return add_from(v, std::integral_constant<int, 0xB1>{});  // quad_perm 1,0,3,2
}

// ------------------------------------------------------------- four genes at once --
// All byte values below are under 128, so that sums and differences with the top bits set do not
// run over into the neighbouring byte.
constexpr uint32_t kTops = 0x80808080u, kOnes = 0x01010101u, kSevens = 0x7F7F7F7Fu;

// 0x7F in the bytes whose top bit is set in t, 0 elsewhere
__device__ __forceinline__ uint32_t spread_tops(uint32_t t) {
  const uint32_t f = t & kTops;
  return f - (f >> 7);
}
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) { return spread_tops(v + kSevens); }
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t yes, uint32_t no) { return (yes & mask) | (no & ~mask); }
__device__ __forceinline__ uint32_t max_bytes(uint32_t x, uint32_t y) { return pick(spread_tops((x | kTops) - y), x, y); }
__device__ __forceinline__ uint32_t min_bytes(uint32_t x, uint32_t y) { return pick(spread_tops((x | kTops) - y), y, x); }

// What the words of codes may hold, and so how their GPUs are counted (the launcher of the evolve kernels decides by the table).
// kNarrow: codes up to 7 (no job of the table takes more than 64 GPUs, the usual case), counted by one
// byte look-up, which is wrong for any larger code.  kMiddle: codes up to 12 (2048 GPUs), by two: the
// first knows the codes up to 7 and counts 8 to 12 as 0 (those selectors of v_perm_b32 pick no byte of this
// table), the second, which counts in 128 GPUs, the other way round (selector 12 - code).  kWide: any code,
// shifted one by one, which takes 14 instructions a word where kMiddle takes 5.  kOneRow: one row
// of job slots, so a word holds a single gene, of any code.
enum Genes { kNarrow, kMiddle, kWide, kOneRow };
constexpr uint32_t kNarrowCodes = 7, kMiddleCodes = 12;

// The GPUs of words of codes, added up.
template <Genes kGenes>
struct GpuSum {
  uint32_t sum = 0, high = 0;
  __device__ __forceinline__ void add(uint32_t codes) {
    if (kGenes == kOneRow) {
      sum += (1u << codes) >> 1;
    } else if (kGenes == kWide) {
#pragma unroll
      for (int k = 0; k < 4; ++k) sum += (1u << ((codes >> (8 * k)) & 31u)) >> 1;
    } else {
      sum = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(0x40201008u, 0x04020100u, codes), 0u, sum);
      if (kGenes == kMiddle)
        high = __builtin_amdgcn_sad_u8(__builtin_amdgcn_perm(0x00000001u, 0x02040810u, 0x0C0C0C0Cu - codes), 0u, high);
    }
  }
  __device__ __forceinline__ uint32_t total() const { return kGenes == kMiddle ? sum + (high << 7) : sum; }
};

// ------------------------------------------------------------- job table in LDS ----
struct Smem {
  // a byte per gene, four rows to a word, word q*64 + lane (like the genomes): codes of the GPU count
  // a waiting job resumes with and of the one at its limit R_j, number of outcomes of a redraw
  // (0: empty slot), last outcome that gives the former; after a table change also the distance
  // from a stored code to the new one (biased; 0: the slot changed hands) and the arrived jobs (0x7F)
  uint32_t *start, *most, *draws, *lift, *shift, *fresh;
  uint32_t *bl;      // log2 of the local batch (when the term table does not fit)
  uint2    *prefix;  // [Q][64] Philox prefixes
  double   *abl, *cc, *d, *Y;   // [Q*256] model parameters (when the term table does not fit)
  double   *terms;   // [E][4Q][64] T_j c_j of job (row, lane) at GPU-count code e, or null
  uint64_t *split;   // [kMaxBuckets] bucket splitters, then [1] the K-th survivor's score bits
  uint2    *rank;    // [Q][64] in the same place, when a new table is served by executed time (no buckets then):
                     // ranks of the four rows, 16 bits each, the top one set
  // start and most again, a byte per slot in the order the repair visits them from lane 0, row 0 on, the first
  // kWindowAhead once more behind the last (only where the repair walks, see Window)
  uint8_t  *start_at, *most_at;
  uint8_t  *coins;   // [waves][coin_stride] the coins of a crossover over the GPUs, then the genes near the start of a repair
  uint32_t *free_in_group; // [groups] free rows in each group of kRowGroupWords bitmap words
  uint32_t *rows;          // [4 * kRound] rows of the slots this workgroup fills in the current round
  uint64_t *drawn;         // [4 * kRound] the draws of those slots (PackedDraw)
  uint32_t *next_item;     // [1] the next work item of the round that no wave has taken yet
};

constexpr uint32_t kRound = 128;                     // survivors' ranks a workgroup covers between two barriers

constexpr uint32_t row_groups(uint32_t rows) {
  return ((rows + 31) / 32 + kRowGroupWords - 1) / kRowGroupWords;
}

// LDS scratch per wave: the coin words of the cluster's GPUs with their running counts, for the crossover
// over the GPUs; one more than they fill, for the count below the GPU after the last, and whole lanes of four.  (With room for
// kMaxCoinGpus on every cluster, and rounds of 256 ranks, one workgroup was resident where two are: 585 slots,
// 3767 GPUs, pool 17084, 35 us a generation's launch; now 30.)
inline uint32_t coin_stride(const EvolveArgs &a) {
  return a.per_gpu ? (a.G / 32 + 4) / 4 * 4 * 8 : 0u;
}

// The genes near the job a repair starts from, in visiting order: kSide lanes' columns before that job's lane and
// kSide from it on, 4Q bytes each (see in_window).
template <int Q>
struct Window {
  static constexpr int kSide = Q <= 2 ? 32 : Q <= 4 ? 16 : 8;
  static constexpr int kPositions = kSide * 4 * Q;   // of either side
  static constexpr int kBytes = 2 * kPositions;
};
constexpr uint32_t kWindowAhead = 256;               // largest kPositions
constexpr uint32_t window_bytes(uint32_t Q) { return (Q <= 2 ? 64 : Q <= 4 ? 32 : 16) * 4 * Q; }
static_assert(Window<1>::kBytes == window_bytes(1) && Window<2>::kBytes == window_bytes(2) && Window<3>::kBytes == window_bytes(3) &&
              Window<4>::kBytes == window_bytes(4) && Window<5>::kBytes == window_bytes(5) && Window<8>::kBytes == window_bytes(8), "the same window");
static_assert(Window<2>::kPositions <= kWindowAhead && Window<4>::kPositions <= kWindowAhead && Window<8>::kPositions <= kWindowAhead,
              "start_at and most_at reach as far as the window");
// Their LDS beside the wave's scratch.
constexpr size_t walk_table_bytes(uint32_t Q) { return 2 * (static_cast<size_t>(Q) * 4 * kLanes + kWindowAhead); }

constexpr uint32_t kTieBytes = kTieClasses * 6;
static_assert(kTieBytes <= 3 * kLanes * 4, "the copies' counts fit in the place of three arrays of one word");
// E = entries per job of the term table kept in LDS, 0 = keep the four model parameters.
constexpr size_t smem_bytes(uint32_t Q, int waves, uint32_t E, uint32_t rows, uint32_t stride, bool walk = false) {
  const size_t words = static_cast<size_t>(Q) * kLanes;
  return words * 4 * 8 * (E ? E : 4) + (kMaxBuckets + 1) * 8 + 4 * kRound * 8 + words * 8 + words * 4 * 7 + (walk ? walk_table_bytes(Q) : 0) +
         static_cast<size_t>(waves) * stride + static_cast<size_t>(row_groups(rows)) * 4 + 4 * kRound * 4 + 16 + (E ? 0 : kTieBytes);
}
// Children of this workgroup that are copies of a class of survivors (see kTieRun), [kTieClasses], and, 16 bits each behind them, the
// bucket they belong to.  Only counted under the table that the genes are stored under, and so in the place of shift, fresh and bl,
// unless the term table does not fit, when all three are staged.  (In a place of their own, 1 KB, they cost shapes at the edge of a
// compute unit's LDS a workgroup or the table of terms: six generations of 32768 candidates, 1516 slots, jobs of up to 512 GPUs 446 us,
// 338 here; 492, 4096, over 2304 GPUs 328 and 279; 1004, 32 GPUs 268 and 257.)
__device__ __forceinline__ uint32_t *tie_counts(const Smem &s, uint32_t E) { return E ? s.shift : s.next_item + 4; }
__device__ __forceinline__ uint16_t *tie_buckets(uint32_t *counts) { return reinterpret_cast<uint16_t *>(counts + kTieClasses); }
// A compute unit hands LDS out in pieces of so much.
constexpr size_t kLdsPiece = 1280;
constexpr size_t lds_taken(size_t bytes) { return (bytes + kLdsPiece - 1) / kLdsPiece * kLdsPiece; }

template <int Q>
__device__ __forceinline__ Smem carve(unsigned char *at, uint32_t E, uint32_t waves, uint32_t stride, bool walk = false) {
  constexpr uint32_t kWords = Q * kLanes;
  Smem s;
  s.abl = reinterpret_cast<double *>(at);
  s.cc = s.abl + 4 * kWords;
  s.d = s.cc + 4 * kWords;
  s.Y = s.d + 4 * kWords;
  s.terms = E ? s.abl : nullptr;
  s.split = reinterpret_cast<uint64_t *>(s.abl + static_cast<size_t>(4 * kWords) * (E ? E : 4));
  static_assert(kWords <= kMaxBuckets, "the ranks fit in the splitters' place");
  s.rank = reinterpret_cast<uint2 *>(s.split);
  s.drawn = s.split + kMaxBuckets + 1;
  s.prefix = reinterpret_cast<uint2 *>(s.drawn + 4 * kRound);
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
  s.rows = reinterpret_cast<uint32_t *>(s.coins + static_cast<size_t>(waves) * stride);
  s.next_item = s.rows + 4 * kRound;
  s.free_in_group = s.next_item + 4 + (E ? 0 : kTieBytes / 4);
  return s;
}

// Distances between codes are kept above 0: the code of 2^(x - mu) GPUs is x - mu + 1, and every log2
// of a batch or a local batch lies in 0 .. 30.
constexpr uint32_t kBias = 31;

// Stages the job table into LDS, the work dealt to the `threads` threads (whole waves) that call it
// with tid = 0 .. threads - 1.  R: rows of job slots (at most 4Q).  changed: genes are stored under
// another table (tab.stored).  No barrier at the end: the caller places one before the first use.
// What a workgroup stages comes from memory in one or two trips: every thread issues all its loads,
// up to kStageBatch of a kind, before the first LDS store waits for one.  (In loops of one load and
// one store each a pool of 8192 spent 4.5 of its workgroups' 9 us here.)
constexpr int kStageBatch = 4;
template <int Q>
__device__ __forceinline__ void stage_table(const EvolveArgs &a, const Smem &s, uint32_t E, bool changed, uint32_t tid,
                                            uint32_t threads, bool walk = false) {
  const JobTable &tab = a.tab;
  const uint32_t R = a.Jp / kLanes;
  constexpr uint32_t kWords = Q * kLanes;
  const uint32_t l = tid % kLanes, tiles = E * 4 * Q, tile_step = threads / kLanes;
  const uint32_t splits = a.bk.nb != 0 ? kMaxBuckets + 1 : 0u;
  uint64_t split[kStageBatch];
  double term[kStageBatch];
  // the term table: global memory holds it row-major ([row][code][lane]); here the code is the slowest
  // index, so that a row's part of the LDS address is a compile-time offset (tiles of 64 entries)
  auto load_splits = [&](uint32_t from) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u) {
      const uint32_t q = from + u * threads;
      if (q < splits) split[u] = q < kMaxBuckets ? a.bk.split[q] : *a.bk.thresh;
    }
  };
  auto load_terms = [&](uint32_t from) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u) {
      const uint32_t tile = from + u * tile_step, e = tile / (4 * Q), row = tile % (4 * Q);
      term[u] = 0.0;
      if (tile < tiles && row < R) term[u] = tab.terms[(row * E + e) * kLanes + l];
    }
  };
  auto store_splits = [&](uint32_t from) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u)
      if (from + u * threads < splits) s.split[from + u * threads] = split[u];
  };
  auto store_terms = [&](uint32_t from) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u)
      if (from + u * tile_step < tiles) s.terms[(from + u * tile_step) * kLanes + l] = term[u];
  };
  load_splits(tid);
  load_terms(tid / kLanes);
  const bool by_time = changed && a.new_first && a.time_rank != nullptr;       // the buckets are off: no splitters
  for (uint32_t w = tid; w < kWords; w += threads) {
    const uint32_t start = tab.start[w], most = tab.most[w], draws = tab.draws[w], lift = tab.lift[w];
    s.prefix[w] = philox_prefix(w, a.key1);
    if (changed || E == 0) {
      uint32_t shift = 0, fresh = 0, bl = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t row = w / kLanes * 4 + k, j = row * kLanes + w % kLanes;
        if (row < R) {
          const uint32_t now = tab.info[j], then = tab.stored[j];
          shift |= (info_reset(then) ? 0u : info_blexp(then) - info_mu(now) + kBias) << (8 * k);
          fresh |= (info_new(now) ? 0x7Fu : 0u) << (8 * k);
          bl |= info_blexp(now) << (8 * k);
        }
      }
      s.shift[w] = shift;
      s.fresh[w] = fresh;
      s.bl[w] = bl;
    }
    if (by_time) {
      uint32_t rank[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t row = w / kLanes * 4 + k;
        rank[k] = row < R ? a.time_rank[row * kLanes + w % kLanes] | 0x8000u : 0xFFFFu;
      }
      s.rank[w] = make_uint2(rank[0] | rank[1] << 16, rank[2] | rank[3] << 16);
    }
    s.start[w] = start;
    s.most[w] = most;
    if (walk) {
      const uint32_t at = w % kLanes * Q + w / kLanes;               // of the word in visiting order
      uint32_t *start_at = reinterpret_cast<uint32_t *>(s.start_at), *most_at = reinterpret_cast<uint32_t *>(s.most_at);
      start_at[at] = start;
      most_at[at] = most;
      if (at < kWindowAhead / 4) {
        start_at[kWords + at] = start;
        most_at[kWords + at] = most;
      }
    }
    s.draws[w] = draws;
    s.lift[w] = lift;
  }
  store_splits(tid);
  store_terms(tid / kLanes);
  for (uint32_t q = tid + kStageBatch * threads; q < splits; q += kStageBatch * threads) { load_splits(q); store_splits(q); }
  for (uint32_t t = tid / kLanes + kStageBatch * tile_step; t < tiles; t += kStageBatch * tile_step) { load_terms(t); store_terms(t); }
  if (E == 0) {
    for (uint32_t j = tid; j < 4 * kWords; j += threads) {
      const bool real = j < a.Jp;
      s.abl[j] = real ? tab.abl[j] : 0.0;
      s.cc[j] = real ? tab.cc[j] : 0.0;
      s.d[j] = real ? tab.d[j] : 0.0;
      s.Y[j] = real ? tab.Y[j] : 0.0;
    }
  }
}

// ------------------------------------------------------------------ draws ----------
// A slot's draw as the waves find it in LDS: genome rows of the two parents (21 bits each; a pool has at
// most 1.25 * 2^20 rows), lane and row of the job the repair starts from.
struct PackedDraw {
  uint32_t lo, hi;
  __device__ __forceinline__ uint32_t row_a() const { return lo & 0x1FFFFFu; }
  __device__ __forceinline__ uint32_t row_b() const { return (lo >> 21) | ((hi & 0x3FFu) << 11); }
  __device__ __forceinline__ uint32_t lane() const { return (hi >> 10) & 63u; }
  __device__ __forceinline__ uint32_t row() const { return hi >> 16; }
};
__device__ __forceinline__ uint64_t pack_draw(uint32_t row_a, uint32_t row_b, uint32_t r, uint32_t R) {
  return static_cast<uint64_t>(row_a) | (static_cast<uint64_t>(row_b) << 21) |
         (static_cast<uint64_t>(r / R) << 42) | (static_cast<uint64_t>(r % R) << 48);
}
__device__ __forceinline__ PackedDraw draw_at(const uint64_t *drawn, uint32_t i) {
  const uint64_t v = drawn[i];
  return PackedDraw{static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))),
                    static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)))};
}

// ------------------------------------------------------------------ free rows ----
// Bits of bitmap word w that stand for free rows (rows beyond P + K count as taken).
__device__ __forceinline__ uint32_t free_bits(const uint32_t *occupied, uint32_t w, uint32_t rows) {
  const uint32_t words = (rows + 31) / 32;
  if (w >= words) return 0u;
  uint32_t f = ~occupied[w];
  if (w == words - 1 && rows % 32 != 0) f &= (1u << (rows % 32)) - 1u;
  return f;
}

// Every workgroup builds the same small index: the number of free rows in each group of
// kRowGroupWords bitmap words.  The first bitmap loads are issued ahead of the rest.
constexpr int kIndexAhead = 4;                       // groups per wave whose words are loaded ahead

struct IndexLoads { uint32_t bits[kIndexAhead]; };

__device__ __forceinline__ IndexLoads index_free_rows_begin(const EvolveArgs &a, int lane) {
  const uint32_t rows = a.P + a.K;
  const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  IndexLoads ld;
#pragma unroll
  for (int k = 0; k < kIndexAhead; ++k) ld.bits[k] = free_bits(a.occupied, (wave + k * waves) * kRowGroupWords + lane, rows);
  return ld;
}

// Ends with a barrier.
__device__ __forceinline__ void index_free_rows_end(const EvolveArgs &a, const Smem &s, const IndexLoads &ld, int lane) {
  const uint32_t rows = a.P + a.K, words = (rows + 31) / 32;
  const uint32_t groups = (words + kRowGroupWords - 1) / kRowGroupWords;
  const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < kIndexAhead; ++k) {
    const uint32_t n = wave_sum(__popc(ld.bits[k]));
    if (lane == 0 && wave + k * waves < groups) s.free_in_group[wave + k * waves] = n;
  }
  for (uint32_t g = wave + kIndexAhead * waves; g < groups; g += waves) {
    const uint32_t n = wave_sum(__popc(free_bits(a.occupied, g * kRowGroupWords + lane, rows)));
    if (lane == 0) s.free_in_group[g] = n;
  }
  __syncthreads();
}

// One wave lists the free rows number q0 .. q0 + count - 1 (in ascending order; all below the
// number of free rows) into dst.
__device__ __forceinline__ void list_free_rows(const EvolveArgs &a, const Smem &s, uint32_t q0, uint32_t count,
                                               uint32_t *dst, int lane) {
  const uint32_t rows = a.P + a.K;
  const uint32_t groups = ((rows + 31) / 32 + kRowGroupWords - 1) / kRowGroupWords;
  // the group that holds free row q0, and the free rows before that group
  uint32_t g = groups, before = 0;
  for (uint32_t g0 = 0; g0 < groups; g0 += kLanes) {
    const uint32_t n = g0 + lane < groups ? s.free_in_group[g0 + lane] : 0u;
    const uint32_t incl = wave_inclusive_scan(n);
    const uint64_t beyond = __ballot(before + incl > q0);
    if (beyond != 0) {
      const int l = __builtin_amdgcn_readfirstlane(__ffsll(static_cast<long long>(beyond)) - 1);
      g = g0 + static_cast<uint32_t>(l);
      before += __builtin_amdgcn_readlane(incl - n, l);
      break;
    }
    before += __builtin_amdgcn_readlane(incl, kLanes - 1);
  }
  // position in dst of the first free row of the group being read
  int32_t base = -static_cast<int32_t>(q0 - before);
  for (; g < groups && base < static_cast<int32_t>(count); ++g) {
    const uint32_t w = g * kRowGroupWords + lane;
    uint32_t bits = free_bits(a.occupied, w, rows);
    const uint32_t n = __popc(bits);
    const uint32_t incl = wave_inclusive_scan(n);
    int32_t pos = base + static_cast<int32_t>(incl - n);
    while (bits) {
      if (pos >= 0 && pos < static_cast<int32_t>(count)) dst[pos] = w * 32 + (__ffs(static_cast<int>(bits)) - 1);
      bits &= bits - 1;
      ++pos;
    }
    base += static_cast<int32_t>(__builtin_amdgcn_readlane(incl, kLanes - 1));
  }
}

// The kernel's own argument block, for values that only a rare path needs: read there, at the
// point of use, they are not carried (and spilled) through every work item.  Valid in kernels
// whose argument block starts with one EvolveArgs passed by value, which every kernel that
// includes this header must take (each of them says so at its signature).
using KernelArgs = const __attribute__((address_space(4))) EvolveArgs;
__device__ __forceinline__ KernelArgs *kernel_args() {
  KernelArgs *ka = (KernelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(ka));
  return ka;
}

// A row index is kept inside the genome array whatever the free-row list holds, so that a mistake
// in it cannot turn into a stray access; but such a mistake must not pass unnoticed either.
// Every row a slot gets passes through checked_row, when the kernel takes or records the rows of a round
// or of a call: a clamp that changes a value raises the context's fault word, which ones_export reports.
// (The survivors' rows are such rows.  The word is raised at once: a note in LDS needs clearing before the
// first check, which cost a barrier, or 0.5 of 87 us on the stress workload where the check waited for one.)
__device__ __forceinline__ uint32_t checked_row(uint32_t row, uint32_t n_rows) {
  if (row >= n_rows) atomicOr(kernel_args()->fault, 1u);
  return min(row, n_rows - 1);
}

// Row listed at position i of the current round (wave-uniform); never outside the genome array.
// (It reads entries that checked_row sees.)
__device__ __forceinline__ uint32_t row_at(const Smem &s, uint32_t i, const EvolveArgs &a) {
  return min(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(s.rows[i])), a.P + a.K - 1);
}

// ------------------------------------------------------------------ genes ----------
// Biased codes pulled inside the job's window (an empty slot's window is 0), the bias taken off.
__device__ __forceinline__ uint32_t into_window(uint32_t biased, uint32_t start, uint32_t most) {
  return min_bytes(max_bytes(biased, start + kBias * kOnes), most + kBias * kOnes) - kBias * kOnes;
}

// Redraw of four genes from k in [0, n) each: 0 = the job is pre-empted, else the batch 2^(lo + k - 1)
// on the GPUs it takes, with the free lift to the per-GPU max batch: the code start while k is at most lift, and one more for
// each outcome beyond (the last one is the batch limit, so nothing has to be cut off above).
__device__ __forceinline__ uint32_t codes_of_draws(const Smem &s, int w, uint32_t k) {
  const uint32_t beyond = (k | kTops) - s.lift[w];               // top bits: not below lift
  return (s.start[w] + (beyond & spread_tops(beyond))) & nonzero_bytes(k);
}

// k of a mutant's four genes, drawn from the lower halves of their words.  (The products' third bytes: k is below 32.)
__device__ __forceinline__ uint32_t outcomes_drawn(const Words &w, uint32_t outcomes) {
  uint32_t product[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) product[u] = (w.w[u] & 0xFFFFu) * ((outcomes >> (8 * u)) & 0xFFu);
  return __builtin_amdgcn_perm(product[1], product[0], 0x0C0C0602u) | __builtin_amdgcn_perm(product[3], product[2], 0x06020C0Cu);
}

// Genes stored under another job table: the batch they stood for, pulled inside the new window and
// lifted for free to the per-GPU max batch; slots that changed hands wait.
template <int Q>
__device__ __forceinline__ void to_new_table(const Smem &s, int lane, uint32_t (&c)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int w = q * kLanes + lane;
    c[q] = into_window(c[q] + s.shift[w], s.start[w], s.most[w]) & nonzero_bytes(c[q]) & nonzero_bytes(s.shift[w]);
  }
}

template <int Q>
__device__ __forceinline__ void load_genes(const uint32_t *genes, uint32_t row, int lane, uint32_t (&c)[Q]) {
  const uint32_t *at = genes + static_cast<size_t>(row) * (Q * kLanes);
#pragma unroll
  for (int q = 0; q < Q; ++q) c[q] = at[q * kLanes + lane];
}

// 0xFF in byte k where words.w[k] < limit
__device__ __forceinline__ uint32_t words_below(const Words &w, uint32_t limit) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) m |= w.w[k] < limit ? 0xFFu << (8 * k) : 0u;
  return m;
}

// ------------------------------------------------------------------ repair ---------
// The bytes of word q that belong to rows before ir, ir > 4q.
__device__ __forceinline__ uint32_t rows_before(uint32_t ir, int q) {
  return ir >= 4u * q + 4u ? 0xFFFFFFFFu : (1u << (8 * (ir & 3u))) - 1u;
}

// Accept the longest prefix, in the rotated visiting order, of the asks (codes v, 0 = none) whose
// running sum of GPUs stays within limit.  Visiting order: column-major (a lane's rows are
// consecutive), starting at lane lr, row ir, wrapping.  On return the bytes of m are cleared where
// the ask was not accepted (elsewhere they stay); returns the accepted sum (wave-uniform).
// A lane's asks lie in one stretch of that order (lane lr's in two), so with the lanes' sums scanned
// every lane knows whether its stretch fits as a whole, and at most one stretch is cut: its rows
// are laid out over the lanes, a row each, scanned, and the outcome is written back to the lane.
// With kOneRow a stretch is a single ask and nothing is cut.
template <int Q, Genes kGenes>
__device__ __forceinline__ uint32_t accept_prefix(const uint32_t (&v)[Q], uint32_t (&m)[Q], uint32_t limit, uint32_t lr,
                                                  uint32_t ir, int lane) {
  static_assert(kGenes != kOneRow || Q == 1, "one row of job slots is one word");
  GpuSum<kGenes> lane_sum;
#pragma unroll
  for (int q = 0; q < Q; ++q) lane_sum.add(v[q]);
  const uint32_t run = lane_sum.total();
  const uint32_t incl = wave_inclusive_scan(run);
  const uint32_t total = __builtin_amdgcn_readlane(incl, kLanes - 1);
  if (total <= limit) return total;                // everything fits
  if (kGenes == kOneRow) {
    const uint32_t base = __builtin_amdgcn_readlane(incl - run, lr);             // asks visited after the wrap
    const uint32_t end = incl - base + (static_cast<uint32_t>(lane) < lr ? total : 0u);
    const bool fits = end <= limit;
    m[0] = fits ? m[0] : 0u;
    // what fits is what comes before the first lane, in visiting order, whose ask does not
    const uint64_t beyond = __ballot(!fits), after = beyond >> lr << lr;
    return __builtin_amdgcn_readlane(end - run, __ffsll(static_cast<long long>(after ? after : beyond)) - 1);
  }
  // lane lr's rows before ir (only that lane's value is used); ir is wave-uniform
  GpuSum<kGenes> pre;
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (ir > 4u * q) pre.add(v[q] & rows_before(ir, q));
  const uint32_t skipped = __builtin_amdgcn_readlane(pre.total(), lr);           // visited last, after the wrap
  const uint32_t base = __builtin_amdgcn_readlane(incl - run, lr) + skipped;     // asks visited after the wrap
  const uint32_t end = incl - base + (static_cast<uint32_t>(lane) < lr ? total : 0u);
  const uint32_t begin = end - (run - (static_cast<uint32_t>(lane) == lr ? skipped : 0u));
  const bool fits = end <= limit;
  uint32_t got = limit;                              // a cut between two stretches uses the limit up
  // the stretch that is cut: its lane, its rows [from, to), what is left for it
  const uint64_t cut = __ballot(begin < limit && !fits);
  const bool wrapped = total - skipped < limit;      // lane lr's second stretch; then every other one fits
  uint32_t b = lr, from = 0, to = ir, room = limit - (total - skipped);
  if (!wrapped) {
    b = cut ? static_cast<uint32_t>(__ffsll(static_cast<long long>(cut)) - 1) : 0u;
    from = b == lr ? ir : 0u;
    to = 4 * Q;
    room = limit - __builtin_amdgcn_readlane(begin, b);
  }
  if (!wrapped) {                                    // lane lr's second stretch lies beyond the limit
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (ir > 4u * q) m[q] &= static_cast<uint32_t>(lane) == lr ? ~rows_before(ir, q) : 0xFFFFFFFFu;
  }
  const uint32_t whole = fits ? 0xFFFFFFFFu : 0u;
  if (!wrapped && cut == 0) {
#pragma unroll
    for (int q = 0; q < Q; ++q) m[q] &= whole;
    return got;
  }
  uint32_t x = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t u = __builtin_amdgcn_readlane(v[q], b);
    x = (lane >> 2) == q ? u : x;
  }
  x = (x >> ((lane & 3) * 8)) & 31u;
  const bool inside = static_cast<uint32_t>(lane) >= from && static_cast<uint32_t>(lane) < to;
  const uint32_t sum = wave_inclusive_scan(inside ? (1u << x) >> 1 : 0u);
  const uint64_t within = __ballot(inside && sum <= room);                       // rows from .. of the accepted prefix
  const uint32_t count = static_cast<uint32_t>(__popcll(within));
  got = limit - room + (count ? __builtin_amdgcn_readlane(sum, from + count - 1) : 0u);
  uint32_t rows = static_cast<uint32_t>(within);
  if (wrapped) rows |= ~((1u << ir) - 1u);           // its first stretch fits
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t bits = (((rows >> (4 * q)) & 15u) * 0x00204081u) & kOnes;     // bit k to byte k
    m[q] &= static_cast<uint32_t>(lane) == b ? bits * 0xFFu : whole;
  }
  return got;
}

// What the repair changes lies near the job it starts from.  A candidate beyond the capacity loses the jobs at the end of
// the visiting order, just before that job, and the idle GPUs are used up by the first asks after it: on the stress
// workload 46 asks are accepted of 1270, in a stretch of some 75 positions, on the large one 17 of 430.  So the genes on both sides
// of it are laid out in LDS in visiting order, and the wave walks along them, a gene per lane, 64 positions a step of some 25
// instructions; a cut and a fill round over whole genomes are 150 and 270 at eight words.
// The kernels are bound by the issue of vector instructions: a generation of the stress workload issued 5.0e7 with whole genomes
// and 3.8e7 walking (86 and 74 us in a search's first 300 generations; other steps have taken both down since); epochs: 200 slots, pool 8192
// 205 -> 192 us, 512 slots, pool 16384 820 -> 779, stress 1771 -> 1679.  A window that the walk leaves (few asks, or many idle GPUs) costs it some 100
// instructions; the round then goes on over whole genomes.  Where more than kPositions GPUs are idle it is not tried.
template <int Q>
__device__ __forceinline__ bool in_window(uint32_t lr, int lane, uint32_t &at) {
  at = (static_cast<uint32_t>(lane) - lr + Window<Q>::kSide) % kLanes;
  return 2 * Window<Q>::kSide >= kLanes || at < 2u * Window<Q>::kSide;
}
template <int Q>
__device__ __forceinline__ void stage_window(const uint32_t (&c)[Q], uint8_t *window, uint32_t lr, int lane) {
  uint32_t at;
  if (in_window<Q>(lr, lane, at)) {
    uint32_t *column = reinterpret_cast<uint32_t *>(window) + at * Q;
#pragma unroll
    for (int q = 0; q < Q; ++q) column[q] = c[q];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");         // the lanes read each other's bytes: one wave, whose LDS operations complete in order
}
template <int Q>
__device__ __forceinline__ void take_window(uint32_t (&c)[Q], const uint8_t *window, uint32_t lr, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  uint32_t at;
  if (in_window<Q>(lr, lane, at)) {
    const uint32_t *column = reinterpret_cast<const uint32_t *>(window) + at * Q;
#pragma unroll
    for (int q = 0; q < Q; ++q) c[q] = column[q];
  }
}

// Jobs from the end of the visiting order wait until the candidate has shed `excess` GPUs: those that more than
// the capacity are held up to, which is those with less than the excess after them.  Returns what they held, at least
// `excess`; 0 if the window ends before that (the registers hold the genes as they were).
template <int Q>
__device__ __forceinline__ uint32_t shed_excess(uint8_t *window, uint32_t excess, uint32_t ir, int lane) {
  const int32_t behind = Window<Q>::kPositions + static_cast<int32_t>(ir);       // positions of the window before the start
  uint32_t before = 0;
  for (int32_t at = behind - 1 - lane, steps = behind; steps > 0; at -= kLanes, steps -= kLanes) {
    const uint32_t code = at >= 0 ? window[at] : 0u, gpus = (1u << code) >> 1;
    const uint32_t incl = wave_inclusive_scan(gpus) + before;
    const bool waits = incl - gpus < excess;
    if (waits && at >= 0) window[at] = 0;
    before = __builtin_amdgcn_readlane(incl, kLanes - 1);
    if (before >= excess) return __builtin_amdgcn_readlane(incl, __popcll(__ballot(waits)) - 1);
  }
  return 0;
}

// Fill rounds as long as they end inside the window.  On return idle is what the last round that began found idle, and left what
// it has not handed out: 0, or that round has gone past the window and goes on behind it.
template <int Q>
__device__ __forceinline__ void fill_window(const Smem &s, uint8_t *window, uint32_t lr, uint32_t ir, int lane, uint32_t &idle, uint32_t &left) {
  const uint32_t ahead = Window<Q>::kPositions - ir;             // positions of the window from the start on
  static_assert(Window<Q>::kPositions - 4 * Q >= kLanes, "the first step lies inside the window");
  const uint32_t base = lr * (4 * Q) + ir + lane;
  uint8_t *genes = window + Window<Q>::kPositions + ir + lane;
  const uint8_t *starts = s.start_at + base, *mosts = s.most_at + base;
  uint32_t code = genes[0];                                      // the first step's stay in registers
  const uint32_t start = starts[0], most = mosts[0];
  for (;;) {
    left = idle;
    const uint32_t fit = 32 - __clz(static_cast<int>(idle));     // a power of two fits when its code is not above that of the idle GPUs
    // one step; true: the round ends in it
    auto step = [&](uint32_t &gene, uint32_t its_start, uint32_t its_most, bool inside, uint32_t from) {
      const bool waits = gene == 0;
      const uint32_t cost = waits ? its_start : gene;
      const bool asks = gene != its_most && cost <= fit && inside;
      if (__ballot(asks) == 0) return false;
      const uint32_t gpus = asks ? (1u << cost) >> 1 : 0u, incl = wave_inclusive_scan(gpus);
      const uint64_t beyond = __ballot(asks && incl > left);
      if (asks && incl <= left) {
        gene = waits ? its_start : gene + 1;
        genes[from] = static_cast<uint8_t>(gene);
      }
      if (beyond == 0) {
        left -= __builtin_amdgcn_readlane(incl, kLanes - 1);
        return left == 0;
      }
      left -= __builtin_amdgcn_readlane(incl - gpus, __ffsll(static_cast<long long>(beyond)) - 1);
      return true;
    };
    bool ends = step(code, start, most, true, 0);
    for (uint32_t from = kLanes; !ends && from < ahead; from += kLanes) {
      uint32_t gene = genes[from];
      ends = step(gene, starts[from], mosts[from], from + lane < ahead, from);
    }
    if (!ends || left == 0) return;
    idle = left;
  }
}

// Refresh + fill (Section 3.2.2) on codes c[]; window and lift already applied.
// kArrivals (only in the generation after a table change): the jobs that arrived with the table
// are served first (refresh (3)): each starts on the GPUs a waiting job resumes with while the
// capacity lasts, in visiting order, and the others are admitted to what is left: in visiting order
// too, or, with by_time (s.rank: position of every job in ascending order of executed time), least executed
// time first, so that the room is taken from the jobs with the largest T_processed.
// window: this wave's LDS for the genes near the start of the repair, with walk.
template <int Q, Genes kGenes, bool kArrivals>
__device__ __forceinline__ void repair(uint32_t (&c)[Q], const Smem &s, uint32_t G, uint32_t lr, uint32_t ir, int lane,
                                       uint32_t Jp, bool by_time, uint8_t *window, bool walk) {
  constexpr bool kWalks = kGenes != kOneRow;         // there one gene per lane is the whole genome
  lane = opaque(lane);                               // (nothing derived from it is kept from one candidate to the next)
  uint32_t used = 0;
  bool staged = false;
  if (kArrivals) {
    uint32_t v[Q], fresh[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t arrived = s.fresh[q * kLanes + lane];
      v[q] = fresh[q] = s.start[q * kLanes + lane] & arrived;
      c[q] &= ~arrived;
    }
    const uint32_t taken = accept_prefix<Q, kGenes>(v, fresh, G, lr, ir, lane);
    if (by_time) {
      // The running sum over the ranks never decreases, so the admitted jobs are the ranks below
      // some bound: the largest n whose first n ranks ask for no more than what is left.
      // The ranks are read from LDS, four with a load, in each of the search's up to log2(Jp) + 1 steps:
      // there is no room for them in registers, and from global memory, a rank a load, the generation
      // that serves the arrivals of 1608 jobs took 96 us where it now takes 44.
      const uint32_t cap = G - taken;
      // 0x7F for the jobs of word q with a rank below n (n <= 2048)
      auto ranked_below = [&](int q, uint32_t n) {
        const uint2 rank = s.rank[q * kLanes + lane];
        const uint32_t lower = rank.x - n * 0x10001u, upper = rank.y - n * 0x10001u;    // top bits: not below
        return spread_tops(~__builtin_amdgcn_perm(upper, lower, 0x07050301u));
      };
      uint32_t lo = 0, hi = Jp, fit = 0;                                   // the first lo ranks fit (sum fit)
      while (lo < hi) {                                                    // at most log2(Jp) + 1 steps
        const uint32_t mid = (lo + hi + 1) / 2;
        GpuSum<kGenes> below;
        phase_fence();                                                     // the ranks are not kept in registers
#pragma unroll
        for (int q = 0; q < Q; ++q) below.add(c[q] & ranked_below(q, mid));
        const uint32_t sum = wave_sum(below.total());
        if (sum <= cap) { lo = mid; fit = sum; } else { hi = mid - 1; }
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) c[q] &= ranked_below(q, lo);
      used = taken + fit;
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = c[q];
      used = taken + accept_prefix<Q, kGenes>(v, c, G - taken, lr, ir, lane);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) c[q] |= fresh[q];
  } else {
    // admit: jobs beyond the capacity in visiting order wait (Eq. 4)
    bool shed = false;
    if (kWalks && walk) {
      GpuSum<kGenes> held;
#pragma unroll
      for (int q = 0; q < Q; ++q) held.add(c[q]);
      used = wave_sum(held.total());
      shed = used <= G;
      // (a window that is expected to hold twice the jobs that have to wait)
      if (!shed && used - G <= used / (4 * kLanes / Window<Q>::kSide)) {
        stage_window<Q>(c, window, lr, lane);
        const uint32_t gone = shed_excess<Q>(window, used - G, ir, lane);
        shed = staged = gone != 0;
        used -= gone;
      }
    }
    if (!shed) {
      uint32_t v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = c[q];
      used = accept_prefix<Q, kGenes>(v, c, G, lr, ir, lane);
    }
  }
  // fill: a waiting job asks for its starting GPUs, a running one below its limit asks to double,
  // both only if the GPUs are there (a power of two fits when its code is not above that of the idle
  // GPUs).  Every round that accepts anything uses up idle GPUs, and a round that accepts nothing ends it.
  uint32_t idle = G - used, left = idle;
  bool behind = false;                               // the round that goes on has gone past the window
  if (kWalks && walk && idle != 0 && idle <= static_cast<uint32_t>(Window<Q>::kPositions)) {
    if (!staged) stage_window<Q>(c, window, lr, lane);
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    staged = true;
    fill_window<Q>(s, window, lr, ir, lane, idle, left);
    behind = left != 0;
  }
  if (kWalks && staged) take_window<Q>(c, window, lr, lane);
  if (left == 0) return;
  uint32_t waits[Q];                                 // 0x7F for the jobs that wait
#pragma unroll
  for (int q = 0; q < Q; ++q) waits[q] = ~nonzero_bytes(c[q]) & kSevens;
  for (;;) {
    const uint32_t fitting = kTops | (static_cast<uint32_t>(32 - __clz(static_cast<int>(idle))) * kOnes);
    uint32_t v[Q], m[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int w = q * kLanes + lane;
      const uint32_t cost = c[q] | (s.start[w] & waits[q]);
      m[q] = spread_tops(((c[q] ^ s.most[w]) + kSevens) & (fitting - cost));   // below its limit, and the GPUs are there
      v[q] = cost & m[q];
    }
    if (kWalks && behind) {                          // what lies in the window has had its turn
      const uint32_t at = (static_cast<uint32_t>(lane) - lr) % kLanes;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t later = at >= static_cast<uint32_t>(Window<Q>::kSide) ? 0xFFFFFFFFu : at != 0 || ir <= 4u * q ? 0u : rows_before(ir, q);
        m[q] &= later;
        v[q] &= later;
      }
    }
    const uint32_t got = accept_prefix<Q, kGenes>(v, m, left, lr, ir, lane);
    if ((got == 0 && left == idle) || got > left) break;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int w = q * kLanes + lane;
      c[q] += pick(waits[q], s.start[w], kOnes) & m[q];          // a running job's code goes up by one
      waits[q] &= ~m[q];
    }
    idle = left -= got;
    behind = false;
    if (idle == 0) break;
  }
}

// Eq. 3: sum over running jobs of T_j c_j = Y_j t_j / (local batch), t = a b + c log2(g) + d.
// Summation order: a lane's rows top to bottom, then a xor butterfly 32,16,..,1 over lanes.
// kRows: rows that can hold job slots (the terms of rows beyond the slots are 0).
// Of tables of few codes (kDirect<Q> at most) a look-up's address is a byte permute of the word of codes: a code's tile of the table
// takes 2^(8 + kTileShift) bytes, so its address is the code, shifted in its byte, above the low byte of the lane's.  Cut out of
// the word, scaled and added it takes two instructions and a quarter more.
template <int Q> constexpr bool kTiled = Q == 1 || Q == 2 || Q == 4 || Q == 8;
template <int Q> constexpr int kTileShift = Q == 1 ? 3 : Q == 2 ? 4 : Q == 4 ? 5 : 6;
template <int Q> constexpr uint32_t kDirect = kTiled<Q> ? 256u >> kTileShift<Q> : 0u;
template <int Q, int kRows = 4 * Q>
__device__ __forceinline__ double score(const uint32_t (&c)[Q], const Smem &s, uint32_t E, int lane) {
  using LdsTerms = const __attribute__((address_space(3))) double;
  double acc = 0.0;
  lane = opaque(lane);
  if (kRows > 1 && E != 0 && E <= kDirect<Q>) {
    const uint32_t column = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((LdsTerms *)(s.terms + lane)));
    const uint32_t above = (column >> 8) * kOnes;                // below 2^kTileShift: the table lies at the beginning of LDS
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t tiles = (c[q] << kTileShift<Q>) + above;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t at = __builtin_amdgcn_perm(tiles, column, 0x0C0C0000u | static_cast<uint32_t>(4 + k) << 8);
        acc = acc + ((LdsTerms *)static_cast<uintptr_t>(at))[(4 * q + k) * kLanes];
      }
      if (q % 2 == 1) { pin(acc); phase_fence(); }
    }
  } else if (E != 0) {
    // the job's term only depends on the code of its GPU count, and the table holds exactly the
    // value the formula below produces
    const double *column = s.terms + lane;
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const uint32_t code = (c[i / 4] >> (8 * (i % 4))) & 0xFFu;
      acc = acc + (column + code * (4 * Q * kLanes))[i * kLanes];
      if (i % 8 == 7) { pin(acc); phase_fence(); }
    }
  } else
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int j = lane + kLanes * i;
    const uint32_t code = (c[i / 4] >> (8 * (i % 4))) & 0xFFu;
    const uint32_t bl = (s.bl[(i / 4) * kLanes + lane] >> (8 * (i % 4))) & 0xFFu;
    const double lg = static_cast<double>(static_cast<int>(code) - 1);
    const double inv_bl = __hiloint2double(static_cast<int>((1023u - bl) << 20), 0);
    const double t = (s.abl[j] + s.cc[j] * lg) + s.d[j];
    const double term = (s.Y[j] * t) * inv_bl;
    acc = acc + (code ? term : 0.0);
    if (i % 4 == 3) { pin(acc); phase_fence(); }
  }
  return butterfly_sum(acc);
}

// The score of pool slot p, for a general selection that follows (the pointer is read from the
// kernel's argument block at the point of use, like the bucket storage below).
__device__ __forceinline__ void note_slot_score(uint32_t p, double f, int lane) {
  if (lane == 0) kernel_args()->slot_score[p] = f;
}

// A child or mutant that beats the K-th survivor joins the bucket of the survivors it falls
// between: bucket = number of splitters <= its score.  Scores at or above the threshold
// cannot be among the best K (the K survivors themselves are in the pool, in smaller slots).
__device__ __forceinline__ void drop_in_bucket(const Smem &s, uint32_t p, double f, int lane) {
  const uint64_t raw = static_cast<uint64_t>(__double_as_longlong(f));
  // the butterfly leaves the same sum in every lane; make that visible to the compiler
  // (the builtin returns a signed int: widen through uint32_t, not by sign extension)
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(raw >> 32)));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(raw)));
  const uint64_t bits = (static_cast<uint64_t>(hi) << 32) | lo;
  if (bits >= s.split[kMaxBuckets]) return;
  // two steps over the ascending splitters (the last ones are +inf): the sixteenth ones, then the
  // sixteen in front of the first of those that is above
  constexpr int kStep = kMaxBuckets / kLanes;
  static_assert(kStep <= kLanes, "one splitter per lane");
  const uint32_t block = kStep * static_cast<uint32_t>(__popcll(__ballot(s.split[lane * kStep + kStep - 1] <= bits)));
  const uint32_t b = block + static_cast<uint32_t>(__popcll(
                                 __ballot(lane < kStep && s.split[min(block + lane, kMaxBuckets - 1u)] <= bits)));
  // (split[b - 1] is the largest splitter that is not above the score)
  if (b >= static_cast<uint32_t>(kTieRun) && s.split[b - kTieRun] == bits && s.split[b - 1] == bits) {
    if (lane == 0) {
      KernelArgs *ka = kernel_args();
      const uint32_t c = (b - 1) / kTieRun, q = p - ka->K;
      uint32_t *counts = tie_counts(s, ka->term_lds);
      atomicAdd(&counts[c], 1u);
      tie_buckets(counts)[c] = static_cast<uint16_t>(b);
      atomicOr(&ka->bk.ties[static_cast<size_t>(c) * tie_words(ka->K) + q / 32], 1u << (q % 32));
    }
    return;
  }
  if (lane == 0) {
    // The pointers of the bucket storage are read from the kernel's argument block here, where
    // the few candidates that get this far need them, instead of being carried (and spilled)
    // through every work item.
    KernelArgs *ka = kernel_args();
    uint32_t *count = ka->bk.count;
    const uint32_t seg = ka->bk.seg;
    const uint32_t slot = atomicAdd(&count[b], 1u);
    if (slot == kManyInBucket) count[kManyFlag] = 1;
    if (slot < seg) {
      const size_t at = static_cast<size_t>(b) * seg + slot;
      ka->bk.keys[at] = bits;
      ka->bk.idx[at] = p;
    } else {                                               // bucket full: shared spill list
      const uint32_t at = atomicAdd(&count[kSpillCounter], 1u);
      ka->bk.spill_keys[at] = bits;
      ka->bk.spill_idx[at] = p;
      ka->bk.spill_bucket[at] = b;
    }
  }
}

// Uniform crossover over the GPUs (Section 3.2.2 on the encoding of Eq. 1).  Both parents are
// laid out as the reorder operator leaves them: the jobs in slot order on consecutive GPUs, cA
// resp. cB GPUs each, GPUs beyond the cluster do not exist.  Every GPU has a fair coin: heads,
// the first parent's job on it goes to the first child and the second parent's to the second
// child; tails, the other way round.  A child then runs each job on the largest power of two
// among the GPUs it inherited for it, inside the job's window.  On return cA holds the first
// child and cB the second.
// Coin of GPU i: bit i mod 32 of word (i mod 128) div 32 of Philox block (i div 128, p0, t, 3);
// lane l draws the coins of GPUs 128 l .. 128 l + 127.  coins: this wave's entries of LDS (coin_stride),
// each a coin word and, above it, the number of heads on the GPUs before it.
// kFeasible: both parents are known to fit the cluster (they were repaired under the current
// job table), so no GPU position needs to be cut off at the cluster's size.
template <int Q, bool kFeasible>
__device__ __forceinline__ void crossover_over_gpus(const EvolveArgs &a, uint32_t t, const Smem &s, uint64_t *coins, uint32_t p0,
                                                    int lane, uint32_t (&cA)[Q], uint32_t (&cB)[Q]) {
  const uint32_t R = a.Jp / kLanes, entries = kernel_args()->coin_stride / 8;
  {
    const Words w = philox4x32_10(static_cast<uint32_t>(lane), p0, t, 3u, a.key0, a.key1);
    const uint32_t heads = __popc(w.w[0]) + __popc(w.w[1]) + __popc(w.w[2]) + __popc(w.w[3]);
    uint32_t before = wave_inclusive_scan(heads) - heads;
    if (4u * lane < entries) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        coins[4 * lane + k] = (static_cast<uint64_t>(before) << 32) | w.w[k];
        before += __popc(w.w[k]);
      }
      if (entries > 4u * kLanes && lane == kLanes - 1) coins[4 * kLanes] = static_cast<uint64_t>(before) << 32;
    }
  }
  // the lanes read each other's entries: one wave, whose LDS operations complete in order
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  phase_fence();
  // From here on a register holds a number for each parent, the second parent's in its upper half: GPUs and heads are at most
  // kMaxCoinGpus, so that one scan, one shift over the lanes and one subtraction serve both.
  static_assert(kMaxCoinGpus < 1 << 15, "two counts, and their sum, in 16 bits each");
  // heads among the GPUs below x: GPU x's word, and of its coins the low x mod 32 (a bit field's width is taken mod 32)
  auto heads_below = [&](uint32_t word, uint32_t x) {
    const uint64_t e = coins[word];
    return static_cast<uint32_t>(e >> 32) + static_cast<uint32_t>(__popc(__builtin_amdgcn_ubfe(static_cast<uint32_t>(e), 0u, x)));
  };
  // A job's first GPU is the GPU after its predecessor's last one (slot order: the lane to the left,
  // or the last lane of the row above), so the heads below a job's range are looked up once, at
  // its end, and its start takes the predecessor's value.
  // Bound by the issue of vector instructions, some 40 a row (70 with a register per parent, a clamp of the word's number and a mask
  // made by shifts: an epoch of eight generations on the stress cluster 1210 us, now 1056).
  uint32_t carry_a = 0, carry_b = 0;                             // GPUs of the rows above (wave-uniform); kFeasible: carry_a, both parents'
  uint32_t above = 0;                                            // heads below the first GPU of the row (wave-uniform)
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    uint32_t first = 0, second = 0;                              // 31 - the children's codes before the window
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (static_cast<uint32_t>(4 * q + k) >= R) {               // no job slots (wave-uniform)
        first |= 31u << (8 * k); second |= 31u << (8 * k);
        continue;
      }
      const uint32_t ga = (1u << ((cA[q] >> (8 * k)) & 31u)) >> 1, gb = (1u << ((cB[q] >> (8 * k)) & 31u)) >> 1;
      uint32_t gpus, end;
      if (kFeasible) {
        gpus = gb << 16 | ga;
        const uint32_t incl = wave_inclusive_scan(gpus);
        end = carry_a + incl;
        carry_a += __builtin_amdgcn_readlane(incl, kLanes - 1);
      } else {
        const uint32_t incl_a = wave_inclusive_scan(ga), incl_b = wave_inclusive_scan(gb);
        const uint32_t end_a = carry_a + incl_a, end_b = carry_b + incl_b;
        end = min(end_b, a.G) << 16 | min(end_a, a.G);
        gpus = end - (min(end_b - gb, a.G) << 16 | min(end_a - ga, a.G));
        carry_a += __builtin_amdgcn_readlane(incl_a, kLanes - 1);
        carry_b += __builtin_amdgcn_readlane(incl_b, kLanes - 1);
      }
      const uint32_t at_end = heads_below(end >> 21, end >> 16) << 16 | heads_below(__builtin_amdgcn_ubfe(end, 5u, 11u), end);
      const uint32_t heads = at_end - from_lane_before(at_end, above);
      above = __builtin_amdgcn_readlane(at_end, kLanes - 1);
      const uint32_t tails = gpus - heads;
      const uint32_t n1 = (heads & 0xFFFFu) + (tails >> 16), n2 = (tails & 0xFFFFu) + (heads >> 16);
      first |= static_cast<uint32_t>(__builtin_clz(2 * n1 + 1)) << (8 * k);            // of 0 GPUs: 31
      second |= static_cast<uint32_t>(__builtin_clz(2 * n2 + 1)) << (8 * k);
    }
    first = 31 * kOnes - first; second = 31 * kOnes - second;    // no byte borrows
    const int w = q * kLanes + lane;
    const uint32_t start = s.start[w], most = s.most[w];
    cA[q] = min_bytes(max_bytes(first, start), most) & nonzero_bytes(first);
    cB[q] = min_bytes(max_bytes(second, start), most) & nonzero_bytes(second);
    phase_fence();
  }
}

}  // namespace
}  // namespace ones
