// Embedding gradients by ID (Alg. 2, push responder): after the occurrences
// are sorted by ID, every run of equal IDs is one segment.  For each segment
// this computes its ID and start (dedup), c_r (number of contributions that
// hold the ID: the divisor of Alg. 2, the count of workers that sent the ID),
// W_r (contributions whose weight for the ID is non-zero), and the weighted
// sum of the rows divided by c_r (or by K).  The weight of a contribution for
// a row is its token weight, or in per-ID mode [max(0, tag[r] - tau_m + 1) <=
// iota] with the tag as it was before this step.
//
// Work is split by sorted position, not by segment, so a Zipf-hot ID with
// millions of occurrences is spread over many blocks and no floating-point
// atomics are used.  Two passes over the sorted positions:
//  * seg_meta: a lane takes four consecutive positions (16-byte key and index
//    loads) and finds the contribution of each occurrence through a bucket
//    table in LDS, its weight, and whether it starts a run of equal IDs or a
//    new contribution inside one.  It numbers the segments, writes their IDs
//    and starts, and packs (occurrence index, flags) into one word per position.
//  * seg_rows: a group of LPR lanes (one 16-byte column slice per lane) walks 8
//    to 128 consecutive positions (rows_span) from their packed words, keeping
//    four row gathers in flight and summing each run in float64, and applies
//    the optimiser to the finished rows where the caller asks for it.  Runs
//    that cross group boundaries are joined in LDS; runs that cross tile
//    boundaries leave one partial per tile end, joined by seg_fixup in a fixed
//    order, so results are deterministic.
//
// With the split hot-key plan the sort hands over the cold keys and, apart,
// the occurrences of each hot ID (a few hundred IDs holding about half of all
// occurrences under Zipf skew).  The passes above then run over the cold keys
// only and write each segment at its place among all IDs; each hot ID is one
// long segment, summed by hot_rows (per chunk of some 1000 to 4096
// occurrences, or more of narrow rows, no per-position segment logic) and
// finished by hot_finish, both in a fixed order.
#include <algorithm>

#include "gba_device.hpp"
#include "gba_internal.hpp"
#include "optim.hpp"
#include "run_heads.hpp"

namespace gba {

constexpr int kSegBlock = 256;
constexpr int kSegWaves = kSegBlock / kWave;                 // 4
constexpr int kRounds = 4;                                   // 16-byte loads per lane and tile in run_heads
constexpr int64_t kMetaTile = (int64_t)kSegBlock * kRounds;  // 1024 positions: 4 per thread of a block
static_assert(kMetaTile == kRunTile, "run-head tiles are the per-position tiles");
constexpr int kGroupSpan = 128;                              // positions per lane group (most; hot_rows)
constexpr int kBatch = 8;                                    // positions per batch of a group
// Row gathers in flight per group: a batch's rows are gathered and summed in
// two parts of four, which leaves the fused row pass 121 VGPRs (4 waves per
// SIMD) instead of 139 (3): more waves in flight beat more loads per wave.
constexpr int kBatchPart = 4;
constexpr int64_t kFineSpanBelow = int64_t(1) << 18;         // positions below which a lane group's span may be 16 or 8
constexpr int64_t kSpanWork = int64_t(1024) * kWave * 32;    // positions * lanes per row of 1024 waves with spans of 32
constexpr int64_t kSpan64From = int64_t(1) << 23;
constexpr int64_t kSpan128From = int64_t(1) << 25;
constexpr int64_t kHotWideFrom = int64_t(1) << 24;           // occurrences from which the hot IDs' spans double
constexpr int kMaxBuckets = 1024;                            // contribution lookup buckets (most)

// packed word of a sorted position
constexpr uint32_t kIndexMask = (1u << 28) - 1u;  // occurrence index j (N < 2^28)
constexpr uint32_t kNonUnit = 1u << 28;           // weight is neither 0 nor 1
constexpr uint32_t kHead = 1u << 29;              // first position of a segment
constexpr uint32_t kNewC = 1u << 30;              // first occurrence of a contribution in its segment
constexpr uint32_t kZeroW = 1u << 31;             // weight 0: the row is never read

enum : uint32_t { kValid = 1, kOpen = 2, kPass = 4 };            // group flags

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

static int lanes_per_row(int D) {
  int l = 1;
  while (l < 64 && l * 4 < D) l <<= 1;
  return l;
}
// Positions per lane group of the cold row pass: 128 for large inputs, fewer
// below, so that a pass over a few million positions still has waves enough
// to keep the memory busy (each group walks its span in batches, one after
// the other).  Below 2^18 positions a span of 32 may leave SIMDs without a
// wave: 16 or 8 then (20,480 positions at D = 16: 40 blocks instead of 10,
// 13.8 us instead of 22).
static int rows_span(int64_t N, int lpr) {
  if (N >= kSpan128From) return 128;
  if (N >= kSpan64From) return 64;
  if (N >= kFineSpanBelow) return 32;
  return N * lpr >= 2 * kSpanWork ? 32 : (N * lpr >= kSpanWork ? 16 : 8);
}
// The same for the hot IDs' pass, whose blocks each sum one chunk (a tile of
// this span) and leave it to hot_finish, one block per ID, to join an ID's
// chunks.  Below 2^25 occurrences chunks of 128 per group would leave less
// than a round of blocks for the chip, but wide rows have few groups per
// block: chunks below some 1000 occurrences cost more in the joining than they
// give the pass.  So 32 per group up to 8 lanes per row, 64 with 16 and 128 with
// more, and twice that from 2^24 with 8 lanes or more.  The means of two skews
// with 32 / 64 / 128 per group, us: D = 16, 4.3 M 283 292 321 and 266 267 323; D
// = 32, 4.3 M 319 319 346 and 308 323 347, 20 M 874 862 872 and 786 759 786; D =
// 64, 6.5 M 564 548 564 and 535 501 523, 20 M 1374 1310 1298 and 1245 1128 1117;
// D = 128, 4.3 M 707 657 639 and 710 617 607; D = 256, 4.3 M 1392 1179 1082 and
// 1546 1181 1021.  From 2^25 half of 128 takes from the pass what the joining of
// twice the chunks costs (D = 32, 65.5 M: pass and joining 783 + 20, 770 + 32).
// Below the sizes that choose hot IDs by themselves 128 keeps the scratch small.
static int hot_span(int64_t N, int lpr) {
  if (N >= kSpan128From || N < kHotPlanFrom) return kGroupSpan;
  const int span = lpr <= 8 ? 32 : (lpr == 16 ? 64 : 128);
  return N >= kHotWideFrom && lpr >= 8 ? std::min(2 * span, kGroupSpan) : span;
}
// The segment count is kept at the start of every group, and every 32
// positions of larger ones.
static int base_shift(int span) { return span >= 32 ? 5 : (span == 16 ? 4 : 3); }
// positions per row-pass tile: 4 waves x (64 / LPR) groups x span positions
static int64_t rows_tile(int lpr, int span) { return (int64_t)kSegWaves * (kWave / lpr) * span; }

// Bucket width 2^q so that at most kMaxBuckets buckets cover [0, N).  Below
// 2^18 positions, where loading the table is a good part of a block's time,
// a few buckets per contribution (64 at least) do.
static int bucket_shift(int64_t N, int32_t K) {
  int64_t most = N < kFineSpanBelow ? 64 : kMaxBuckets;
  while (most < kMaxBuckets && most < 4 * (int64_t)K) most <<= 1;
  int q = 0;
  while (((N - 1) >> q) >= most) ++q;
  return q;
}

struct SegPartials {
  double* first_acc;   // [tiles][D] chain that began in an earlier tile
  double* last_acc;    // [tiles][D] chain that continues into the next tile
  int32_t* first_cc;
  int32_t* first_ww;
  int32_t* last_cc;
  int32_t* last_ww;
  u32x4* fix_list;       // per tile whose last chain continues into the next
                         // tile: (tile, segment, last tile of the segment, 0)
  uint32_t* fix_count;   // entries of fix_list (cleared before the row pass)
};

constexpr int kHotSlots = 256;   // at least the sort's largest number of hot IDs (+1)
constexpr int kRecipMax = 256;   // divisors with a reciprocal in the row pass's table

struct SegLayout {
  int64_t meta_tiles, row_tiles, hot_chunks;
  int span, hot_span;    // positions per lane group of the row pass and of the hot IDs' pass
  size_t off_heads, off_buckets, off_packed, off_base, off_cnt, off_first_acc, off_last_acc, off_fix, off_start,
      off_cnum, off_hot_acc, off_hot_cnt, bytes;
};

static SegLayout seg_layout(int64_t N, int32_t D) {
  SegLayout L{};
  const int lpr = lanes_per_row(D);
  L.span = rows_span(N, lpr);
  L.meta_tiles = N > 0 ? ceil_div(N, kMetaTile) : 1;
  L.row_tiles = N > 0 ? ceil_div(N, rows_tile(lpr, L.span)) : 1;
  const size_t mt = (size_t)L.meta_tiles, rt = (size_t)L.row_tiles;
  const size_t n = (size_t)(N > 0 ? N : 1);
  size_t o = 0;
  L.off_heads = o;     o += align_up(mt * 4);
  L.off_buckets = o;   o += align_up(kMaxBuckets * 4);
  L.off_packed = o;    o += align_up((n + kGroupSpan) * 4);   // padded: whole-group vector loads stay inside
  L.off_base = o;      o += align_up(((n >> base_shift(L.span)) + 2) * 4);
  L.off_cnt = o;       o += align_up(rt * 16);
  L.off_fix = o;       o += 256 + align_up(rt * 16);  // count, then the list
  L.off_first_acc = o; o += align_up(rt * (size_t)D * 8);
  L.off_last_acc = o;  o += align_up(rt * (size_t)D * 8);
  // the position where each (cold) segment starts, and its end
  L.off_start = o;     o += align_up((n + 1) * 4);
  // per hot ID: the cold segments below it, the chunk prefix of its run, and
  // the cold positions below it
  L.off_cnum = o;      o += align_up(3 * (kHotSlots + 1) * 4);
  // per chunk of a hot run: float64 sums and (contributions, active, first and last contribution)
  L.hot_span = hot_span(N, lpr);
  L.hot_chunks = (N > 0 ? ceil_div(N, rows_tile(lpr, L.hot_span)) : 1) + kHotSlots;
  // (the run-head groups' counts lie here too: they are last read by the
  // position pass, before the hot sums are written; hot_chunks * D * 8 is at
  // least N / 1024 + 8192 bytes, the groups take at most N / 4096 + 4096)
  L.off_hot_acc = o;   o += align_up((size_t)L.hot_chunks * D * 8);
  L.off_hot_cnt = o;   o += align_up((size_t)L.hot_chunks * 16);
  L.bytes = o;
  return L;
}

// Where a lane group's span grows with N, the partial sums of the tiles
// shrink: the most of any size up to N, so that a workspace for N positions
// holds every smaller input too.
size_t segments_workspace_bytes(int64_t N, int32_t D) {
  const int lpr = lanes_per_row(D);
  size_t most = seg_layout(N, D).bytes;
  for (const int64_t from : {kSpanWork / lpr, 2 * kSpanWork / lpr, kFineSpanBelow, kSpan64From, kHotWideFrom, kSpan128From})
    if (from <= N) most = std::max(most, seg_layout(from - 1, D).bytes);
  return most;
}

// ------------------------------------------------------------------ helpers
// First index in [lo, hi) whose offset exceeds j, or hi (off non-decreasing).
__device__ __forceinline__ int count_le(const int32_t* off, int lo, int hi, uint32_t j) {
  int len = hi - lo;
  while (len > 0) {
    const int half = len >> 1;
    if ((uint32_t)off[lo + half] <= j) {
      lo += half + 1;
      len -= half + 1;
    } else {
      len = half;
    }
  }
  return lo;
}

// Entries of the ascending s[0, n) that are at most x (n <= 256): a fixed
// sequence of halving steps, with no loop for the compiler to keep registers
// live across.
__device__ __forceinline__ uint32_t count_at_most(const uint32_t* s, uint32_t n, int64_t x) {
  uint32_t pos = 0;
#pragma unroll
  for (uint32_t step = 128; step >= 1; step >>= 1) {
    const uint32_t next = pos + step;
    if (next <= n && (int64_t)s[next - 1] <= x) pos = next;
  }
  return pos;
}

// Hot IDs below `key` (split plan): the sort's bucket table narrows the
// search to the hot IDs that share the key's top bits, then halving.
__device__ __forceinline__ uint32_t hot_below(uint32_t key, const uint16_t* bucket, const uint32_t* ids, uint32_t H,
                                              int bshift) {
  const uint32_t t = key >> bshift;
  uint32_t lo = bucket[t];
  uint32_t hi = t + 1 < 1024u ? (uint32_t)bucket[t + 1] : H;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (ids[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Contribution m of occurrence j (off[m] <= j < off[m+1]): start from the
// bucket table, step past at most one boundary, else search the rest.
__device__ __forceinline__ int contribution_of(const int32_t* s_off, const int32_t* s_bucket, int q,
                                               int K, uint32_t j) {
  int m = s_bucket[j >> q];
  if ((uint32_t)s_off[m + 1] <= j) {
    ++m;
    // first index past m + 1 whose offset exceeds j, minus one
    if ((uint32_t)s_off[m + 1] <= j) m = count_le(s_off, m + 1, K, j) - 1;
  }
  return m < K ? m : K - 1;
}

// Row accesses through the caches or past them.
template <bool CACHED>
__device__ __forceinline__ f32x4 load_row(const f32x4* p) { return CACHED ? *p : load_stream(p); }
template <bool CACHED>
__device__ __forceinline__ void store_row(f32x4* p, f32x4 v) {
  if (CACHED) *p = v;
  else store_stream(p, v);
}

// The optimiser on one lane's 4 floats of a row (mode 1 Adagrad, 2 Adam), with
// the row apply's arithmetic.
__device__ __forceinline__ void update4(int mode, const OptF32& c, f32x4& pv, f32x4& s1, f32x4& s2, f32x4 g) {
  float pe[4] = {pv.x, pv.y, pv.z, pv.w}, ae[4] = {s1.x, s1.y, s1.z, s1.w}, ve[4] = {s2.x, s2.y, s2.z, s2.w};
  const float ge[4] = {g.x, g.y, g.z, g.w};
  if (mode == 2) {
#pragma unroll
    for (int e = 0; e < 4; ++e) adam_update_f32(pe[e], ae[e], ve[e], ge[e], c);
    s2 = f32x4{ve[0], ve[1], ve[2], ve[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) adagrad_update_f32(pe[e], ae[e], ge[e], c);
  }
  pv = f32x4{pe[0], pe[1], pe[2], pe[3]};
  s1 = f32x4{ae[0], ae[1], ae[2], ae[3]};
}

// Row r updated with mean g (one lane's 16 bytes): load, update, store.
__device__ __forceinline__ void apply_row_part(const RowApply& ap, int mode, int64_t r, int D, int lane, f32x4 g) {
  const int64_t at = r * D + lane * 4;
  f32x4 pv = load_stream(reinterpret_cast<const f32x4*>(ap.p + at));
  f32x4 s1 = load_stream(reinterpret_cast<const f32x4*>(ap.s1 + at));
  f32x4 s2 = mode == 2 ? load_stream(reinterpret_cast<const f32x4*>(ap.s2 + at)) : f32x4{0.f, 0.f, 0.f, 0.f};
  update4(mode, ap.c, pv, s1, s2, g);
  store_stream(reinterpret_cast<f32x4*>(ap.p + at), pv);
  store_stream(reinterpret_cast<f32x4*>(ap.s1 + at), s1);
  if (mode == 2) store_stream(reinterpret_cast<f32x4*>(ap.s2 + at), s2);
}

// out: the segment's place among all distinct IDs.  The mean goes to agg
// (when given) and, with a fused apply (mode 1 Adagrad, 2 Adam; a constant in
// the row pass), into the optimiser update of row `row`, or where row < 0 of
// the ID the position pass wrote for this place (written by an earlier
// launch); that row's tag then carries the step (per-ID decay: every tag of
// this call was read by an earlier launch, or is the hot ID's own).
__device__ __forceinline__ void finalize_segment(const SegmentArgs& a, int64_t seg, f64x4 acc,
                                                 int cc, int ww, int lane, bool lane_on, int mode,
                                                 int64_t row = -1) {
  if (seg < 0 || seg >= a.N) return;   // unreachable when the numbering is consistent
  const double div = (a.norm == GBA_NORM_BY_K) ? (double)a.K : (double)cc;
  const f32x4 g = narrow(div_rounded(acc, div));
  if (lane_on && a.agg)
    store_stream(reinterpret_cast<f32x4*>(a.agg + seg * (int64_t)a.D + lane * 4), g);   // read once, by the apply
  if (mode != 0 && lane_on && ww > 0) {
    const int64_t r = row >= 0 ? row : a.unique_ids[seg];
    if (r >= 0 && r < a.R) {   // always in range when the numbering is consistent
      apply_row_part(a.ap, mode, r, a.D, lane, g);
      if (a.decay == GBA_DECAY_ID_TAG && lane == 0) a.tag[r] = (int32_t)a.step;
    }
  }
  if (lane == 0) {
    a.contrib_count[seg] = cc;
    a.active_count[seg] = ww;
  }
}

// Loads the per-contribution tables every block keeps in LDS: offsets [K+1],
// token weights [K], staleness step - tau [K] and the bucket table [nb].
__device__ __forceinline__ void load_contrib_tables(const SegmentArgs& a, const int32_t* buckets, int nb,
                                                    int32_t* s_off, float* s_w, int32_t* s_sm,
                                                    int32_t* s_bucket) {
  for (int i = threadIdx.x; i <= a.K; i += kSegBlock) {
    int64_t o = a.offsets[i];
    o = o < 0 ? 0 : (o > a.N ? a.N : o);
    s_off[i] = (int32_t)o;
    if (i < a.K) {
      s_w[i] = a.w[i];
      int64_t sm = a.step - a.tokens[i];
      sm = sm < -(1 << 30) ? -(1 << 30) : (sm > (1 << 30) ? (1 << 30) : sm);
      s_sm[i] = (int32_t)sm;
    }
  }
  for (int i = threadIdx.x; i < nb; i += kSegBlock) s_bucket[i] = buckets[i];
}

// The same tables in two halves, for K < 2 * kSegBlock: issue() loads a
// thread's entries into registers with clamped indices (no branch, so the
// caller can issue more loads before any is waited for) and store() writes
// them to LDS.
struct ContribTableRegs {
  static constexpr int kR = 2;                            // K + 1 <= 2 * kSegBlock entries
  static constexpr int kB = kMaxBuckets / kSegBlock;      // bucket entries per thread
  int64_t off[kR], tok[kR];
  float w[kR];
  int32_t bucket[kB];

  __device__ __forceinline__ void issue(const SegmentArgs& a, const int32_t* buckets, int nb) {
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int i = threadIdx.x + r * kSegBlock;
      off[r] = a.offsets[i <= a.K ? i : a.K];
      w[r] = a.w[i < a.K ? i : a.K - 1];
      tok[r] = a.tokens[i < a.K ? i : a.K - 1];
    }
#pragma unroll
    for (int r = 0; r < kB; ++r) {
      const int i = threadIdx.x + r * kSegBlock;
      bucket[r] = buckets[i < nb ? i : nb - 1];
    }
  }
  __device__ __forceinline__ void store(const SegmentArgs& a, int nb, int32_t* s_off, float* s_w, int32_t* s_sm,
                                        int32_t* s_bucket) const {
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int i = threadIdx.x + r * kSegBlock;
      if (i <= a.K) {
        const int64_t o = off[r] < 0 ? 0 : (off[r] > a.N ? a.N : off[r]);
        s_off[i] = (int32_t)o;
      }
      if (i < a.K) {
        s_w[i] = w[r];
        int64_t sm = a.step - tok[r];
        sm = sm < -(1 << 30) ? -(1 << 30) : (sm > (1 << 30) ? (1 << 30) : sm);
        s_sm[i] = (int32_t)sm;
      }
    }
#pragma unroll
    for (int r = 0; r < kB; ++r) {
      const int i = threadIdx.x + r * kSegBlock;
      if (i < nb) s_bucket[i] = bucket[r];
    }
  }
};
static_assert(kMaxBuckets % kSegBlock == 0, "whole bucket rounds");

// ------------------------------------------------------------------ kernels
// What the last block of run_heads does beside the run heads for the segment
// passes (all null / zero for a caller that needs the heads only): checks the
// contribution offsets, builds the contribution lookup buckets and clears the
// row pass's fixup count.
struct HeadsPrep {
  const int64_t* off = nullptr;   // [K + 1]
  int32_t* bucket = nullptr;      // [nb] contribution of occurrence b << q
  uint32_t* fix_count = nullptr;
  int32_t* err = nullptr;
  int64_t N = 0;                  // occurrences
  int K = 0, q = 0, nb = 0;
};

// An offset of contribution_of's table: clamped into [0, N].
__device__ __forceinline__ int32_t clamp_offset(int64_t o, int64_t N) {
  return (int32_t)(o < 0 ? 0 : (o > N ? N : o));
}

__device__ __forceinline__ void heads_prep(const HeadsPrep& pr, int32_t* s_off) {
  bool bad = false;
  for (int m = threadIdx.x; m <= pr.K; m += (int)blockDim.x) {
    const int64_t o = pr.off[m];
    bad |= (m == 0 && o != 0) || (m == pr.K && o != pr.N) || (m < pr.K && o > pr.off[m + 1]);
    s_off[m] = clamp_offset(o, pr.N);
  }
  if (bad) raise_error(pr.err, GBA_DERR_OFFSETS);
  if (threadIdx.x == 0) *pr.fix_count = 0u;   // the row pass appends to the fixup list
  __syncthreads();
  for (int b = threadIdx.x; b < pr.nb; b += (int)blockDim.x) {
    const int m = count_le(s_off, 1, pr.K, (uint32_t)b << pr.q) - 1;
    pr.bucket[b] = m < pr.K ? m : pr.K - 1;
  }
}

// Run heads: a block takes a group of WAVES consecutive 1024-position tiles,
// one per wave, and writes the heads before each tile inside its group and
// the group's total.  Lane l holds positions t0 + 4 (l + 64 c) + e (c, e <
// 4): each 16-byte load of the wave covers 1 KB of consecutive keys, and the
// key before a lane's first one is the last key of the lane before.  The last
// block of a launch with PREP does heads_prep instead.
template <int WAVES, bool PREP>
__global__ void __launch_bounds__(WAVES * kWave)
run_heads_kernel(const uint32_t* __restrict__ keys, int64_t N_arg, const uint32_t* __restrict__ n_dev, int64_t tiles,
                 uint32_t* __restrict__ tile_prefix, uint32_t* __restrict__ group_count, HeadsPrep prep) {
  __shared__ uint32_t s_cnt[WAVES];
  __shared__ int32_t s_off[PREP ? GBA_MAX_K + 1 : 1];
  if (PREP && blockIdx.x == gridDim.x - 1) {
    heads_prep(prep, s_off);
    return;
  }
  const int lane = lane_id();
  const int w = threadIdx.x / kWave;
  const int64_t tile = (int64_t)blockIdx.x * WAVES + w;
  const int64_t N = n_dev ? (int64_t)*n_dev : N_arg;   // the grid is sized for the most keys
  const int64_t t0 = tile * kMetaTile;
  uint32_t cnt = 0;
  if (t0 < N) {   // the same for the whole wave
    uint32_t carry = t0 > 0 ? keys[t0 - 1] : 0u;   // position 0 is always a head
#pragma unroll
    for (int c = 0; c < kRounds; ++c) {
      const int64_t i0 = t0 + 4 * ((int64_t)lane + (int64_t)kWave * c);
      uint32_t k[4] = {0u, 0u, 0u, 0u};
      if (i0 + 3 < N) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(keys + i0);
        k[0] = v.x; k[1] = v.y; k[2] = v.z; k[3] = v.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) k[e] = (i0 + e < N) ? keys[i0 + e] : 0u;
      }
      uint32_t prev = __shfl_up(k[3], 1, kWave);
      if (lane == 0) prev = carry;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t p = i0 + e;
        if (p < N) cnt += (p == 0 || k[e] != prev) ? 1u : 0u;
        prev = k[e];
      }
      carry = __shfl(k[3], kWave - 1, kWave);
    }
    cnt = wave_sum(cnt);
  }
  if (lane == 0) s_cnt[w] = cnt;
  __syncthreads();
  if (threadIdx.x < WAVES) {
    uint32_t before = 0;
    for (int k = 0; k < (int)threadIdx.x; ++k) before += s_cnt[k];
    if ((int64_t)blockIdx.x * WAVES + threadIdx.x < tiles) tile_prefix[(int64_t)blockIdx.x * WAVES + threadIdx.x] = before;
    if (threadIdx.x == WAVES - 1) group_count[blockIdx.x] = before + s_cnt[WAVES - 1];
  }
}

// Exclusive scan of the group counts in place, one block: thread t owns
// kRunScanItems consecutive groups (four 16-byte loads).
constexpr int kRunScanBlock = 1024;
constexpr int kRunScanItems = 16;
__global__ void __launch_bounds__(kRunScanBlock)
run_group_scan_kernel(uint32_t* __restrict__ group, int groups) {
  __shared__ uint32_t tmp[kRunScanBlock / kWave + 1];
  const int g0 = threadIdx.x * kRunScanItems;
  uint32_t v[kRunScanItems], sum = 0;
#pragma unroll
  for (int k = 0; k < kRunScanItems; ++k) v[k] = g0 + k < groups ? group[g0 + k] : 0u;
#pragma unroll
  for (int k = 0; k < kRunScanItems; ++k) sum += v[k];
  uint32_t total;
  uint32_t run = block_exclusive_scan<kRunScanBlock>(sum, tmp, &total);
#pragma unroll
  for (int k = 0; k < kRunScanItems; ++k) {
    if (g0 + k < groups) group[g0 + k] = run;
    run += v[k];
  }
}

// No occurrences: no segments.
__global__ void __launch_bounds__(kSegBlock)
seg_empty_kernel(const int64_t* __restrict__ off, int K, int64_t* __restrict__ num_unique,
                 int64_t* __restrict__ seg_offsets, int32_t* __restrict__ err) {
  bool bad = false;
  for (int m = threadIdx.x; m <= K; m += kSegBlock) bad |= off[m] != 0;
  if (bad) raise_error(err, GBA_DERR_OFFSETS);
  if (threadIdx.x == 0) {
    *num_unique = 0;
    seg_offsets[0] = 0;
  }
}

// Per-position pass: numbering, segment IDs and starts, packed words.
// TPB consecutive 1024-position tiles per block; in a tile each lane takes 4
// consecutive positions (16-byte loads and stores), and the segment numbers
// come from a scan of the lanes' head counts, from the heads before the tile
// in its group and before the group (run_base).  The lane that holds the last
// position also writes U, the end of the last segment and the places of the
// hot IDs above every cold key.
constexpr int kMetaPer = 4;   // consecutive positions per lane
static_assert(kSegBlock * kMetaPer == kMetaTile, "a block covers one tile per pass");
template <int TPB>
__global__ void __launch_bounds__(kSegBlock)
seg_meta_kernel(SegmentArgs a, RunHeads heads, const int32_t* __restrict__ buckets, int q, int nbuckets,
                int64_t num_tiles, uint32_t* __restrict__ packed, uint32_t* __restrict__ base, int bshift,
                uint32_t* __restrict__ seg_start, uint32_t* __restrict__ cnum, uint32_t* __restrict__ cold_below) {
  constexpr int kMetaTilesPerBlock = TPB;
  extern __shared__ int32_t s_dyn[];
  __shared__ uint32_t s_wave_heads[kSegWaves];
  __shared__ uint32_t s_group[kSegWaves];
  // split plan: the hot IDs, their buckets and the hot occurrences below each
  __shared__ uint32_t s_hbucket[512];
  __shared__ uint32_t s_hids[kHotSlots];
  __shared__ uint32_t s_hprefix[kHotSlots];
  const int K = a.K;
  const int64_t N = a.N;                                        // occurrences
  const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.N;          // sorted positions (the cold ones when split)
  const bool split = a.n_dev != nullptr;
  int32_t* s_off = s_dyn;
  float* s_w = reinterpret_cast<float*>(s_dyn + K + 1);
  int32_t* s_sm = s_dyn + 2 * K + 1;
  int32_t* s_bucket = s_dyn + 3 * K + 1;
  // The lookup tables' loads are issued first (branch-free when K is below
  // 512), then, when every position of the block exists, all loads of its
  // tiles, so that the tables are waited for while the tiles are in flight.
  const int64_t blk0 = (int64_t)blockIdx.x * kMetaTilesPerBlock * kMetaTile;
  if (blk0 >= n) {   // the grid is sized for every occurrence
    if (n == 0 && blockIdx.x == 0) {   // every occurrence is a hot ID's
      const uint32_t hots = *a.hot.meta;
      for (uint32_t h = threadIdx.x; h < hots; h += kSegBlock) {
        cnum[h] = 0u;
        cold_below[h] = 0u;
      }
      if (threadIdx.x == 0) {
        *a.num_unique = (int64_t)hots;
        a.seg_offsets[hots] = N;
        seg_start[0] = 0u;
      }
    }
    return;
  }
  const bool full = blk0 + kMetaTilesPerBlock * kMetaTile <= n;
  uint32_t H = 0;
  if (split) {
    H = *a.hot.meta;
    const uint32_t* b32 = reinterpret_cast<const uint32_t*>(a.hot.bucket);
    for (int i = threadIdx.x; i < 512; i += kSegBlock) s_hbucket[i] = b32[i];
    s_hids[threadIdx.x] = a.hot.ids[threadIdx.x];
    s_hprefix[threadIdx.x] = a.hot.prefix[threadIdx.x];
  }
  const uint16_t* hbucket = reinterpret_cast<const uint16_t*>(s_hbucket);
  const bool small_k = K < ContribTableRegs::kR * kSegBlock;
  ContribTableRegs tables;
  if (small_k) tables.issue(a, buckets, nbuckets);
  // Loaded unconditionally (a branch would make the compiler wait for them
  // where its paths join): a block that is not full clamps its indices into
  // the arrays (the key and value arrays are padded to 64 entries, so a
  // 16-byte load at the last multiple of 4 below N stays inside them) and
  // uses none of these values.
  u32x4 kv[kMetaTilesPerBlock], vv[kMetaTilesPerBlock];
  uint32_t kpv[kMetaTilesPerBlock], jpv[kMetaTilesPerBlock], sb[kMetaTilesPerBlock];
  {
    const int64_t last4 = (n - 1) & ~int64_t(kMetaPer - 1);
#pragma unroll
    for (int kt = 0; kt < kMetaTilesPerBlock; ++kt) {
      int64_t p0 = blk0 + kt * kMetaTile + (int64_t)threadIdx.x * kMetaPer;
      p0 = p0 < last4 ? p0 : last4;
      kv[kt] = *reinterpret_cast<const u32x4*>(a.keys + p0);
      vv[kt] = *reinterpret_cast<const u32x4*>(a.vals + p0);
      const int64_t pp = p0 > 0 ? p0 - 1 : 0;   // used by lane 0 only, when p0 > 0
      kpv[kt] = a.keys[pp];
      jpv[kt] = a.vals[pp];
      int64_t t = (int64_t)blockIdx.x * kMetaTilesPerBlock + kt;
      sb[kt] = heads.tile_prefix[t < num_tiles ? t : num_tiles - 1];
    }
  }
  if (small_k)
    tables.store(a, nbuckets, s_off, s_w, s_sm, s_bucket);
  else
    load_contrib_tables(a, buckets, nbuckets, s_off, s_w, s_sm, s_bucket);
  run_base(heads, (int64_t)blockIdx.x * kMetaTilesPerBlock, s_group);
  __syncthreads();
  const uint32_t group_base = run_base_sum(s_group);

  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  // One tile: key/jv are this lane's 4 positions from p0, kprev/jprev the
  // position before p0 (when p0 > 0), seg_base the segments before the tile.
  auto tile_body = [&](int64_t p0, const uint32_t* key, const uint32_t* jv, uint32_t kprev, uint32_t jprev,
                       uint32_t seg_base) {
    int m[kMetaPer];
#pragma unroll
    for (int e = 0; e < kMetaPer; ++e)
      m[e] = (p0 + e < n && (int64_t)jv[e] < N) ? contribution_of(s_off, s_bucket, q, K, jv[e]) : 0;
    // the position before this lane's first: the previous lane's last, or
    // (first lane of a wave) the one loaded for it
    uint32_t kp = __shfl_up(key[kMetaPer - 1], 1, kWave);
    int mp = __shfl_up(m[kMetaPer - 1], 1, kWave);
    bool prev_ok = true;
    if (lane == 0) {
      prev_ok = p0 > 0 && p0 - 1 < n;
      if (prev_ok) {
        kp = kprev;
        mp = (int64_t)jprev < N ? contribution_of(s_off, s_bucket, q, K, jprev) : 0;
      }
    }
    uint32_t word[kMetaPer];
    float weight[kMetaPer];
    bool any_nonunit = false;
    uint32_t nheads = 0, head_bits = 0;
#pragma unroll
    for (int e = 0; e < kMetaPer; ++e) {
      const bool valid = p0 + e < n;
      const bool head = valid && (e == 0 ? (!prev_ok || key[0] != kp) : key[e] != key[e - 1]);
      const bool newc = valid && (head || m[e] != (e == 0 ? mp : m[e - 1]));
      float wt = 0.0f;
      if (valid) {
        if (a.decay == GBA_DECAY_TOKEN) {
          wt = s_w[m[e]];
        } else {
          const int64_t tg = ((int64_t)key[e] < a.R) ? (int64_t)a.tag[key[e]] : -1;
          int64_t st = tg - a.step + (int64_t)s_sm[m[e]] + 1;
          st = st < 0 ? 0 : st;
          wt = (st <= a.iota) ? 1.0f : 0.0f;
        }
      }
      word[e] = (jv[e] & kIndexMask) | (head ? kHead : 0u) | (newc ? kNewC : 0u) |
                (wt == 0.0f ? kZeroW : 0u) | ((wt != 0.0f && wt != 1.0f) ? kNonUnit : 0u);
      weight[e] = wt;
      any_nonunit |= wt != 0.0f && wt != 1.0f;
      nheads += head ? 1u : 0u;
      head_bits |= head ? (1u << e) : 0u;
    }
    if (p0 + kMetaPer - 1 < n) {
      *reinterpret_cast<u32x4*>(packed + p0) = u32x4{word[0], word[1], word[2], word[3]};
    } else {
#pragma unroll
      for (int e = 0; e < kMetaPer; ++e)
        if (p0 + e < n) packed[p0 + e] = word[e];
    }
    if (any_nonunit) {   // the row pass reads weights other than 0 and 1 (the array is padded to 64 entries)
      *reinterpret_cast<f32x4*>(a.weights + p0) = f32x4{weight[0], weight[1], weight[2], weight[3]};
    }
    // segment numbers: the tile's base, the waves before, the lanes before
    const uint32_t incl = wave_inclusive_scan(nheads);
    if (lane == kWave - 1) s_wave_heads[w] = incl;
    __syncthreads();
    uint32_t before = group_base + seg_base + incl - nheads;
    for (int k = 0; k < w; ++k) before += s_wave_heads[k];
    // segments that start before each group-aligned position
    if ((p0 & ((int64_t(1) << bshift) - 1)) == 0 && p0 < n) base[p0 >> bshift] = before;
#pragma unroll
    for (int e = 0; e < kMetaPer; ++e) {
      if ((head_bits >> e) & 1u) {
        // split plan: the hot IDs below this key come before it among all IDs
        // (and their occurrences before its start); those above the key
        // before it (none for position 0) lie between the two segments
        uint32_t below = 0;
        if (split) {
          below = hot_below(key[e], hbucket, s_hids, H, a.hot.bshift);
          const uint32_t kprev = e == 0 ? kp : key[e - 1];
          const uint32_t from = (p0 + e > 0) ? hot_below(kprev, hbucket, s_hids, H, a.hot.bshift) : 0u;
          for (uint32_t h = from; h < below; ++h) {
            cnum[h] = before;
            cold_below[h] = (uint32_t)(p0 + e);
          }
        }
        const int64_t out = (int64_t)before + below;
        if (out < N) {   // always true when the numbering is consistent
          a.unique_ids[out] = (int64_t)key[e];
          a.seg_offsets[out] = p0 + e + (split ? (int64_t)s_hprefix[below] : 0);
          seg_start[before] = (uint32_t)(p0 + e);
        }
        ++before;
      }
    }
    if (p0 < n && p0 + kMetaPer >= n) {   // the last position: before = U
      const int64_t U = before;
      if (U + H <= N) {   // always true when the numbering is consistent
        *a.num_unique = U + H;
        a.seg_offsets[U + H] = N;
        seg_start[U] = (uint32_t)n;
      }
      // hot IDs above every cold key
      if (split)
        for (uint32_t h = hot_below(a.keys[n - 1], hbucket, s_hids, H, a.hot.bshift); h < H; ++h) {
          cnum[h] = (uint32_t)U;
          cold_below[h] = (uint32_t)n;
        }
    }
    __syncthreads();   // s_wave_heads is rewritten by the next tile
  };

  if (full) {
#pragma unroll
    for (int kt = 0; kt < kMetaTilesPerBlock; ++kt) {
      const int64_t p0 = blk0 + kt * kMetaTile + (int64_t)threadIdx.x * kMetaPer;
      const uint32_t key[kMetaPer] = {kv[kt].x, kv[kt].y, kv[kt].z, kv[kt].w};
      const uint32_t jv[kMetaPer] = {vv[kt].x, vv[kt].y, vv[kt].z, vv[kt].w};
      tile_body(p0, key, jv, kpv[kt], jpv[kt], sb[kt]);
    }
    return;
  }
  for (int kt = 0; kt < kMetaTilesPerBlock; ++kt) {
    const int64_t tile = (int64_t)blockIdx.x * kMetaTilesPerBlock + kt;
    if (tile >= num_tiles) break;
    const int64_t p0 = tile * kMetaTile + (int64_t)threadIdx.x * kMetaPer;
    uint32_t key[kMetaPer] = {0u, 0u, 0u, 0u}, jv[kMetaPer] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < kMetaPer; ++e)
      if (p0 + e < n) {
        key[e] = a.keys[p0 + e];
        jv[e] = a.vals[p0 + e];
      }
    uint32_t kprev = 0, jprev = 0;
    if (p0 > 0 && p0 - 1 < n) {
      kprev = a.keys[p0 - 1];
      jprev = a.vals[p0 - 1];
    }
    tile_body(p0, key, jv, kprev, jprev, heads.tile_prefix[tile]);
  }
}

// Per-group pass: gather the kept rows and sum every run in float64.  APPLY
// (1 Adagrad, 2 Adam) updates each finished segment's row in the table as well.
// Each group walks `span` positions (a multiple of kBatch and of 1 << bshift).
//
// A segment that closes is parked in LDS: its mean, place, counts and (with a
// row apply) row go to the next free entry of the wave's ring, numbered by a
// ballot of the closing groups.  When kPop entries wait, the wave writes them
// together, GW rows per store with every lane busy and the table and state
// rows of kR such rounds requested before the first is used; otherwise each
// group would store and update as its segments close while the lanes of the
// other groups idle.  Wide rows that are only stored (two groups per wave or
// one) are written as they close (D = 128, 300,007 positions: 71 us, parked
// 100).  The segments a group closes after its last position go through the
// ring too, so the wave's last updates share two or three memory latencies
// instead of taking two each (20,480 positions at D = 16: 20 -> 17.5 us; 6.5 M
// at D = 32 with Adam 299 -> 291).  Bound: random row accesses, some 34-36 G 128-byte lines a second
// read and written at 16, 32 and 64 floats (a read-only gather reaches 47-50); D = 32
// with Adam, 6.5 M positions, per-ID decay: 303 us for this pass against 144 +
// 183 + 22 for the pass, the row apply and the tags as launches of their own;
// D = 16 with Adam 219 against 104 + 119, D = 64 with Adagrad 137 against 63 +
// 74 (both storing the means too), so every width applies its rows here.
//
// With a row apply, rows below 128 bytes that are not whole 64-byte pieces
// (CACHED) are read and written through the caches, where neighbouring rows
// that share a line meet; all others past them (Adagrad, means kept, us past
// the caches and through them: uniform IDs, D = 20, 3 M positions 515 and 427,
// D = 4, 300,007 158 and 116, D = 28, 4.3 M 858 and 689; Zipf IDs, D = 28, 1.6 M 211
// and 219, 4.3 M 459 and 449; 64-byte rows, uniform, D = 16, 1.6 M 247 and 264, D =
// 48 408 and 475; the means alone, D = 24, 1.6 M 174 and 203).
template <int LPR, int APPLY, bool CACHED>
__global__ void __launch_bounds__(kSegBlock) __attribute__((amdgpu_waves_per_eu(4)))
seg_rows_kernel(SegmentArgs a, const uint32_t* __restrict__ packed, const uint32_t* __restrict__ base, int span,
                int bshift, SegPartials part, const uint32_t* __restrict__ seg_start,
                const uint32_t* __restrict__ cnum) {
  constexpr int GW = kWave / LPR;            // groups per wave
  constexpr int G = kSegWaves * GW;          // groups per block
  const int SPAN = span;
  const int64_t TILE = (int64_t)G * SPAN;
  static_assert(APPLY >= 0 && APPLY <= 2, "none, Adagrad, Adam");
  // rows gathered at a time: the batch in parts of kPart (registers: each
  // lane holds kPart 16-byte row pieces while they are in flight)
  constexpr int kPart = kBatchPart;
  constexpr bool kPark = APPLY != 0 || LPR <= 16;
  // Rounds of rows in flight: what 128 registers and 40 KB of LDS per block
  // (four waves per SIMD) allow.  With one or two lanes per row, where a ring
  // entry is mostly its place, counts and row, the arrays take 51 and 41 KB:
  // three waves.  Chain sums that share the ring would bring two lanes to four
  // waves, but are slower (20,480 Zipf positions, D = 8 55 and 58 us).  Four
  // rounds leave no LDS for chain sums of their own (kOwnAcc): those then share
  // the ring, which has to be emptied once more.  Measured in turn in one
  // process: Adagrad, D = 32, 65.5 M positions 3399 us with four rounds, 3416 with
  // two and sums of their own; D = 64, a step of 852 K 249 and 254; where two rounds
  // are the most either way the sums of their own win (D = 32 with Adam, 6.5 M
  // positions 612 and 618; D = 16, a step of 20,480 56 and 58).
  constexpr bool kOwnAcc = !(APPLY == 1 && LPR >= 8);
  constexpr int kR = LPR <= 4 ? 1 : (kOwnAcc ? 2 : 4);
  constexpr int kPop = kR * GW;
  // a part, or the two segments that a group may close after its last one,
  // adds at most kPart * GW entries to fewer than kPop
  constexpr int kAccSlots = kWave * (int)sizeof(f64x4) / (LPR * (int)sizeof(f32x4));   // entries that hold a wave's chain sums
  constexpr int kSlots = kPark ? kPop + kPart * GW : 1;
  auto ring = [](int x) { return x < kSlots ? x : x - kSlots; };   // x < 2 kSlots
  __shared__ f32x4 s_park[kPark ? kSegWaves : 1][kSlots][LPR];
  __shared__ uint32_t s_park_out[kPark ? kSegWaves : 1][kPark ? kSlots : 1];
  __shared__ uint32_t s_park_cw[kPark ? kSegWaves : 1][kPark ? kSlots : 1];
  __shared__ uint32_t s_park_key[APPLY ? kSegWaves : 1][APPLY ? kSlots : 1];
  // per-lane chain sums at the end of the groups, in their own array or in the
  // last entries of the ring of the lane's own wave, which is empty by then (the
  // segments that the chains close take its first GW entries)
  static_assert(kOwnAcc || GW + kAccSlots <= kSlots, "chain sums beside the last segments");
  __shared__ f64x4 s_acc[kOwnAcc ? kSegBlock : 1];
  auto s_acc_at = [&](int t) -> f64x4& {
    if constexpr (kOwnAcc) return s_acc[t];
    else return reinterpret_cast<f64x4*>(&s_park[t / kWave][kSlots - kAccSlots][0])[t % kWave];
  };
  __shared__ int32_t s_cc[G], s_ww[G];
  __shared__ uint32_t s_seg[G], s_flags[G];
  __shared__ uint32_t s_cnum[kHotSlots];
  // rounded reciprocals of the small divisors (a segment's contribution count)
  __shared__ double s_recip[kRecipMax + 1];
  static_assert(LPR < 4 || sizeof(s_park) + sizeof(s_park_out) + sizeof(s_park_cw) + sizeof(s_park_key) +
                                   sizeof(s_acc) + sizeof(s_cc) + sizeof(s_ww) + sizeof(s_seg) + sizeof(s_flags) +
                                   sizeof(s_cnum) + sizeof(s_recip) <= 40960,
                "four blocks per compute unit");

  const int64_t N = a.N;                                   // occurrences
  const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.N;     // sorted positions
  const int D = a.D;
  if ((int64_t)blockIdx.x * TILE >= n) return;   // the grid is sized for every occurrence
  // split plan: hot ID h comes before cold segment s among all IDs when
  // cnum[h] <= s (cnum ascending)
  const uint32_t H = a.n_dev ? *a.hot.meta : 0u;
  if (threadIdx.x < H) s_cnum[threadIdx.x] = cnum[threadIdx.x];
  for (int i = threadIdx.x; i <= kRecipMax; i += kSegBlock) s_recip[i] = 1.0 / (double)i;
  __syncthreads();
  const bool by_k = a.norm == GBA_NORM_BY_K;
  const double recip_k = 1.0 / (double)a.K;

  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  const int gl = lane % LPR;                 // lane inside its group
  const int grp = w * GW + lane / LPR;       // group inside the block
  const bool lane_on = gl * 4 < D;

  {
    const int64_t tile = blockIdx.x;
    const int64_t p0 = tile * TILE + (int64_t)grp * SPAN;
    const int nvalid = (n - p0) >= SPAN ? SPAN : (n - p0 > 0 ? (int)(n - p0) : 0);
    const uint32_t gbase = nvalid > 0 ? base[p0 >> bshift] : 0u;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    int cc = 0, ww = 0;
    int64_t seg = (int64_t)gbase - 1;
    // hot IDs before segment seg among all IDs (its output is seg + hb)
    uint32_t hb = H ? count_at_most(s_cnum, H, seg) : 0u;
    const uint32_t hb0 = hb;
    // the first segment number that has hot ID hb before it
    uint32_t hnext = hb < H ? s_cnum[hb] : 0xffffffffu;   // positions (and segments) stay below 2^32 - 1
    bool first_open = false;
    bool in_first = true;
    f64x4 facc = {0.0, 0.0, 0.0, 0.0};
    int fcc = 0, fww = 0;
    bool owner = false;
    int parked = 0, first_parked = 0;   // entries of the wave's ring, and its first (the same in every lane)
    const uint32_t key0 = (APPLY && nvalid > 0) ? a.keys[p0] : 0u;
    uint32_t cur_key = key0;   // row of the open segment (row apply)
    auto mean_of = [&](f64x4 sum, int count) {
      const double div = by_k ? (double)a.K : (double)count;
      // counts are at most K unless the offsets are out of order
      const double y = by_k ? recip_k : ((uint32_t)count <= (uint32_t)kRecipMax ? s_recip[count] : 1.0 / div);
      return narrow(div_rounded(sum, div, y));
    };
    // A segment of this group is finished (mc: the lanes of the wave's groups
    // that finish one at the same time; the caller adds them to `parked`).
    auto park = [&](uint64_t mc, f32x4 g, int64_t out, int count, int active, uint32_t key) {
      if (kPark) {
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(mc >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mc, 0u));
        const int slot = ring(ring(first_parked + parked) + (int)(below / LPR));
        if (lane_on) s_park[w][slot][gl] = g;
        if (gl == 0) {
          s_park_out[w][slot] = (uint32_t)out;
          s_park_cw[w][slot] = (uint32_t)count | ((uint32_t)active << 16);
          if (APPLY) s_park_key[w][slot] = key;
        }
      } else if (out >= 0 && out < N) {   // always true when the numbering is consistent
        if (lane_on) store_stream(reinterpret_cast<f32x4*>(a.agg + out * D + gl * 4), g);
        if (gl == 0) {
          a.contrib_count[out] = count;
          a.active_count[out] = active;
        }
      }
    };
    // Words of the batch at i0 (the packed array is padded by a group span, so
    // whole vectors stay in bounds past the group's end).
    auto load_words = [&](int i0, uint32_t (&word)[kBatch]) {
      // a group past its positions (waves loop to their longest group) reads the first words, ignored
      const u32x4* wp = reinterpret_cast<const u32x4*>(packed + (i0 < nvalid ? p0 + i0 : 0));
#pragma unroll
      for (int v = 0; v < kBatch / 4; ++v) {
        const u32x4 x = wp[v];
        word[4 * v] = x.x; word[4 * v + 1] = x.y; word[4 * v + 2] = x.z; word[4 * v + 3] = x.w;
      }
    };
    // Keys of the batch at i0, for the row apply (zero past the sorted positions).
    auto load_keys = [&](int i0, uint32_t (&kk)[kBatch]) {
      const int64_t pk = (i0 < nvalid) ? p0 + i0 : 0;
      if (pk + kBatch <= n) {
        const u32x4* kp = reinterpret_cast<const u32x4*>(a.keys + pk);
#pragma unroll
        for (int v = 0; v < kBatch / 4; ++v) {
          const u32x4 x = kp[v];
          kk[4 * v] = x.x; kk[4 * v + 1] = x.y; kk[4 * v + 2] = x.z; kk[4 * v + 3] = x.w;
        }
      } else {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) kk[u] = (pk + u < n) ? a.keys[pk + u] : 0u;
      }
    };
    // Every lane issues all of a batch's gathers: one whose row is not needed
    // (past the group, a zero weight, a lane past D) reads the first 16
    // bytes of the rows, which stay in cache, and is zeroed when summed.  With
    // no load inside a branch, the compiler can count the loads in flight and
    // never waits for all of them at once.
    // rows u0 .. u0 + kPart - 1 of the batch into rv[0 .. kPart)
    auto gather = [&](int i0, int u0, const uint32_t (&word)[kBatch], f32x4 (&rv)[kPart], uint32_t& use) {
#pragma unroll
      for (int v = 0; v < kPart; ++v) {
        const int u = u0 + v;
        const uint32_t jv = word[u] & kIndexMask;
        const bool on = i0 + u < nvalid && !(word[u] & kZeroW) && lane_on && (int64_t)jv < N;
        use |= on ? (1u << u) : 0u;
        rv[v] = *reinterpret_cast<const f32x4*>(a.rows + (on ? (int64_t)jv * D + gl * 4 : 0));
      }
    };
    // positions u0 .. u0 + kPart - 1 of the batch, their rows in rv[0 .. kPart)
    auto sum_batch = [&](int i0, int u0, const uint32_t (&word)[kBatch], const uint32_t (&kk)[kBatch],
                         f32x4 (&rv)[kPart], uint32_t use, bool weighted, f32x4 wv) {
#pragma unroll
      for (int v = 0; v < kPart; ++v)
        if (!((use >> (u0 + v)) & 1u)) rv[v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < kPart; ++v) {
        const int u = u0 + v;
        const int i = i0 + u;
        // keep each row's float64 widening next to its use: hoisting all of
        // them costs registers and the waves that keep gathers in flight
        __builtin_amdgcn_sched_barrier(0);
        // groups whose open segment ends before this position, apart from one that began before the group
        const bool head = i < nvalid && (word[u] & kHead);
        const bool closes = head && i > 0 && !(in_first && first_open);
        const uint64_t mc = kPark ? __ballot(closes) : 0ull;
        if (i < nvalid) {
          if (head) {
            if (i > 0) {
              if (!closes) {
                facc = acc; fcc = cc; fww = ww; owner = true;
              } else {
                park(mc, mean_of(acc, cc), seg + hb, cc, ww, cur_key);
              }
              in_first = false;
            }
            ++seg;
            if (APPLY) cur_key = kk[u];
            if ((uint32_t)seg >= hnext) {
              do ++hb; while (hb < H && (int64_t)s_cnum[hb] <= seg);
              hnext = hb < H ? s_cnum[hb] : 0xffffffffu;
            }
            acc = f64x4{0.0, 0.0, 0.0, 0.0};
            cc = ww = 0;
          }
          const bool zero = word[u] & kZeroW;
          if (!weighted) {
            acc += widen(rv[v]);
          } else if (!zero) {
            const double wd = (word[u] & kNonUnit) ? (double)wv[v] : 1.0;
            acc = fma_widen(wd, rv[v], acc);
          }
          const int nc = (word[u] & kNewC) ? 1 : 0;
          cc += nc;
          ww += (nc && !zero) ? 1 : 0;
        }
        parked += __popcll(mc) / LPR;
      }
    };
    // The first `count` (at most kPop) parked segments, written by the whole
    // wave: the group of lane / LPR takes entries lane / LPR + GW r.
    auto pop = [&](int count) {
      __builtin_amdgcn_wave_barrier();
      f32x4 pv[kR], sv[kR], vv[kR];
      int slot[kR];
      int64_t outv[kR], row[kR];
      bool act[kR];
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        const int e = r * GW + lane / LPR;
        slot[r] = ring(first_parked + e);
        outv[r] = e < count ? (int64_t)s_park_out[w][slot[r]] : N;   // out < N when the numbering is consistent
        if (APPLY) {
          // sorted keys are below R; a lane without a row reads the table's first 16 bytes and writes nothing
          const uint32_t k = s_park_key[w][slot[r]];
          act[r] = outv[r] < N && (s_park_cw[w][slot[r]] >> 16) > 0 && lane_on && (int64_t)k < a.R;
          row[r] = act[r] ? (int64_t)k : 0;
          const int64_t at = act[r] ? row[r] * D + gl * 4 : 0;
          pv[r] = load_row<CACHED>(reinterpret_cast<const f32x4*>(a.ap.p + at));
          sv[r] = load_row<CACHED>(reinterpret_cast<const f32x4*>(a.ap.s1 + at));
          if (APPLY == 2) vv[r] = load_row<CACHED>(reinterpret_cast<const f32x4*>(a.ap.s2 + at));
        }
      }
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        if (outv[r] >= N) continue;
        const f32x4 g = s_park[w][slot[r]][gl];
        if (lane_on && (!APPLY || a.agg)) store_row<CACHED>(reinterpret_cast<f32x4*>(a.agg + outv[r] * D + gl * 4), g);
        if (gl == 0) {
          const uint32_t v = s_park_cw[w][slot[r]];
          a.contrib_count[outv[r]] = (int32_t)(v & 0xffffu);
          a.active_count[outv[r]] = (int32_t)(v >> 16);
          // the tags of this call were read by the position pass
          if (APPLY && a.decay == GBA_DECAY_ID_TAG && act[r]) a.tag[row[r]] = (int32_t)a.step;
        }
        if (APPLY && act[r]) {
          const int64_t at = row[r] * D + gl * 4;
          update4(APPLY, a.ap.c, pv[r], sv[r], vv[r], g);
          store_row<CACHED>(reinterpret_cast<f32x4*>(a.ap.p + at), pv[r]);
          store_row<CACHED>(reinterpret_cast<f32x4*>(a.ap.s1 + at), sv[r]);
          if (APPLY == 2) store_row<CACHED>(reinterpret_cast<f32x4*>(a.ap.s2 + at), vv[r]);
        }
      }
      first_parked = ring(first_parked + count);
      parked -= count;
      __builtin_amdgcn_wave_barrier();   // the entries are reused from here
    };
    // every group of a wave runs the wave's longest group's batches, so that
    // the whole wave takes part in every ballot and pop
    int iters = nvalid;
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      const int o = __shfl_xor(iters, off, kWave);
      iters = o > iters ? o : iters;
    }
    for (int i0 = 0; i0 < iters; i0 += kBatch) {
      uint32_t word[kBatch], kk[kBatch];
      load_words(i0, word);
      if (APPLY) load_keys(i0, kk);
      if (i0 == 0) first_open = !(word[0] & kHead);
      // unless some position of the wave's batch has a weight other than 0
      // and 1, rows are added without a multiply (a weight-0 row is zeroed),
      // a branch the whole wave takes together; such weights are read from
      // where the position pass left them (a search of the offsets in global
      // memory per position before: D = 128, 300,007 positions of fractional
      // weights 71 us, now 40)
      bool nonunit = false;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) nonunit |= i0 + u < nvalid && (word[u] & kNonUnit);
      const bool weighted = __ballot(nonunit) != 0ull;
      uint32_t use = 0;
#pragma unroll
      for (int u0 = 0; u0 < kBatch; u0 += kPart) {
        f32x4 rv[kPart];
        f32x4 wv = {1.f, 1.f, 1.f, 1.f};
        if (weighted) wv = *reinterpret_cast<const f32x4*>(a.weights + (i0 < nvalid ? p0 + i0 + u0 : 0));
        gather(i0, u0, word, rv, use);
        sum_batch(i0, u0, word, kk, rv, use, weighted, wv);
        if (kPark)
          while (parked >= kPop) pop(kPop);
      }
    }

    bool last_open = false, pass = false, last_closes = false;
    if (nvalid > 0) {
      last_open = nvalid == SPAN && (p0 + SPAN) < n && !(packed[p0 + SPAN] & kHead);
      if (last_open) {
        pass = in_first && first_open;
        if (gl == 0) {
          s_cc[grp] = cc;
          s_ww[grp] = ww;
          s_seg[grp] = (uint32_t)seg;
        }
      } else if (in_first && first_open) {
        facc = acc; fcc = cc; fww = ww; owner = true;
      } else {
        last_closes = true;
      }
    }
    {
      const uint64_t mc = kPark ? __ballot(last_closes) : 0ull;
      if (last_closes) park(mc, mean_of(acc, cc), seg + hb, cc, ww, cur_key);
      parked += __popcll(mc) / LPR;
      if (!kOwnAcc) {
        while (parked > 0) pop(parked < kPop ? parked : kPop);
        first_parked = 0;
      }
    }
    if (last_open) s_acc_at(threadIdx.x) = acc;
    if (gl == 0) s_flags[grp] = (nvalid > 0 ? kValid : 0u) | (last_open ? kOpen : 0u) | (pass ? kPass : 0u);
    __syncthreads();

    // a group whose first run began before it closes the chain of runs
    {
      bool closes = false;
      f64x4 tot = facc;
      int tcc = fcc, tww = fww;
      if (owner) {
        for (int gg = grp - 1; gg >= 0; --gg) {
          tot += s_acc_at(gg * LPR + gl);
          tcc += s_cc[gg];
          tww += s_ww[gg];
          if (!(s_flags[gg] & kPass)) {
            closes = true;
            break;
          }
        }
        if (!closes) {   // the chain began in an earlier tile
          if (lane_on) *reinterpret_cast<f64x4*>(part.first_acc + tile * D + gl * 4) = tot;
          if (gl == 0) {
            part.first_cc[tile] = tcc;
            part.first_ww[tile] = tww;
          }
        }
      }
      const uint64_t mc = kPark ? __ballot(closes) : 0ull;
      if (closes) park(mc, mean_of(tot, tcc), (int64_t)gbase - 1 + hb0, tcc, tww, key0);
      parked += __popcll(mc) / LPR;
    }
    if (kPark)
      while (parked > 0) pop(parked < kPop ? parked : kPop);
    // the chain that runs into the next tile
    if (grp == G - 1 && (s_flags[G - 1] & kOpen)) {
      f64x4 tot = s_acc_at((G - 1) * LPR + gl);
      int tcc = s_cc[G - 1], tww = s_ww[G - 1];
      int gg = G - 1;
      while (gg > 0 && (s_flags[gg] & kPass)) {
        --gg;
        tot += s_acc_at(gg * LPR + gl);
        tcc += s_cc[gg];
        tww += s_ww[gg];
      }
      if (s_flags[gg] & kPass) {   // the whole tile is inside one segment
        if (lane_on) *reinterpret_cast<f64x4*>(part.first_acc + tile * D + gl * 4) = tot;
        if (gl == 0) {
          part.first_cc[tile] = tcc;
          part.first_ww[tile] = tww;
        }
      } else {
        if (lane_on) *reinterpret_cast<f64x4*>(part.last_acc + tile * D + gl * 4) = tot;
        if (gl == 0) {
          part.last_cc[tile] = tcc;
          part.last_ww[tile] = tww;
          // one lane per tile: the fixup pass takes the tiles from this list,
          // with the segment and the last tile it covers
          const uint32_t seg = s_seg[G - 1];
          int64_t end = (int64_t)seg + 1 <= n ? (int64_t)seg_start[seg + 1] : n;   // written by the position pass
          end = end < 1 ? 1 : (end > n ? n : end);
          part.fix_list[atomicAdd(part.fix_count, 1u)] =
              u32x4{(uint32_t)tile, seg, (uint32_t)((end - 1) / TILE), hb};
        }
      }
    }
  }
}

// Joins, for each segment that runs past the end of the tile holding its
// head, the partial sums of every later tile it covers.  Only the tiles the
// row pass listed are visited (about a third of them for Zipf IDs), spread
// over a fixed grid.  A lane group takes one listed tile whose segment covers
// at most kFixShort (and at most 256/LPR) later tiles, which is nearly all of
// them (the hot IDs have their own pass), with all its loads in flight at
// once; a longer chain (some 1700 tiles for the hottest ID at 65M positions
// without the hot-key plan) is summed by the whole block, 256/LPR groups with
// eight loads in flight each.  Both add the tail of the first tile, then the
// later tiles' partials in tile order.
constexpr int kFixBlock = 256;
constexpr int64_t kFixGrid = 2048;
constexpr int kFixShort = 8;
template <int LPR>
__global__ void __launch_bounds__(kFixBlock)
seg_fixup_kernel(SegmentArgs a, SegPartials part) {
  constexpr int G = kFixBlock / LPR;
  // a chain of at most G later tiles is summed in the same order by both paths
  constexpr int kShort = kFixShort < G ? kFixShort : G;
  __shared__ f64x4 s_acc[kFixBlock];
  __shared__ int32_t s_cc[G], s_ww[G];
  __shared__ uint32_t s_long[G];
  __shared__ uint32_t s_nlong;
  const int lane = threadIdx.x % LPR;
  const int grp = threadIdx.x / LPR;
  const bool lane_on = lane * 4 < a.D;
  const int D = a.D;
  const uint32_t count = *part.fix_count;
  // the listed tiles in any order: each one's sum is taken in a fixed order
  for (uint32_t k0 = blockIdx.x * (uint32_t)G; k0 < count; k0 += gridDim.x * (uint32_t)G) {
    if (threadIdx.x == 0) s_nlong = 0u;
    __syncthreads();
    const uint32_t k = k0 + grp;
    if (k < count) {
      const u32x4 rec = part.fix_list[k];
      const int64_t b = rec.x, seg = rec.y, b_end = rec.z, hb = rec.w;   // hb: hot IDs before it (split plan)
      if (seg < a.N) {   // always true when the numbering is consistent
        if (b_end - b <= kShort) {
          f64x4 v[kShort];
          int32_t c[kShort], ww[kShort];
#pragma unroll
          for (int u = 0; u < kShort; ++u) {
            const int64_t bb = b + 1 + u;
            const int64_t bc = bb <= b_end ? bb : b;   // clamped: read, then ignored
            v[u] = lane_on ? *reinterpret_cast<const f64x4*>(part.first_acc + bc * D + lane * 4)
                           : f64x4{0.0, 0.0, 0.0, 0.0};
            c[u] = part.first_cc[bc];
            ww[u] = part.first_ww[bc];
          }
          f64x4 tot = lane_on ? *reinterpret_cast<const f64x4*>(part.last_acc + b * D + lane * 4)
                              : f64x4{0.0, 0.0, 0.0, 0.0};
          int tcc = part.last_cc[b], tww = part.last_ww[b];
#pragma unroll
          for (int u = 0; u < kShort; ++u) {
            if (b + 1 + u > b_end) break;
            tot += v[u];
            tcc += c[u];
            tww += ww[u];
          }
          finalize_segment(a, seg + hb, tot, tcc, tww, lane, lane_on, a.ap.mode);
        } else if (lane == 0) {
          s_long[atomicAdd(&s_nlong, 1u)] = k;
        }
      }
    }
    __syncthreads();
    const uint32_t nlong = s_nlong;
    for (uint32_t i = 0; i < nlong; ++i) {
      const u32x4 rec = part.fix_list[s_long[i]];
      const int64_t b = rec.x, seg = rec.y, b_end = rec.z, hb = rec.w;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      int cc = 0, ww = 0;
#pragma unroll 8
      for (int64_t bb = b + 1 + grp; bb <= b_end; bb += G) {
        if (lane_on) acc += *reinterpret_cast<const f64x4*>(part.first_acc + bb * D + lane * 4);
        cc += part.first_cc[bb];
        ww += part.first_ww[bb];
      }
      s_acc[threadIdx.x] = acc;
      if (lane == 0) {
        s_cc[grp] = cc;
        s_ww[grp] = ww;
      }
      __syncthreads();
      if (grp == 0) {
        f64x4 tot = lane_on ? *reinterpret_cast<const f64x4*>(part.last_acc + b * D + lane * 4)
                            : f64x4{0.0, 0.0, 0.0, 0.0};
        int tcc = part.last_cc[b], tww = part.last_ww[b];
        for (int g = 0; g < G; ++g) {
          tot += s_acc[g * LPR + lane];
          tcc += s_cc[g];
          tww += s_ww[g];
        }
        finalize_segment(a, seg + hb, tot, tcc, tww, lane, lane_on, a.ap.mode);
      }
      __syncthreads();   // s_acc is rewritten for the next long chain
    }
  }
}

// ------------------------------------------------------------ hot IDs (split plan)
// Each hot ID's occurrences are one segment, split into chunks of `span`
// occurrences per lane group (hot_span), TILE per block.  The chunk prefix of the runs is
// rebuilt by every block from the hot occurrence counts.
struct HotPartials {
  double* acc;     // [chunks][D] float64 sums of the weighted rows
  int32_t* cnt;    // [chunks][4]: contributions, active contributions, first and last contribution
  uint32_t* cp;    // [H + 1] first chunk of each hot ID's run (written by block 0 of hot_rows)
};

// Weight of contribution m for the row with tag `tg` (per-ID mode) or its
// token weight, from the LDS tables.
__device__ __forceinline__ float row_weight(const SegmentArgs& a, const float* s_w, const int32_t* s_sm, int m,
                                           int64_t tg) {
  if (a.decay == GBA_DECAY_TOKEN) return s_w[m];
  int64_t st = tg - a.step + (int64_t)s_sm[m] + 1;
  st = st < 0 ? 0 : st;
  return st <= a.iota ? 1.0f : 0.0f;
}

template <int LPR>
__global__ void __launch_bounds__(kSegBlock)
hot_rows_kernel(SegmentArgs a, const int32_t* __restrict__ buckets, int q, int nbuckets, int span, HotPartials hp) {
  constexpr int GW = kWave / LPR;            // groups per wave
  constexpr int G = kSegWaves * GW;          // groups per block
  const int64_t TILE = (int64_t)G * span;
  extern __shared__ int32_t s_dyn[];
  __shared__ uint32_t s_cp[kHotSlots + 1];
  __shared__ uint32_t s_tmp[kSegWaves + 1];
  __shared__ f64x4 s_acc[kSegBlock];
  __shared__ int32_t s_c[G], s_a[G], s_first[G], s_last[G];
  const int K = a.K;
  const int D = a.D;
  int32_t* s_off = s_dyn;
  float* s_w = reinterpret_cast<float*>(s_dyn + K + 1);
  int32_t* s_sm = s_dyn + 2 * K + 1;
  int32_t* s_bucket = s_dyn + 3 * K + 1;
  const uint32_t H = *a.hot.meta;
  const int t = threadIdx.x;
  // chunks of every hot ID's run, and their prefix
  uint32_t nch = 0;
  if ((uint32_t)t < H) nch = (uint32_t)((a.hot.prefix[t + 1] - a.hot.prefix[t] + TILE - 1) / TILE);
  uint32_t total;
  const uint32_t ex = block_exclusive_scan<kSegBlock>(nch, s_tmp, &total);
  if ((uint32_t)t < H) s_cp[t] = ex;
  if (t == 0) s_cp[H] = total;
  if (blockIdx.x == 0) {
    if ((uint32_t)t < H) hp.cp[t] = ex;
    if (t == 0) hp.cp[H] = total;
  }
  const uint32_t b = blockIdx.x;
  if (b >= total) return;   // block-uniform; the grid is sized for the most chunks
  load_contrib_tables(a, buckets, nbuckets, s_off, s_w, s_sm, s_bucket);
  __syncthreads();
  // the run holding chunk b: the last h with s_cp[h] <= b
  uint32_t h = count_at_most(s_cp, H, (int64_t)b) - 1;
  const int64_t run_end = a.hot.prefix[h + 1];
  const int64_t c0 = (int64_t)a.hot.prefix[h] + (int64_t)(b - s_cp[h]) * TILE;
  const int64_t key = a.hot.ids[h];
  const int64_t tg = (a.decay == GBA_DECAY_ID_TAG && key < a.R) ? (int64_t)a.tag[key] : -1;

  const int w = t / kWave;
  const int lane = lane_id();
  const int gl = lane % LPR;
  const int grp = w * GW + lane / LPR;
  const bool lane_on = gl * 4 < D;
  const int64_t p0 = c0 + (int64_t)grp * span;
  const int64_t left = (p0 < run_end) ? run_end - p0 : 0;
  const int nvalid = left >= span ? span : (int)left;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  int cg = 0, ag = 0, first = -1, last = -1;
  for (int i0 = 0; i0 < nvalid; i0 += kBatch) {
    // the lanes of a group read the same indices (clamped into the run)
    uint32_t j[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int64_t pi = p0 + i0 + u;
      j[u] = a.hot.hot_vals[pi < run_end ? pi : run_end - 1];
    }
    int m[kBatch];
    float wt[kBatch];
    f32x4 rv[kBatch];
    uint32_t use = 0;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const bool valid = i0 + u < nvalid && (int64_t)j[u] < a.N;
      m[u] = valid ? contribution_of(s_off, s_bucket, q, K, j[u]) : 0;
      wt[u] = valid ? row_weight(a, s_w, s_sm, m[u], tg) : 0.0f;
      const bool on = valid && wt[u] != 0.0f && lane_on;
      use |= on ? (1u << u) : 0u;
      rv[u] = *reinterpret_cast<const f32x4*>(a.rows + (on ? (int64_t)j[u] * D + gl * 4 : 0));
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      if (i0 + u < nvalid) {
        if ((use >> u) & 1u) acc = fma_widen((double)wt[u], rv[u], acc);
        const bool newc = m[u] != last;   // occurrences of one contribution are consecutive
        cg += newc ? 1 : 0;
        ag += (newc && wt[u] != 0.0f) ? 1 : 0;
        if (first < 0) first = m[u];
        last = m[u];
      }
    }
  }
  s_acc[t] = acc;
  if (gl == 0) {
    s_c[grp] = cg;
    s_a[grp] = ag;
    s_first[grp] = first;
    s_last[grp] = last;
  }
  __syncthreads();
  if (grp == 0) {
    // groups in order; a contribution that runs across two groups counts once
    f64x4 tot = {0.0, 0.0, 0.0, 0.0};
    int C = 0, A = 0, f = -1, l = -1;
    for (int g = 0; g < G; ++g) {
      if (s_first[g] < 0) continue;   // an empty group (past the end of the run)
      tot += s_acc[g * LPR + gl];
      C += s_c[g];
      A += s_a[g];
      if (s_first[g] == l) {
        C -= 1;
        if (row_weight(a, s_w, s_sm, l, tg) != 0.0f) A -= 1;
      }
      if (f < 0) f = s_first[g];
      l = s_last[g];
    }
    if (lane_on) *reinterpret_cast<f64x4*>(hp.acc + (int64_t)b * D + gl * 4) = tot;
    if (gl == 0) {
      int32_t* c = hp.cnt + (int64_t)b * 4;
      c[0] = C;
      c[1] = A;
      c[2] = f;
      c[3] = l;
    }
  }
}

// One block per hot ID: joins the chunks of its run in a fixed order and
// writes its place among all IDs (after the cold segments below it, cnum),
// its start (the cold occurrences below it plus the hot ones before it), c_r,
// W_r and the weighted sum divided by c_r (or K).  From 2^25 occurrences the
// blocks have 1024 threads (the hottest ID then has some 1,800 chunks, joined
// by 128 lane groups), below that 256.
template <int LPR, int BLOCK>
__global__ void __launch_bounds__(BLOCK)
hot_finish_kernel(SegmentArgs a, HotPartials hp, const uint32_t* __restrict__ cnum,
                  const uint32_t* __restrict__ cold_below) {
  constexpr int G = BLOCK / LPR;
  __shared__ f64x4 s_acc[BLOCK];
  __shared__ int32_t s_c[G], s_a[G];
  const uint32_t H = *a.hot.meta;
  const uint32_t h = blockIdx.x;
  if (h >= H) return;
  const int D = a.D;
  const int t = threadIdx.x;
  const int lane = t % LPR;
  const int grp = t / LPR;
  const bool lane_on = lane * 4 < D;
  const int64_t key = a.hot.ids[h];
  const int64_t tg = (a.decay == GBA_DECAY_ID_TAG && key < a.R) ? (int64_t)a.tag[key] : -1;
  // cold occurrences below the hot ID (found by the position pass)
  const uint32_t below_all = cold_below[h];
  const uint32_t b0 = hp.cp[h], b1 = hp.cp[h + 1];
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  int C = 0, A = 0;
  // group grp takes chunks b0 + grp, b0 + grp + G, ... in that order, eight
  // loads in flight at a time
  constexpr int kFin = 8;
  for (uint32_t base = b0 + grp; base < b1; base += kFin * G) {
    f64x4 v[kFin];
    int32_t c0[kFin], c1[kFin], c2[kFin], prev_last[kFin];
#pragma unroll
    for (int u = 0; u < kFin; ++u) {
      const uint32_t bb = base + u * G;
      const uint32_t bc = bb < b1 ? bb : b1 - 1;   // clamped: read, then ignored
      v[u] = lane_on ? *reinterpret_cast<const f64x4*>(hp.acc + (int64_t)bc * D + lane * 4)
                     : f64x4{0.0, 0.0, 0.0, 0.0};
      const int32_t* c = hp.cnt + (int64_t)bc * 4;
      c0[u] = c[0];
      c1[u] = c[1];
      c2[u] = c[2];
      prev_last[u] = bc > b0 ? hp.cnt[(int64_t)(bc - 1) * 4 + 3] : -1;
    }
#pragma unroll
    for (int u = 0; u < kFin; ++u) {
      if (base + u * G >= b1) break;
      acc += v[u];
      C += c0[u];
      A += c1[u];
      if (c2[u] == prev_last[u]) {   // a contribution across two chunks counts once
        C -= 1;
        const int m = c2[u];
        float wm;
        if (a.decay == GBA_DECAY_TOKEN) {
          wm = a.w[m];
        } else {
          int64_t st = tg - a.tokens[m] + 1;
          st = st < 0 ? 0 : st;
          wm = st <= a.iota ? 1.0f : 0.0f;
        }
        if (wm != 0.0f) A -= 1;
      }
    }
  }
  s_acc[t] = acc;
  if (lane == 0) {
    s_c[grp] = C;
    s_a[grp] = A;
  }
  __syncthreads();
  if (grp == 0) {
    f64x4 tot = {0.0, 0.0, 0.0, 0.0};
    int tc = 0, ta = 0;
    for (int g = 0; g < G; ++g) {
      tot += s_acc[g * LPR + lane];
      tc += s_c[g];
      ta += s_a[g];
    }
    const int64_t out = (int64_t)h + cnum[h];
    if (out < a.N) {   // always true when the numbering is consistent
      finalize_segment(a, out, tot, tc, ta, lane, lane_on, a.ap.mode, (int64_t)key);
      if (lane == 0) {
        a.unique_ids[out] = key;
        a.seg_offsets[out] = (int64_t)below_all + a.hot.prefix[h];
      }
    }
  }
}

// Per-ID decay: every row with a non-zero weight now carries the current step.
__global__ void __launch_bounds__(kSegBlock)
tag_update_kernel(const int64_t* __restrict__ unique_ids, const int32_t* __restrict__ active_count,
                  const int64_t* __restrict__ num_unique, int32_t* __restrict__ tag, int32_t step) {
  const int64_t U = *num_unique;
  const int64_t stride = (int64_t)gridDim.x * kSegBlock;
  for (int64_t s = (int64_t)blockIdx.x * kSegBlock + threadIdx.x; s < U; s += stride)
    if (active_count[s] > 0) tag[unique_ids[s]] = step;
}

// Groups of 4 tiles below 4096 tiles, of 16 from there: a consumer's blocks
// add up the counts of the groups before theirs, or, past kRunFoldGroups
// groups, read them scanned.  A launch costs 4.5 us on a busy stream however
// little it does; the check of the offsets, the lookup buckets, the scan of
// the counts (one launch or three) and the segment total are six of them less
// here (26,624-ID pull request 57 -> 50 us, 6.5 M positions 673 -> 653 us).
static int run_group_shift(int64_t tiles) { return tiles >= 4096 ? 4 : 2; }

int64_t run_groups(int64_t N) {
  const int64_t tiles = N > 0 ? ceil_div(N, kMetaTile) : 1;
  return ceil_div(tiles, int64_t(1) << run_group_shift(tiles));
}

static hipError_t launch_run_heads_prep(const uint32_t* keys, int64_t N, uint32_t* tile_prefix, uint32_t* group,
                                        RunHeads* out, hipStream_t stream, const uint32_t* n_dev,
                                        const HeadsPrep* prep) {
  const int64_t tiles = ceil_div(N, kMetaTile);
  const int64_t groups = run_groups(N);
  out->tile_prefix = tile_prefix;
  out->group = group;
  out->shift = run_group_shift(tiles);
  out->groups = (int)groups;
  out->scanned = groups > kRunFoldGroups;
  static_assert((kMaxN >> 10 >> 4) + 1 <= (int64_t)kRunScanBlock * kRunScanItems, "one block scans every group");
  const dim3 grid((unsigned)(groups + (prep ? 1 : 0)));
  const HeadsPrep pr = prep ? *prep : HeadsPrep{};
#define GBA_RUN_HEADS(WAVES, PREP)                                                                                  \
  hipLaunchKernelGGL((run_heads_kernel<WAVES, PREP>), grid, dim3(WAVES * kWave), 0, stream, keys, N, n_dev, tiles, \
                     tile_prefix, group, pr)
  if (out->shift == 4) {
    if (prep) GBA_RUN_HEADS(16, true);
    else GBA_RUN_HEADS(16, false);
  } else {
    if (prep) GBA_RUN_HEADS(4, true);
    else GBA_RUN_HEADS(4, false);
  }
#undef GBA_RUN_HEADS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !out->scanned) return e;
  hipLaunchKernelGGL(run_group_scan_kernel, dim3(1), dim3(kRunScanBlock), 0, stream, group, (int)groups);
  return hipGetLastError();
}

hipError_t launch_run_heads(const uint32_t* keys, int64_t N, uint32_t* tile_prefix, uint32_t* group, RunHeads* out,
                            hipStream_t stream) {
  return launch_run_heads_prep(keys, N, tile_prefix, group, out, stream, nullptr, nullptr);
}

template <int LPR>
static hipError_t launch_rows(const SegmentArgs& a, const uint32_t* packed, const uint32_t* base,
                              SegPartials part, const uint32_t* seg_start, const uint32_t* cnum, HotPartials hp,
                              const int32_t* buckets, int q, int nb, const SegLayout& L, hipStream_t stream) {
  const int64_t tiles = L.row_tiles;
  const dim3 grid((unsigned)tiles), block(kSegBlock);
  const int span = L.span, bshift = base_shift(span);
#define GBA_ROWS(AP, CACHED)                                                                                          \
  hipLaunchKernelGGL((seg_rows_kernel<LPR, AP, CACHED>), grid, block, 0, stream, a, packed, base, span, bshift, part, \
                     seg_start, cnum)
  // rows of up to 32 floats that are not whole 64-byte pieces: below 128 bytes
  constexpr bool kNarrow = LPR <= 8;
  const bool cached = kNarrow && a.D % 16 != 0;
  if (a.ap.mode == 1) {
    if (cached) GBA_ROWS(1, kNarrow);
    else GBA_ROWS(1, false);
  } else if (a.ap.mode == 2) {
    if (cached) GBA_ROWS(2, kNarrow);
    else GBA_ROWS(2, false);
  } else {
    GBA_ROWS(0, false);
  }
#undef GBA_ROWS
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the listed tiles (at most all of them) are spread over a fixed grid
  const int64_t fix_blocks = tiles < kFixGrid ? tiles : kFixGrid;
  hipLaunchKernelGGL(seg_fixup_kernel<LPR>, dim3((unsigned)fix_blocks), dim3(kFixBlock), 0, stream, a, part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (a.n_dev) {
    const size_t lds = (size_t)(3 * a.K + 1 + nb) * sizeof(int32_t);
    hipLaunchKernelGGL(hot_rows_kernel<LPR>, dim3((unsigned)L.hot_chunks), dim3(kSegBlock), lds, stream, a, buckets,
                       q, nb, L.hot_span, hp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.N >= (int64_t(1) << 25))
      hipLaunchKernelGGL((hot_finish_kernel<LPR, 1024>), dim3(kHotSlots), dim3(1024), 0, stream, a, hp, cnum,
                         cnum + 2 * (kHotSlots + 1));
    else
      hipLaunchKernelGGL((hot_finish_kernel<LPR, 256>), dim3(kHotSlots), dim3(256), 0, stream, a, hp, cnum,
                         cnum + 2 * (kHotSlots + 1));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

// Tiles per block of the position pass: four share one load of the
// contribution tables; below 1024 tiles one each, so that the pass has blocks
// for every compute unit (20 tiles: 5.4 us instead of 12.4; 832 tiles: 9.3
// instead of 14.7; 293 tiles: 7.4 instead of 15.9).
static int meta_tiles_per_block(int64_t tiles) { return tiles >= 1024 ? 4 : 1; }

hipError_t launch_segments(const SegmentArgs& a, void* ws, hipStream_t stream) {
  const SegLayout L = seg_layout(a.N, a.D);
  char* base = static_cast<char*>(ws);
  uint32_t* tile_prefix = reinterpret_cast<uint32_t*>(base + L.off_heads);
  uint32_t* group = reinterpret_cast<uint32_t*>(base + L.off_hot_acc);   // shared with the later hot sums
  int32_t* buckets = reinterpret_cast<int32_t*>(base + L.off_buckets);
  uint32_t* packed = reinterpret_cast<uint32_t*>(base + L.off_packed);
  uint32_t* seg_base = reinterpret_cast<uint32_t*>(base + L.off_base);
  SegPartials part;
  int32_t* cnt = reinterpret_cast<int32_t*>(base + L.off_cnt);
  part.first_cc = cnt;
  part.first_ww = cnt + L.row_tiles;
  part.last_cc = cnt + 2 * L.row_tiles;
  part.last_ww = cnt + 3 * L.row_tiles;
  part.first_acc = reinterpret_cast<double*>(base + L.off_first_acc);
  part.last_acc = reinterpret_cast<double*>(base + L.off_last_acc);
  part.fix_count = reinterpret_cast<uint32_t*>(base + L.off_fix);
  part.fix_list = reinterpret_cast<u32x4*>(base + L.off_fix + 256);
  uint32_t* seg_start = reinterpret_cast<uint32_t*>(base + L.off_start);
  uint32_t* cnum = reinterpret_cast<uint32_t*>(base + L.off_cnum);
  HotPartials hp;
  hp.acc = reinterpret_cast<double*>(base + L.off_hot_acc);
  hp.cnt = reinterpret_cast<int32_t*>(base + L.off_hot_cnt);
  hp.cp = cnum + kHotSlots + 1;
  uint32_t* cold_below = cnum + 2 * (kHotSlots + 1);

  if (a.N <= 0) {
    hipLaunchKernelGGL(seg_empty_kernel, dim3(1), dim3(kSegBlock), 0, stream, a.offsets, a.K, a.num_unique,
                       a.seg_offsets, a.err);
    return hipGetLastError();
  }
  const int q = bucket_shift(a.N, a.K);
  const int nb = (int)(((a.N - 1) >> q) + 1);
  HeadsPrep prep;
  prep.off = a.offsets;
  prep.bucket = buckets;
  prep.fix_count = part.fix_count;
  prep.err = a.err;
  prep.N = a.N;
  prep.K = a.K;
  prep.q = q;
  prep.nb = nb;
  RunHeads heads;
  hipError_t e = launch_run_heads_prep(a.keys, a.N, tile_prefix, group, &heads, stream, a.n_dev, &prep);
  if (e != hipSuccess) return e;
  const size_t lds = (size_t)(3 * a.K + 1 + nb) * sizeof(int32_t);
  const int tpb = meta_tiles_per_block(L.meta_tiles);
  const dim3 mgrid((unsigned)ceil_div(L.meta_tiles, tpb));
  if (tpb == 4)
    hipLaunchKernelGGL(seg_meta_kernel<4>, mgrid, dim3(kSegBlock), lds, stream, a, heads, (const int32_t*)buckets, q, nb,
                       L.meta_tiles, packed, seg_base, base_shift(L.span), seg_start, cnum, cold_below);
  else
    hipLaunchKernelGGL(seg_meta_kernel<1>, mgrid, dim3(kSegBlock), lds, stream, a, heads, (const int32_t*)buckets, q, nb,
                       L.meta_tiles, packed, seg_base, base_shift(L.span), seg_start, cnum, cold_below);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  switch (lanes_per_row(a.D)) {
    case 1: e = launch_rows<1>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 2: e = launch_rows<2>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 4: e = launch_rows<4>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 8: e = launch_rows<8>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 16: e = launch_rows<16>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 32: e = launch_rows<32>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    case 64: e = launch_rows<64>(a, packed, seg_base, part, seg_start, cnum, hp, buckets, q, nb, L, stream); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (a.decay == GBA_DECAY_ID_TAG && a.ap.mode == 0) {   // a fused apply writes the tags as it goes
    int64_t blocks = ceil_div(a.N, kSegBlock);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(tag_update_kernel, dim3((unsigned)blocks), dim3(kSegBlock), 0, stream,
                       (const int64_t*)a.unique_ids, (const int32_t*)a.active_count,
                       (const int64_t*)a.num_unique, a.tag, (int32_t)a.step);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gba
