// The ID sort of small inputs without hot keys: stable LSD radix passes as in
// the large sort, but with as few launches as the size allows, since a launch
// costs 4 to 5 us on a busy stream however few keys it moves.
//  * Digits of up to 11 bits where a wider digit saves a pass that costs more
//    (pass_bits).
//  * Up to kSelfMost keys, one launch per pass: every block counts the digits
//    of all keys itself (before and after its own tile), so no launch has to
//    count for it.
//  * Above, two launches per pass: the counts per tile and per chunk of
//    tiles, and a scatter whose blocks add up the chunk rows (128 at most)
//    themselves instead of reading them scanned by a launch in between.  That
//    costs every block, so from 2^20 keys the large sort's three launches per
//    pass are as fast or faster (small_sort_takes).
// Bound by the launches' latency, not by bytes.  Measured: 20,480 17-bit keys
// 18.6 us (34 with three launches per byte), 26,624 24-bit keys 27.5 (41),
// 256,000 27-bit keys 47 (53, and four launches more between), 300,007 21-bit
// keys 37 (42), 851,968 24-bit keys 50 (56).
#include <algorithm>

#include "gba_device.hpp"
#include "gba_internal.hpp"
#include "sort_device.hpp"

namespace gba {

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- shared
// Four consecutive keys from position i0 (a multiple of 4), those past n as
// 0: int64 IDs on the first pass (one outside [0, R) is reported and sorted
// as 0), else the u32 keys.
template <bool FIRST>
__device__ __forceinline__ void load4(const void* __restrict__ src, int64_t i0, int64_t n, int64_t R, uint32_t (&k)[4],
                                      bool* bad) {
  if (FIRST) {
    const int64_t* ids = static_cast<const int64_t*>(src);
    int64_t v[4];
    if (i0 + 3 < n) {
      const i64x2 a = *reinterpret_cast<const i64x2*>(ids + i0);
      const i64x2 b = *reinterpret_cast<const i64x2*>(ids + i0 + 2);
      v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = i0 + e < n ? ids[i0 + e] : 0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool out = v[e] < 0 || v[e] >= R;
      *bad |= out;
      k[e] = out ? 0u : (uint32_t)v[e];
    }
  } else {
    const uint32_t* keys = static_cast<const uint32_t*>(src);
    if (i0 + 3 < n) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(keys + i0);
      k[0] = v.x; k[1] = v.y; k[2] = v.z; k[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) k[e] = i0 + e < n ? keys[i0 + e] : 0u;
    }
  }
}

// One add to counts[digit * copies + copy] per run of equal digits among a
// lane's `valid` (0 to 4) consecutive keys.
__device__ __forceinline__ void count4(const uint32_t (&k)[4], int valid, int shift, uint32_t mask, uint32_t* counts,
                                       int copy_shift, uint32_t copy) {
  uint32_t cur = (k[0] >> shift) & mask;
  uint32_t len = valid > 0 ? 1u : 0u;
#pragma unroll
  for (int e = 1; e < 4; ++e) {
    if (e < valid) {
      const uint32_t d = (k[e] >> shift) & mask;
      if (d == cur) {
        ++len;
      } else {
        atomicAdd(&counts[(cur << copy_shift) + copy], len);
        cur = d;
        len = 1;
      }
    }
  }
  if (len) atomicAdd(&counts[(cur << copy_shift) + copy], len);
}

// Key of position i (i < n) on its own.
template <bool FIRST>
__device__ __forceinline__ uint32_t load1(const void* __restrict__ src, int64_t i, int64_t R) {
  if (FIRST) {
    const uint64_t id = static_cast<const uint64_t*>(src)[i];
    return id < (uint64_t)R ? (uint32_t)id : 0u;
  }
  return static_cast<const uint32_t*>(src)[i];
}

// ------------------------------------------------- one launch per pass
// A block of 16 waves ranks a tile of 2048 keys and counts the digits of
// every other key into two LDS arrays (before its tile, after it), so that it
// knows where each digit's keys of its tile go.  Positions fit 16 bits.
constexpr int kSelfBlock = 1024;
constexpr int kSelfWaves = kSelfBlock / kWave;
constexpr int kSelfItems = 2;
constexpr int kSelfTile = kSelfBlock * kSelfItems;
// Where counting every key in every block still costs less (4 us a pass at
// 26,624 keys) than the launch that would count for the scatter.
constexpr int64_t kSelfMost = 32768;
static_assert(kSelfMost < 65536, "16-bit positions");

template <bool FIRST, int BITS>
__global__ void __launch_bounds__(kSelfBlock)
self_sort_kernel(const void* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
                 uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, int n, int shift, uint32_t mask,
                 int64_t R, int32_t* __restrict__ err) {
  constexpr int BINS = 1 << BITS;
  constexpr int kCopyShift = BINS >= 1024 ? 0 : 10 - BITS;      // 1024 counters at least
  constexpr int PER = BINS > kSelfBlock ? BINS / kSelfBlock : 1;   // bins per thread
  constexpr int kUnroll = 4;                                     // vectors of 4 keys in flight per lane
  __shared__ uint32_t cnt32[kSelfWaves][BINS / 2];               // 16-bit counts, then positions, per (wave, digit)
  __shared__ uint32_t s_before[BINS << kCopyShift];
  __shared__ uint32_t s_after[BINS << kCopyShift];
  __shared__ uint32_t tmp[kSelfWaves + 1];
  uint16_t(*cnt)[BINS] = reinterpret_cast<uint16_t(*)[BINS]>(&cnt32[0][0]);
  const int tile0 = (int)blockIdx.x * kSelfTile;
  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  for (int i = lane; i < BINS / 2; i += kWave) cnt32[w][i] = 0u;
  for (int i = threadIdx.x; i < (BINS << kCopyShift); i += kSelfBlock) {
    s_before[i] = 0u;
    s_after[i] = 0u;
  }
  // the tile's keys: wave w takes positions [w * 128, +128) of the tile
  uint32_t key[kSelfItems], val[kSelfItems];
  bool active[kSelfItems];
#pragma unroll
  for (int r = 0; r < kSelfItems; ++r) {
    const int i = tile0 + w * (kWave * kSelfItems) + r * kWave + lane;
    active[r] = i < n;
    const int ic = active[r] ? i : n - 1;
    key[r] = load1<FIRST>(keys_in, ic, R);
    val[r] = FIRST ? (uint32_t)ic : vals_in[ic];
  }
  __syncthreads();
  bool bad = false;
  const uint32_t copy = (uint32_t)lane & ((1u << kCopyShift) - 1u);
  const int vectors = (n + 3) / 4;
  for (int v0 = 0; v0 < vectors; v0 += kUnroll * kSelfBlock) {
    uint32_t k[kUnroll][4];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int v = v0 + u * kSelfBlock + (int)threadIdx.x;
      load4<FIRST>(keys_in, 4 * (int64_t)(v < vectors ? v : vectors - 1), n, R, k[u], &bad);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int i0 = 4 * (v0 + u * kSelfBlock + (int)threadIdx.x);
      if (i0 >= n || (i0 >= tile0 && i0 < tile0 + kSelfTile)) continue;   // the tile's own keys are ranked below
      count4(k[u], n - i0 < 4 ? n - i0 : 4, shift, mask, i0 < tile0 ? s_before : s_after, kCopyShift, copy);
    }
  }
  if (FIRST && bad) raise_error(err, GBA_DERR_ID_RANGE);
  // stable ranks within (wave, digit): rounds in index order, lanes in order
  uint32_t rank[kSelfItems];
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < kSelfItems; ++r) {
    const uint32_t digit = (key[r] >> shift) & mask;
    const uint64_t m = match_digit_n<BITS>(digit, active[r]);
    uint32_t earlier = 0;
    if (active[r]) earlier = cnt[w][digit];
    __builtin_amdgcn_wave_barrier();   // every lane has read the counter before its leader updates it
    if (active[r] && (m & lt) == 0) cnt[w][digit] = (uint16_t)(earlier + (uint32_t)__popcll(m));
    rank[r] = earlier + (uint32_t)__popcll(m & lt);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  uint32_t before[PER], total[PER], sum = 0;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int b = (int)threadIdx.x * PER + p;
    before[p] = total[p] = 0;
    if (b < BINS) {
#pragma unroll
      for (int c = 0; c < (1 << kCopyShift); ++c) {
        before[p] += s_before[(b << kCopyShift) + c];
        total[p] += s_after[(b << kCopyShift) + c];
      }
      total[p] += before[p];
#pragma unroll
      for (int k = 0; k < kSelfWaves; ++k) total[p] += cnt[k][b];
    }
    sum += total[p];
  }
  uint32_t all;
  uint32_t start = block_exclusive_scan<kSelfBlock>(sum, tmp, &all);
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int b = (int)threadIdx.x * PER + p;
    if (b < BINS) {
      uint32_t run = start + before[p];
#pragma unroll
      for (int k = 0; k < kSelfWaves; ++k) {
        const uint32_t c = cnt[k][b];
        cnt[k][b] = (uint16_t)run;
        run += c;
      }
    }
    start += total[p];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSelfItems; ++r) {
    if (!active[r]) continue;
    const uint32_t out = cnt[w][(key[r] >> shift) & mask] + rank[r];
    if (out < (uint32_t)n) {   // always true when the counts are consistent
      keys_out[out] = key[r];
      vals_out[out] = val[r];
    }
  }
}

// ------------------------------------------------ two launches per pass
constexpr int kMidBlock = 256;
constexpr int kMidWaves = kMidBlock / kWave;
constexpr int kHistWaves = 16;

// Digit counts of a chunk of TILES tiles by one block of 16 waves, 16 / TILES
// waves per tile (few keys per wave: the launch is over in one round of loads
// on as many compute units as there are chunks).  Each tile's row holds the
// counts of the chunk's earlier tiles, the chunk row the chunk's counts.
// Interleaved copies of each counter, as far as 64 KB of LDS allow: lanes
// that add to one frequent digit touch different words.
template <bool FIRST, int ITEMS, int BITS, int TILES>
__global__ void __launch_bounds__(kHistWaves * kWave)
mid_hist_kernel(const void* __restrict__ keys_in, int64_t n, int shift, uint32_t mask, int64_t R,
                uint32_t* __restrict__ hist, uint32_t* __restrict__ chunk, int64_t tiles, int32_t* __restrict__ err) {
  constexpr int BINS = 1 << BITS;
  constexpr int kCopyShift = TILES * BINS * 4 <= 16384 ? 2 : (TILES * BINS * 2 <= 16384 ? 1 : 0);
  constexpr int kCopies = 1 << kCopyShift;
  constexpr int kPerTile = kHistWaves / TILES;                         // waves per tile
  constexpr int kKeys = kMidBlock * ITEMS / kPerTile;                  // keys per wave
  constexpr int kVecs = kKeys / (4 * kWave);                           // vectors of 4 keys per lane
  static_assert(kVecs >= 1 && kVecs * 4 * kWave == kKeys, "whole vectors");
  __shared__ uint32_t h[TILES][BINS * kCopies];
  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  const int64_t tile = (int64_t)blockIdx.x * TILES + w / kPerTile;
  const int64_t i00 = tile * (kMidBlock * ITEMS) + (w % kPerTile) * kKeys;
  bool bad = false;
  uint32_t k[kVecs][4];
#pragma unroll
  for (int u = 0; u < kVecs; ++u) {
    // lane l holds keys i00 + 4 (l + 64 u) + e: 1 KB of consecutive keys per vector load of the wave
    const int64_t i0 = i00 + 4 * ((int64_t)lane + (int64_t)kWave * u);
    load4<FIRST>(keys_in, i0 < n ? i0 : (n - 1) & ~int64_t(3), n, R, k[u], &bad);
  }
  for (int i = threadIdx.x; i < TILES * BINS * kCopies; i += kHistWaves * kWave) (&h[0][0])[i] = 0u;
  __syncthreads();
  const uint32_t copy = (uint32_t)lane & (uint32_t)(kCopies - 1);
#pragma unroll
  for (int u = 0; u < kVecs; ++u) {
    const int64_t left = n - (i00 + 4 * ((int64_t)lane + (int64_t)kWave * u));
    count4(k[u], left < 0 ? 0 : (left < 4 ? (int)left : 4), shift, mask, h[w / kPerTile], kCopyShift, copy);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < BINS; d += kHistWaves * kWave) {
    const int64_t t0 = (int64_t)blockIdx.x * TILES;
    uint32_t s = 0;
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      if (t0 + t < tiles) hist[(t0 + t) * BINS + d] = s;
#pragma unroll
      for (int j = 0; j < kCopies; ++j) s += h[t][d * kCopies + j];
    }
    chunk[(int64_t)blockIdx.x * BINS + d] = s;
  }
  if (FIRST && bad) raise_error(err, GBA_DERR_ID_RANGE);
}

// PER consecutive words (PER a power of two, the address a multiple of their size).
template <int PER>
__device__ __forceinline__ void load_per(const uint32_t* __restrict__ p, uint32_t (&v)[PER]) {
  if constexpr (PER == 1) {
    v[0] = *p;
  } else if constexpr (PER == 2) {
    const u32x2 x = *reinterpret_cast<const u32x2*>(p);
    v[0] = x.x; v[1] = x.y;
  } else {
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
      const u32x4 x = reinterpret_cast<const u32x4*>(p)[q];
      v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
    }
  }
}

// Scatter of one tile: thread t owns bins [t * PER, +PER).  The digit starts
// and the tile's place in each digit come from the chunk rows, added up here.
// Keys, then values, are staged through LDS in digit order, so that runs of
// equal digits are written together (written where they are ranked: 14-18 us
// a pass instead of 11-13).
template <bool FIRST, int ITEMS, int BITS>
__global__ void __launch_bounds__(kMidBlock)
mid_scatter_kernel(const void* __restrict__ keys_in, const uint32_t* __restrict__ vals_in,
                   uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, int64_t n, int shift,
                   uint32_t mask, int64_t R, const uint32_t* __restrict__ hist, const uint32_t* __restrict__ chunk,
                   int nchunks, int chunk_shift) {
  constexpr int BINS = 1 << BITS;
  constexpr int PER = BINS / kMidBlock;
  constexpr int kTile = kMidBlock * ITEMS;
  constexpr int kBatch = 16;          // chunk rows in flight per wave
  __shared__ uint32_t cnt[kMidWaves][BINS];
  __shared__ uint32_t gshift[BINS];   // per digit: first its keys in earlier chunks, then output minus tile position
  __shared__ uint32_t s_tot[BINS];    // per digit: its keys in all chunks
  __shared__ uint32_t tmp[2 * kMidWaves];
  __shared__ uint32_t s_keys[kTile];
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t tile0 = tile * kTile;
  const int tile_n = n - tile0 < kTile ? (int)(n - tile0) : kTile;
  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  const int lbase = w * (kWave * ITEMS) + lane;
  uint32_t key[ITEMS], val[FIRST ? 1 : ITEMS], rank[ITEMS];
  // every lane loads (past the end the last key again), so no branch waits on a load
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int li = lbase + r * kWave;
    const int64_t ic = tile0 + (li < tile_n ? li : tile_n - 1);
    key[r] = load1<FIRST>(keys_in, ic, R);
    if (!FIRST) val[FIRST ? 0 : r] = vals_in[ic];
  }
  uint32_t off[PER];
  load_per<PER>(hist + tile * BINS + threadIdx.x * PER, off);
  for (int i = threadIdx.x; i < BINS; i += kMidBlock) {
    gshift[i] = 0u;
    s_tot[i] = 0u;
  }
  __syncthreads();
  // the chunk rows, a lane four bins at a time: a wave takes every 256th
  // block of bins (kShare waves share one where there are fewer than four,
  // each every kShare-th row), and the sums meet in LDS
  {
    constexpr int kShare = BINS >= 1024 ? 1 : 1024 / BINS;
    const int mine = (int)(tile >> chunk_shift);
#pragma unroll
    for (int q = w / kShare; q < BINS / 256; q += kMidWaves / kShare) {
      const int b0 = q * 256 + lane * 4;
      u32x4 t4 = {0u, 0u, 0u, 0u}, o4 = {0u, 0u, 0u, 0u};
      for (int c0 = w % kShare; c0 < nchunks; c0 += kShare * kBatch) {
        u32x4 v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int c = c0 + k * kShare < nchunks ? c0 + k * kShare : nchunks - 1;
          v[k] = *reinterpret_cast<const u32x4*>(chunk + (int64_t)c * BINS + b0);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int c = c0 + k * kShare;
          t4 += c < nchunks ? v[k] : u32x4{0u, 0u, 0u, 0u};
          o4 += c < mine ? v[k] : u32x4{0u, 0u, 0u, 0u};
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        atomicAdd(&s_tot[b0 + e], t4[e]);
        atomicAdd(&gshift[b0 + e], o4[e]);
      }
    }
  }
  for (int i = lane; i < BINS; i += kWave) cnt[w][i] = 0u;
  __builtin_amdgcn_wave_barrier();
  auto active_at = [&](int r) -> bool { return lbase + r * kWave < tile_n; };
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool active = active_at(r);
    const uint32_t digit = (key[r] >> shift) & mask;
    const uint64_t m = match_digit_n<BITS>(digit, active);
    uint32_t earlier = 0;
    if (active) earlier = cnt[w][digit];
    __builtin_amdgcn_wave_barrier();   // every lane has read the counter before its leader updates it
    if (active && (m & lt) == 0) cnt[w][digit] = earlier + (uint32_t)__popcll(m);
    rank[r] = opaque(earlier + (uint32_t)__popcll(m & lt));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  {
    uint32_t own[PER], tot[PER], own_sum = 0, tot_sum = 0;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      tot[p] = s_tot[threadIdx.x * PER + p];
      off[p] += gshift[threadIdx.x * PER + p];
      own[p] = 0;
#pragma unroll
      for (int k = 0; k < kMidWaves; ++k) own[p] += cnt[k][threadIdx.x * PER + p];
      own_sum += own[p];
      tot_sum += tot[p];
    }
    // exclusive scans of both sums over the block, behind one barrier
    const uint32_t inc_own = wave_inclusive_scan(own_sum), inc_tot = wave_inclusive_scan(tot_sum);
    if (lane == kWave - 1) {
      tmp[w] = inc_own;
      tmp[kMidWaves + w] = inc_tot;
    }
    __syncthreads();
    uint32_t ex = inc_own - own_sum, start = inc_tot - tot_sum;
    for (int k = 0; k < w; ++k) {
      ex += tmp[k];
      start += tmp[kMidWaves + k];
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int b = threadIdx.x * PER + p;
      gshift[b] = start + off[p] - ex;   // modulo 2^32
      uint32_t run = ex;
#pragma unroll
      for (int k = 0; k < kMidWaves; ++k) {
        const uint32_t c = cnt[k][b];
        cnt[k][b] = run;
        run += c;
      }
      ex += own[p];
      start += tot[p];
    }
  }
  __syncthreads();
  uint32_t pos[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) pos[r] = cnt[w][(opaque(key[r]) >> shift) & mask] + rank[r];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (active_at(r)) s_keys[pos[r]] = key[r];
  __syncthreads();
  uint32_t out[ITEMS];   // staged position i = threadIdx.x + r * kMidBlock goes to out[r]
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int i = threadIdx.x + r * kMidBlock;
    out[r] = 0u;
    if (i < tile_n) {
      const uint32_t k = s_keys[i];
      out[r] = gshift[(k >> shift) & mask] + (uint32_t)i;
      if ((int64_t)out[r] < n) keys_out[out[r]] = k;   // always true when the counts are consistent
    }
  }
  __syncthreads();   // every key is read out before the values take the buffer
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (active_at(r)) s_keys[pos[r]] = FIRST ? (uint32_t)(tile0 + lbase + r * kWave) : val[FIRST ? 0 : r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int i = threadIdx.x + r * kMidBlock;
    if (i < tile_n && (int64_t)out[r] < n) vals_out[out[r]] = s_keys[i];
  }
}

// ---------------------------------------------------------------- host
struct SmallPlan {
  bool self;            // one launch per pass
  int passes, bins_log2;
  int bits[4], shift[4];
  int items;            // keys per lane in the scatter (tiles of 256 * items keys)
  int chunk_shift;
  int64_t tiles, chunks;
};

constexpr int64_t kDigit11Below = int64_t(1) << 19;
constexpr int64_t kDigit10Below = int64_t(1) << 20;
constexpr int64_t kFourTileChunks = 512;   // most tiles of a pass with chunks of four, not eight

// Bits of the widest digit of a key of key_bits: as few passes as digits of 9
// bits allow, or wider ones where the pass they save costs more than they do.
// us per pass, digits of 8, 9, 10 and 11 bits: 130,000 keys 11.7 12.3 14.1 16.1,
// 260,000 12.4 13.3 16.4 18.8, 400,000 13.1 15.3 20.5 23.3, 850,000 18.2 22.3
// 31.8 -: two passes of 11 bits instead of three of 8 pay to about 200,000 keys
// (22-bit keys, 130,000: 32 us and 35, 400,000: 47 and 39), two of 10 to about
// 330,000, three of 10 instead of four of 8 to about 200,000, three of 11 as
// long as a pass is one launch (32-bit keys, 20,000: 36 us and 37, 65,000: 46
// and 44); one pass of either pays as far as its counts fit.
static int pass_bits(int64_t n, int key_bits) {
  for (int passes = 1;; ++passes) {
    const int bits = (key_bits + passes - 1) / passes;
    if (bits <= 9) return bits;
    if (bits == 10 && n < (passes == 1 ? kDigit10Below : (passes == 2 ? 5 << 16 : 3 << 16))) return bits;
    if (bits == 11 && n < (passes == 1 ? kDigit11Below : (passes == 2 ? 3 << 16 : kSelfMost + 1))) return bits;
  }
}

// From 2^20 keys the chunk rows that every scatter block adds up cost what the
// scan between them would (850,000 24-bit keys 54.6 us, 55.3 with the large
// sort; 1.7 M 76 and 71, 3.3 M 109 and 92): the large sort then, but for keys
// that 9-bit digits take in a pass less, and for these as far as that pass
// pays: one pass to 2^22 keys (9-bit keys, 3.3 M: 51 us and 60), two to 3 * 2^20
// (18-bit, 2.6 M: 72 and 80, 3.3 M: 89 and 88), three to 2^21 (27-bit, 1.7 M: 85
// and 93, 2.1 M: 95 and 93).
bool small_sort_takes(int64_t n, int key_bits) {
  if (n < kDigit10Below) return true;
  const int passes = (key_bits + 8) / 9;
  return passes < (key_bits + 7) / 8 && n < (int64_t)(5 - passes) << 20;
}
static_assert(kSmallSortBelow == int64_t(4) << 20, "one pass");

// The widest digit of any key for n keys.
static int widest_digit(int64_t n) { return n < kDigit11Below ? 11 : (n < kDigit10Below ? 10 : 9); }

static SmallPlan small_plan(int64_t n, int key_bits) {
  SmallPlan p{};
  p.self = n <= kSelfMost;
  const int bits = pass_bits(n, key_bits);
  p.passes = (key_bits + bits - 1) / bits;
  // the narrowest digits first, as the first pass reads the widest keys
  int at = 0, widest = 8;
  for (int k = 0; k < p.passes; ++k) {
    p.bits[k] = key_bits / p.passes + (k >= p.passes - key_bits % p.passes ? 1 : 0);
    p.shift[k] = at;
    at += p.bits[k];
    if (p.bits[k] > widest) widest = p.bits[k];
  }
  p.bins_log2 = widest;   // the rows' width: 256 counters at least
  // 2048-key tiles below 2^20 keys (blocks for every compute unit), 4096 above (longer runs)
  p.items = n < kDigit10Below ? 8 : 16;
  p.tiles = ceil_div(n > 0 ? n : 1, (int64_t)kMidBlock * p.items);
  p.chunk_shift = p.tiles <= kFourTileChunks ? 2 : 3;   // at most 128 chunk rows for a scatter block to add up
  p.chunks = ceil_div(p.tiles, int64_t(1) << p.chunk_shift);
  return p;
}

struct SmallLayout {
  size_t off_keys[2], off_vals[2], off_hist, off_chunk, bytes;
};

static SmallLayout small_layout(int64_t n, const SmallPlan& p) {
  SmallLayout L{};
  const size_t arr = align_up((size_t)(n > 0 ? n : 1) * sizeof(uint32_t));
  size_t o = 0;
  for (int k = 0; k < 2; ++k) {
    L.off_keys[k] = o; o += arr;
    L.off_vals[k] = o; o += arr;
  }
  L.off_hist = o;  o += p.self ? 0 : align_up((size_t)p.tiles * (4u << p.bins_log2));
  L.off_chunk = o; o += p.self ? 0 : align_up((size_t)p.chunks * (4u << p.bins_log2));
  L.bytes = o;
  return L;
}

// Every size takes the most at the widest digits its size allows; the counts
// shrink where these, or the tiles, change.
size_t small_sort_count_room(int64_t n) {
  auto counts = [](int64_t m) {
    SmallPlan p = small_plan(m, 1);
    p.bins_log2 = widest_digit(m);
    const SmallLayout L = small_layout(m, p);
    return L.bytes - L.off_hist;
  };
  size_t most = counts(n);
  for (const int64_t end : {kDigit11Below - 1, kDigit10Below - 1, kFourTileChunks * kMidBlock * 16})
    if (end < n) most = std::max(most, counts(end));
  return most;
}

hipError_t launch_small_sort(const int64_t* ids, int64_t n, int64_t R, int key_bits, void* ws, const uint32_t** keys_out,
                             const uint32_t** vals_out, uint32_t** idle_out, int32_t* err, hipStream_t stream) {
  const SmallPlan p = small_plan(n, key_bits);
  const SmallLayout L = small_layout(n, p);
  char* base = static_cast<char*>(ws);
  uint32_t *keys[2], *vals[2];
  for (int k = 0; k < 2; ++k) {
    keys[k] = reinterpret_cast<uint32_t*>(base + L.off_keys[k]);
    vals[k] = reinterpret_cast<uint32_t*>(base + L.off_vals[k]);
  }
  uint32_t* hist = reinterpret_cast<uint32_t*>(base + L.off_hist);
  uint32_t* chunk = reinterpret_cast<uint32_t*>(base + L.off_chunk);
  const int last = (p.passes - 1) & 1;
  *keys_out = keys[last];
  *vals_out = vals[last];
  if (idle_out) *idle_out = vals[1 - last];
  for (int pass = 0; pass < p.passes && n > 0; ++pass) {
    const int out = pass & 1;
    const void* kin = pass == 0 ? (const void*)ids : (const void*)keys[1 - out];
    const uint32_t* vin = pass == 0 ? nullptr : vals[1 - out];
    const uint32_t mask = (1u << p.bits[pass]) - 1u;
    const int shift = p.shift[pass];
    hipError_t e;
    if (p.self) {
      const dim3 grid((unsigned)ceil_div(n, kSelfTile)), block(kSelfBlock);
#define GBA_SELF(F, B)                                                                                         \
  hipLaunchKernelGGL((self_sort_kernel<F, B>), grid, block, 0, stream, kin, vin, keys[out], vals[out], (int)n, \
                     shift, mask, R, err)
#define GBA_SELF_BITS(F)          \
  switch (p.bins_log2) {          \
    case 8: GBA_SELF(F, 8); break;   \
    case 9: GBA_SELF(F, 9); break;   \
    case 10: GBA_SELF(F, 10); break; \
    default: GBA_SELF(F, 11); break; \
  }
      if (pass == 0) {
        GBA_SELF_BITS(true)
      } else {
        GBA_SELF_BITS(false)
      }
#undef GBA_SELF_BITS
#undef GBA_SELF
      if ((e = hipGetLastError()) != hipSuccess) return e;
      continue;
    }
    const dim3 hgrid((unsigned)p.chunks), hblock(kHistWaves * kWave), grid((unsigned)p.tiles), block(kMidBlock);
#define GBA_MID_HIST(F, IT, B, T)                                                                                  \
  hipLaunchKernelGGL((mid_hist_kernel<F, IT, B, T>), hgrid, hblock, 0, stream, kin, n, shift, mask, R, hist, chunk, \
                     p.tiles, err)
    // (from 2^20 keys small_sort_takes leaves keys with a 9-bit digit only)
#define GBA_MID_HIST_BITS(F)                             \
  if (p.items == 16) {                                   \
    if (p.chunk_shift == 2) GBA_MID_HIST(F, 16, 9, 4);   \
    else GBA_MID_HIST(F, 16, 9, 8);                      \
  } else {                                               \
    switch (p.bins_log2) {                               \
      case 8: GBA_MID_HIST(F, 8, 8, 4); break;           \
      case 9: GBA_MID_HIST(F, 8, 9, 4); break;           \
      case 10: GBA_MID_HIST(F, 8, 10, 4); break;         \
      default: GBA_MID_HIST(F, 8, 11, 4); break;         \
    }                                                    \
  }
    if (pass == 0) {
      GBA_MID_HIST_BITS(true)
    } else {
      GBA_MID_HIST_BITS(false)
    }
#undef GBA_MID_HIST_BITS
#undef GBA_MID_HIST
    if ((e = hipGetLastError()) != hipSuccess) return e;
#define GBA_MID(F, IT, B)                                                                                        \
  hipLaunchKernelGGL((mid_scatter_kernel<F, IT, B>), grid, block, 0, stream, kin, vin, keys[out], vals[out], n, shift, \
                     mask, R, (const uint32_t*)hist, (const uint32_t*)chunk, (int)p.chunks, p.chunk_shift)
#define GBA_MID_BITS(F)                          \
  if (p.items == 8) {                            \
    switch (p.bins_log2) {                       \
      case 8: GBA_MID(F, 8, 8); break;           \
      case 9: GBA_MID(F, 8, 9); break;           \
      case 10: GBA_MID(F, 8, 10); break;         \
      default: GBA_MID(F, 8, 11); break;         \
    }                                            \
  } else {                                       \
    GBA_MID(F, 16, 9);                           \
  }
    if (pass == 0) {
      GBA_MID_BITS(true)
    } else {
      GBA_MID_BITS(false)
    }
#undef GBA_MID_BITS
#undef GBA_MID
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gba
