// Pull side of the PS (Alg. 2, pull responder): a worker sends the embedding
// IDs of its batch and receives their parameters.  The rows are looked up once
// per distinct ID: the request's IDs are sorted (the push path's radix sort),
// runs of equal IDs are numbered, every request position learns the number of
// its ID's run (the inverse map), and one row per distinct ID is gathered.  The
// worker expands rows[inverse[i]] locally, so a Zipf-skewed request moves
// U rows instead of n.
#include <algorithm>

#include "gba_device.hpp"
#include "gba_internal.hpp"
#include "run_heads.hpp"

namespace gba {

constexpr int kPullBlock = 256;
constexpr int kPullWaves = kPullBlock / kWave;
constexpr int kPullTiles = (int)(kRunTile / kPullBlock);   // quarters of a 1024-position run tile
constexpr int64_t kPullSplitFrom = int64_t(1) << 25;       // request IDs from which map and gather are two launches
constexpr int64_t kGatherMaxBlocks = 4096;

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

struct PullLayout {
  size_t off_tile, off_group, bytes;
};

static PullLayout pull_layout(int64_t n) {
  PullLayout L{};
  const size_t tiles = (size_t)(n > 0 ? ceil_div(n, kRunTile) : 1);
  size_t o = 0;
  L.off_tile = o;  o += align_up(tiles * 4);
  // (the groups grow fourfold at 4096 tiles: their counts keep the room of the smaller sizes)
  L.off_group = o; o += align_up((size_t)std::max(run_groups(n), std::min<int64_t>((int64_t)tiles / 4, 1024)) * 4);
  L.bytes = o;
  return L;
}

size_t pull_workspace_bytes(int64_t n) { return pull_layout(n).bytes; }

__global__ void pull_empty_kernel(int64_t* __restrict__ num_unique) { *num_unique = 0; }

// PER positions per thread: a quarter of a 1024-position tile per block (PER =
// 1) or a whole one (4), each wave's positions in a row (their places in the
// inverse map then share more lines: 25 M positions of 65,536 IDs 344 us for the
// map, 526 with 256 positions between a thread's).  The run number of position p is the
// number of run heads at positions <= p, minus one (the last position's gives
// U): the heads before the tile, those in the tile's earlier quarters (their
// keys read again here), and the block's own.  The block then gathers the rows
// of the runs that begin in it, LPR lanes and 16-byte accesses per row, four
// rows in flight per lane group (not with LPR = 0).  One launch instead of a
// map and a gather: 256,000 IDs (72,000 distinct, D = 32) 9.2 us against 6.8 +
// 5.6, 26,624 (15,500, D = 64) 5.2 against 5.0 + 3.3, and a launch less on a
// busy stream each.
template <int LPR, int PER>
__global__ void __launch_bounds__(kPullBlock)
pull_rows_kernel(PullArgs a, RunHeads heads) {
  constexpr int kEarlier = PER == 1 ? kPullTiles - 1 : 0;   // most quarters of the tile before the block's
  static_assert(PER == 1 || PER == kPullTiles, "a quarter or a whole tile");
  __shared__ uint32_t s_heads[kPullWaves];        // heads of the block's waves
  __shared__ uint32_t s_earlier[kPullWaves];      // heads of the tile's earlier quarters, per wave
  __shared__ uint32_t s_group[kPullWaves];
  __shared__ uint32_t s_key[LPR ? PER * kPullBlock : 1];   // IDs of the runs that begin in the block
  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  const int64_t p0 = (int64_t)blockIdx.x * (PER * kPullBlock) + w * (PER * kWave) + lane;
  const int64_t tile = p0 / kRunTile;
  const int64_t last = a.n - 1;
  // every load is clamped, not branched around, so that all are in flight together
  uint32_t key[PER], kprev[PER], j[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int64_t p = p0 + r * kWave;
    const int64_t pc = p < last ? p : last;
    key[r] = a.keys[pc];
    kprev[r] = a.keys[pc > 0 ? pc - 1 : 0];
    j[r] = a.vals[pc];
  }
  uint32_t ek[kEarlier + 1], ep[kEarlier + 1];
#pragma unroll
  for (int s = 0; s < kEarlier; ++s) {
    const int64_t q = tile * kRunTile + s * kPullBlock + threadIdx.x;
    const int64_t qc = q < last ? q : last;
    ek[s] = a.keys[qc];
    ep[s] = a.keys[qc > 0 ? qc - 1 : 0];
  }
  const uint32_t tile_prefix = heads.tile_prefix[tile];
  run_base(heads, tile, s_group);
  uint32_t earlier = 0;
#pragma unroll
  for (int s = 0; s < kEarlier; ++s) {
    const int64_t q = tile * kRunTile + s * kPullBlock + threadIdx.x;   // an earlier quarter is whole
    earlier += (s < (int)(blockIdx.x % kPullTiles) && (q == 0 || ek[s] != ep[s])) ? 1u : 0u;
  }
  if (kEarlier > 0) earlier = wave_sum(earlier);
  uint64_t hm[PER];
  uint32_t heads_w = 0;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int64_t p = p0 + r * kWave;
    hm[r] = __ballot(p <= last && (p == 0 || key[r] != kprev[r]));
    heads_w += (uint32_t)__popcll(hm[r]);
  }
  if (lane == 0) {
    s_earlier[w] = earlier;
    s_heads[w] = heads_w;
  }
  __syncthreads();
  uint32_t first = tile_prefix + run_base_sum(s_group);   // runs that begin before the block
#pragma unroll
  for (int k = 0; k < kPullWaves; ++k) first += s_earlier[k];
  uint32_t before = 0, all = 0;   // runs that begin in the block before the wave's round, and in all
#pragma unroll
  for (int k = 0; k < kPullWaves; ++k) {
    if (k < w) before += s_heads[k];
    all += s_heads[k];
  }
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int64_t p = p0 + r * kWave;
    const uint32_t mine = before + (uint32_t)__popcll(hm[r] & lanemask_lt());   // ... before this position
    const bool head = (hm[r] >> lane) & 1ull;
    const int64_t run = (int64_t)first + mine + (head ? 1 : 0) - 1;
    if (p <= last && run >= 0 && run < a.n && (int64_t)j[r] < a.n) {   // always true when the numbering is consistent
      a.inverse[j[r]] = (int32_t)run;
      if (head) a.unique_ids[run] = (int64_t)key[r];
      if (p == last) *a.num_unique = run + 1;
    }
    if (LPR && head) s_key[mine] = key[r];
    before += (uint32_t)__popcll(hm[r]);
  }
  if constexpr (LPR > 0) {
    constexpr int G = kPullBlock / LPR;
    constexpr int kRows = 4;
    __syncthreads();
    const int gl = threadIdx.x % LPR;
    const int grp = threadIdx.x / LPR;
    if (gl * 4 >= a.D || (int64_t)first + all > a.n) return;   // no barrier follows
    for (uint32_t h0 = grp; h0 < all; h0 += kRows * G) {
      f32x4 v[kRows];
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const uint32_t h = h0 + k * G < all ? h0 + k * G : all - 1;
        const int64_t r = (int64_t)s_key[h] < a.R ? (int64_t)s_key[h] : 0;   // the IDs were range-checked by the sort
        v[k] = *reinterpret_cast<const f32x4*>(a.table + r * a.D + gl * 4);
      }
#pragma unroll
      for (int k = 0; k < kRows; ++k)
        if (h0 + k * G < all)
          *reinterpret_cast<f32x4*>(a.rows + ((int64_t)first + h0 + k * G) * a.D + gl * 4) = v[k];
    }
  }
}

// rows[s] = table[unique_ids[s]] for every distinct ID: a lane group per row,
// a fixed grid (their number is on the device).
template <int LPR>
__global__ void __launch_bounds__(kPullBlock)
pull_gather_kernel(PullArgs a) {
  constexpr int G = kPullBlock / LPR;
  const int gl = threadIdx.x % LPR;
  if (gl * 4 >= a.D) return;
  const int64_t U = *a.num_unique < a.n ? *a.num_unique : a.n;
  for (int64_t s = (int64_t)blockIdx.x * G + threadIdx.x / LPR; s < U; s += (int64_t)gridDim.x * G) {
    const int64_t id = a.unique_ids[s];
    const int64_t r = id >= 0 && id < a.R ? id : 0;   // the IDs were range-checked by the sort
    *reinterpret_cast<f32x4*>(a.rows + s * a.D + gl * 4) =
        *reinterpret_cast<const f32x4*>(a.table + r * a.D + gl * 4);
  }
}

// A quarter of a tile per block, so that small requests have blocks for every
// compute unit and wide rows more of them in flight (3.2 M IDs, D = 128 426 us,
// 464 with whole tiles); a whole tile, whose group's runs are then counted once
// and not four times, for rows of up to 16 floats from 2^19 IDs (600,000, D = 16
// 45 and 44 us, 10 M 319 and 262) and of up to 32 from 3 * 2^20 (10 M 404 and 383,
// but 1.5 M 154 and 161).  From 2^25 IDs the map, whose scattered stores the
// gather's loads would wait behind, is a launch of its own (40 M, D = 32 2390 us in
// one launch, 2099 in two; 17 M 1133 and 1168).
template <int LPR>
static hipError_t launch_pull_rows(const PullArgs& a, const RunHeads& heads, hipStream_t stream) {
  const dim3 quarters((unsigned)ceil_div(a.n, kPullBlock)), tiles((unsigned)ceil_div(a.n, kRunTile)), block(kPullBlock);
  if (a.n >= kPullSplitFrom) {
    hipLaunchKernelGGL((pull_rows_kernel<0, kPullTiles>), tiles, block, 0, stream, a, heads);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pull_gather_kernel<LPR>, dim3((unsigned)kGatherMaxBlocks), block, 0, stream, a);
    return hipGetLastError();
  }
  if constexpr (LPR <= 8) {
    if (a.n >= (LPR <= 4 ? int64_t(1) << 19 : int64_t(3) << 20)) {
      hipLaunchKernelGGL((pull_rows_kernel<LPR, kPullTiles>), tiles, block, 0, stream, a, heads);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((pull_rows_kernel<LPR, 1>), quarters, block, 0, stream, a, heads);
  return hipGetLastError();
}

hipError_t launch_pull(const PullArgs& a, void* ws, hipStream_t stream) {
  const PullLayout L = pull_layout(a.n);
  char* base = static_cast<char*>(ws);
  if (a.n <= 0) {
    hipLaunchKernelGGL(pull_empty_kernel, dim3(1), dim3(1), 0, stream, a.num_unique);
    return hipGetLastError();
  }
  RunHeads heads;
  hipError_t e = launch_run_heads(a.keys, a.n, reinterpret_cast<uint32_t*>(base + L.off_tile),
                                  reinterpret_cast<uint32_t*>(base + L.off_group), &heads, stream);
  if (e != hipSuccess) return e;
  int lpr = 1;
  while (lpr < 64 && lpr * 4 < a.D) lpr <<= 1;
  switch (lpr) {
    case 1: return launch_pull_rows<1>(a, heads, stream);
    case 2: return launch_pull_rows<2>(a, heads, stream);
    case 4: return launch_pull_rows<4>(a, heads, stream);
    case 8: return launch_pull_rows<8>(a, heads, stream);
    case 16: return launch_pull_rows<16>(a, heads, stream);
    case 32: return launch_pull_rows<32>(a, heads, stream);
    case 64: return launch_pull_rows<64>(a, heads, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gba
