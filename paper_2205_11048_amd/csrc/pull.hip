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
constexpr int kPullTiles = (int)(kRunTile / kPullBlock);   // blocks per 1024-position run tile

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

// A quarter of a 1024-position tile per block, one position per thread.  The
// run number of position p is the number of run heads at positions <= p,
// minus one (the last position's gives U): the heads before the tile, those in
// the tile's earlier quarters (their keys read again here), and the block's
// own.  The block then gathers the rows of the runs that begin in it, LPR
// lanes and 16-byte accesses per row, four rows in flight per lane group.
// One launch instead of a map and a gather: 256,000 IDs (72,000 distinct, D =
// 32) 9.2 us against 6.8 + 5.6, 26,624 (15,500, D = 64) 5.2 against 5.0 + 3.3,
// and a launch less on a busy stream each.
template <int LPR>
__global__ void __launch_bounds__(kPullBlock)
pull_rows_kernel(PullArgs a, RunHeads heads) {
  constexpr int G = kPullBlock / LPR;
  constexpr int kRows = 4;
  __shared__ uint32_t s_heads[kPullWaves];     // heads of the block's waves
  __shared__ uint32_t s_earlier[kPullWaves];   // heads of the tile's earlier quarters, per wave
  __shared__ uint32_t s_group[kPullWaves];
  __shared__ uint32_t s_key[kPullBlock];       // IDs of the runs that begin in the block
  const int w = threadIdx.x / kWave;
  const int lane = lane_id();
  const int64_t tile = blockIdx.x / kPullTiles;
  const int sub = (int)(blockIdx.x % kPullTiles);
  const int64_t p = (int64_t)blockIdx.x * kPullBlock + threadIdx.x;
  const int64_t last = a.n - 1;
  const bool valid = p <= last;
  // every load is clamped, not branched around, so that all are in flight together
  const int64_t pc = valid ? p : last;
  const uint32_t key = a.keys[pc], kprev = a.keys[pc > 0 ? pc - 1 : 0], j = a.vals[pc];
  uint32_t ek[kPullTiles - 1], ep[kPullTiles - 1];
#pragma unroll
  for (int s = 0; s < kPullTiles - 1; ++s) {
    const int64_t q = tile * kRunTile + s * kPullBlock + threadIdx.x;
    const int64_t qc = q < last ? q : last;
    ek[s] = a.keys[qc];
    ep[s] = a.keys[qc > 0 ? qc - 1 : 0];
  }
  const uint32_t tile_prefix = heads.tile_prefix[tile];
  run_base(heads, tile, s_group);
  uint32_t earlier = 0;
#pragma unroll
  for (int s = 0; s < kPullTiles - 1; ++s) {
    const int64_t q = tile * kRunTile + s * kPullBlock + threadIdx.x;   // an earlier quarter is whole
    earlier += (s < sub && (q == 0 || ek[s] != ep[s])) ? 1u : 0u;
  }
  earlier = wave_sum(earlier);
  const bool head = valid && (p == 0 || key != kprev);
  const uint64_t hm = __ballot(head);
  if (lane == 0) {
    s_earlier[w] = earlier;
    s_heads[w] = (uint32_t)__popcll(hm);
  }
  __syncthreads();
  uint32_t first = tile_prefix + run_base_sum(s_group);   // runs that begin before the block
  uint32_t mine = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kPullWaves; ++k) {
    first += s_earlier[k];
    if (k < w) mine += s_heads[k];
    all += s_heads[k];
  }
  mine += (uint32_t)__popcll(hm & lanemask_lt());          // runs that begin in the block before this position
  const int64_t run = (int64_t)first + mine + (head ? 1 : 0) - 1;
  if (valid && run >= 0 && run < a.n && (int64_t)j < a.n) {   // always true when the numbering is consistent
    a.inverse[j] = (int32_t)run;
    if (head) a.unique_ids[run] = (int64_t)key;
    if (p == last) *a.num_unique = run + 1;
  }
  if (head) s_key[mine] = key;
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
      if (h0 + k * G < all) *reinterpret_cast<f32x4*>(a.rows + ((int64_t)first + h0 + k * G) * a.D + gl * 4) = v[k];
  }
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
  const dim3 grid((unsigned)ceil_div(a.n, kPullBlock));
#define GBA_GATHER_CASE(LPR_)                                                                          \
  case LPR_:                                                                                           \
    hipLaunchKernelGGL((pull_rows_kernel<LPR_>), grid, dim3(kPullBlock), 0, stream, a, heads);          \
    break;
  switch (lpr) {
    GBA_GATHER_CASE(1)
    GBA_GATHER_CASE(2)
    GBA_GATHER_CASE(4)
    GBA_GATHER_CASE(8)
    GBA_GATHER_CASE(16)
    GBA_GATHER_CASE(32)
    GBA_GATHER_CASE(64)
    default:
      return hipErrorInvalidValue;
  }
#undef GBA_GATHER_CASE
  return hipGetLastError();
}

}  // namespace gba
