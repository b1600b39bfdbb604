// Tile binning: per-tile, depth-ordered Gaussian lists.
//
// The ray list of Eq. 1 is the depth-ordered sequence of Gaussians covering
// the pixel; as in 3D-GS it is built per 16x16 tile. Instead of one global
// sort of (tile, depth) keys this is a bucket sort by tile followed by an
// independent sort of each tile's bucket:
//   1. count: every (Gaussian, covered tile) pair increments its tile's
//      counter (each wave spreads one Gaussian's tiles over its lanes);
//   2. exclusive scan of the counts -> tile_offsets (CSR) and the pair count;
//   3. scatter: each pair claims a slot in its tile's bucket with an atomic
//      cursor and stores the 64-bit key (float bits of depth << 32 | id);
//   4. sort: one workgroup per tile sorts its bucket. The keys are unique
//      (they contain the id), so the result is the exact (depth, id) order
//      whatever order step 3 produced. Buckets of up to kSortItems keys are
//      bitonic-sorted in registers (lane exchanges inside a wave, LDS across
//      waves); longer ones take a single-workgroup LSD radix sort through a
//      workspace segment.
// Counters and cursors are in LDS: a view's records are cut into chunks, one
// workgroup counts a chunk's pairs over the view's whole tile grid, the
// chunks' counts are scanned per tile, and in the scatter a workgroup's
// cursors start where its chunk's pairs begin in each tile. (Counters in
// global memory, one atomic per pair and pass, ran at the rate of atomics at
// memory: 16 views of 200k Gaussians at 640x480: count 125 -> 24 us, scatter
// 144 -> 58 us, which the scattered 8-byte key stores bound now.) Grids too large for LDS keep global counters.
// Depth is positive (z > z_near > 0), so its IEEE bit pattern orders like
// the value. No kernel synchronises with the host: grids are sized by the
// caller's capacity and every kernel reads the pair count from device memory.
#include <algorithm>
#include <mutex>

#include "common.h"

namespace qr {

constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 8;
constexpr int kScanItems = kScanThreads * kScanPerThread;  // 2048
// Keys of a tile sorted in registers (eight per thread), exchanged through 16
// KB. (Beside three resident renderer workgroups a CU has 10 KB and 56
// registers a lane left, so neither the sort nor the chunk kernels run there:
// binning beside a persistent render starts as that drains. Made to fit, with
// 256-thread chunk workgroups and an 8 KB exchange buffer, a step of 16 views
// took 2.147 instead of 2.154 ms overlapped, and up to 2.50 where the small
// workgroups' LDS leaves a renderer none in one piece; binning alone took 25%
// to 32% longer: 4 views of 1M records 153 against 127 us.)
constexpr int kSortItems = 2048;
constexpr int kRadix = 256;

// ---- device-wide exclusive scan (u32) --------------------------------------
__global__ void __launch_bounds__(kScanThreads)
scan_reduce_kernel(const uint32_t* __restrict__ in, int64_t n, uint32_t* __restrict__ part) {
  __shared__ uint32_t lds4[4];
  const int64_t base = blockIdx.x * static_cast<int64_t>(kScanItems);
  uint32_t s = 0;
  for (int j = 0; j < kScanPerThread; ++j) {
    const int64_t i = base + j * kScanThreads + threadIdx.x;
    if (i < n) s += in[i];
  }
  uint32_t total;
  block_scan_exclusive(s, lds4, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// one block scans the block sums in chunks; part[nb] = out_total[0] = total
// (out_total2 receives a second copy when given)
__global__ void __launch_bounds__(kScanThreads)
scan_top_kernel(uint32_t* __restrict__ part, int64_t nb, uint32_t* __restrict__ out_total,
                uint32_t* __restrict__ out_total2) {
  __shared__ uint32_t lds4[4];
  uint32_t carry = 0;
  for (int64_t c = 0; c < nb; c += kScanThreads) {
    const int64_t i = c + threadIdx.x;
    const uint32_t v = i < nb ? part[i] : 0u;
    uint32_t total;
    const uint32_t ex = block_scan_exclusive(v, lds4, &total);
    if (i < nb) part[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) {
    part[nb] = carry;
    *out_total = carry;
    if (out_total2) *out_total2 = carry;
  }
}

__global__ void __launch_bounds__(kScanThreads)
scan_down_kernel(const uint32_t* __restrict__ in, int64_t n, const uint32_t* __restrict__ part,
                 uint32_t* __restrict__ out) {
  __shared__ uint32_t lds4[4];
  const int64_t base = blockIdx.x * static_cast<int64_t>(kScanItems) +
                       threadIdx.x * static_cast<int64_t>(kScanPerThread);
  uint32_t v[kScanPerThread];
  uint32_t s = 0;
  for (int j = 0; j < kScanPerThread; ++j) {
    const int64_t i = base + j;
    v[j] = i < n ? in[i] : 0u;
    s += v[j];
  }
  uint32_t run = part[blockIdx.x] + block_scan_exclusive(s, lds4, nullptr);
  for (int j = 0; j < kScanPerThread; ++j) {
    const int64_t i = base + j;
    if (i < n) out[i] = run;
    run += v[j];
  }
}

// Exclusive scan of one value per thread over a workgroup of 1,024 (16
// waves; lds16: 16 words). Every thread must call it.
constexpr int kWideThreads = 1024;
__device__ __forceinline__ uint32_t wide_scan_exclusive(uint32_t v, uint32_t* lds16, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(inc, off, 64);
    if (lane >= off) inc += t;
  }
  if (lane == 63) lds16[wave] = inc;
  __syncthreads();
  uint32_t base = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const uint32_t x = lds16[w];
    base += w < wave ? x : 0u;
    sum += x;
  }
  *total = sum;
  return base + inc - v;
}

// The whole scan in one workgroup, for short arrays (the per-tile counters of
// an image or a batch): one launch instead of three, the values held in
// registers between the two halves. out[n] = total (and *total2 if given).
// (19,200 entries: 24 -> 10 us against 256 threads with a carry.)
constexpr int kWidePerThread = 32;
__global__ void __launch_bounds__(kWideThreads)
scan_small_kernel(const uint32_t* __restrict__ in, int n, uint32_t* __restrict__ out,
                  uint32_t* __restrict__ total2) {
  __shared__ uint32_t lds16[16];
  // a wave's values lie together, lanes side by side: value j of a lane is
  // 64 j after its first
  const int per = (n + kWideThreads - 1) / kWideThreads;
  const int lane = threadIdx.x & 63, first = (threadIdx.x >> 6) * 64 * per;
  uint32_t v[kWidePerThread];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kWidePerThread; ++j) {
    const int i = first + 64 * j + lane;
    v[j] = j < per && i < n ? in[i] : 0u;
    s += v[j];
  }
  // the wave's base: scan of the lanes' sums gives the total before the wave
  uint32_t total;
  uint32_t run = wide_scan_exclusive(s, lds16, &total);
  run = __builtin_amdgcn_readfirstlane(run);  // lane 0: everything before the wave
#pragma unroll
  for (int j = 0; j < kWidePerThread; ++j) {
    if (j >= per) break;  // uniform
    const uint32_t x = v[j];
    uint32_t inc = x;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t t = __shfl_up(inc, off, 64);
      if (lane >= off) inc += t;
    }
    const int i = first + 64 * j + lane;
    if (i < n) out[i] = run + inc - x;
    run += __builtin_amdgcn_readlane(inc, 63);
  }
  if (threadIdx.x == 0) {
    out[n] = total;
    if (total2) *total2 = total;
  }
}

constexpr int64_t kSmallScanMax = kWideThreads * kWidePerThread;  // 32768 entries

static int64_t scan_parts(int64_t n) { return std::max<int64_t>(ceil_div(n, kScanItems), 1); }

// out[0..n) = exclusive scan of in, out[n] = total (and *total2 if given).
// `part` needs scan_parts(n) + 1 entries; in and out must not overlap.
static void scan_exclusive(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* part,
                           uint32_t* total2, hipStream_t s) {
  if (n <= kSmallScanMax) {
    hipLaunchKernelGGL(scan_small_kernel, dim3(1), dim3(kWideThreads), 0, s, in, static_cast<int>(n), out,
                       total2);
    return;
  }
  const int64_t nb = scan_parts(n);
  hipLaunchKernelGGL(scan_reduce_kernel, dim3(static_cast<unsigned>(nb)), dim3(kScanThreads), 0, s,
                     in, n, part);
  hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(kScanThreads), 0, s, part, nb, out + n, total2);
  hipLaunchKernelGGL(scan_down_kernel, dim3(static_cast<unsigned>(nb)), dim3(kScanThreads), 0, s,
                     in, n, part, out);
}

// ---- bucket by tile: counters in LDS -----------------------------------------
// The pairs of 64 consecutive records of a view, called by a whole wave: a
// lane visits the tiles of its own record if there are at most kOwnTiles (no
// division, 64 records side by side; neighbouring lanes start from different
// corners, so that records of one rectangle meet less on its counters: 4,096
// records over all of 16 tiles, 207 us from one corner, 141 from four); the records with more are visited one
// after the other, their tiles spread over the 64 lanes, so a Gaussian that
// covers a thousand tiles costs sixteen lane-rounds instead of a thousand
// serial iterations of one thread. (All records one after the other: 68 and
// 88 us instead of 24 and 58 for count and scatter of 16 views of 200k
// Gaussians, 52 instead of 5 us for 1,000 in one workgroup; limits of 8 and
// 32 differ from 16 by less than 10 us either way.) cnt, r, d: the lane's record (tile count, rectangle, depth
// bits); pair(tile of the view, key) is called for every pair.
constexpr uint32_t kOwnTiles = 16;
template <class Pair>
__device__ __forceinline__ void for_pairs(uint32_t cnt, const int4& r, uint32_t d, uint32_t id, int tiles_x,
                                          const Pair& pair) {
  const int lane = threadIdx.x & 63;
  if (cnt <= kOwnTiles) {
    const unsigned long long key = (static_cast<unsigned long long>(d) << 32) | id;
    const int w = r.z - r.x, dx = lane & 1 ? -1 : 1;
    const int next_row = (lane & 2 ? -tiles_x : tiles_x) - dx * (w - 1);
    int t = (lane & 2 ? r.w - 1 : r.y) * tiles_x + (lane & 1 ? r.z - 1 : r.x), left = w;
    for (uint32_t k = 0; k < cnt; ++k) {
      pair(t, key);
      const bool wrap = --left == 0;
      t += wrap ? next_row : dx;
      left = wrap ? w : left;
    }
  }
  for (uint64_t todo = __ballot(cnt > kOwnTiles); todo; todo &= todo - 1) {
    const int j = __builtin_ctzll(todo);
    const uint32_t c = __builtin_amdgcn_readlane(cnt, j);
    const int rx = __builtin_amdgcn_readlane(r.x, j), row0 = __builtin_amdgcn_readlane(r.y, j);
    const int w = __builtin_amdgcn_readlane(r.z, j) - rx;
    const unsigned long long key =
        (static_cast<unsigned long long>(static_cast<uint32_t>(__builtin_amdgcn_readlane(d, j))) << 32) |
        static_cast<uint32_t>(__builtin_amdgcn_readlane(id, j));
    for (uint32_t k = lane; k < c; k += 64)
      pair((row0 + static_cast<int>(k) / w) * tiles_x + rx + static_cast<int>(k) % w, key);
  }
}

// Records [first, last) by a workgroup of kWideThreads. The next records' tile
// counts are requested before the current ones are visited. place(i, r): the
// id in record i's keys; may move its rectangle.
template <bool kDepth, class Place, class Pair>
__device__ __forceinline__ void for_records(int64_t first, int64_t last, const int4* __restrict__ rect,
                                            const uint32_t* __restrict__ touched, const float* __restrict__ depth,
                                            int tiles_x, const Place& place, const Pair& pair) {
  int64_t i = first + threadIdx.x;
  uint32_t next = i < last ? touched[i] : 0u;
  for (int64_t w0 = first + (threadIdx.x & ~63); w0 < last; w0 += kWideThreads, i += kWideThreads) {
    const uint32_t cnt = next;
    next = i + kWideThreads < last ? touched[i + kWideThreads] : 0u;
    int4 r = make_int4(0, 0, 0, 0);
    uint32_t d = 0, id = 0;
    if (cnt) {
      r = rect[i];
      if (kDepth) d = __float_as_uint(depth[i]);
      id = place(i, r);
    }
    for_pairs(cnt, r, d, id, tiles_x, pair);
  }
}

// The records of chunk c of a view.
template <bool kDepth, class Pair>
__device__ __forceinline__ void for_chunk(int64_t view, int64_t n_per_view, int64_t c, int64_t chunk,
                                          const int4* __restrict__ rect, const uint32_t* __restrict__ touched,
                                          const float* __restrict__ depth, int tiles_x, const Pair& pair) {
  const int64_t base = view * n_per_view;
  for_records<kDepth>(base + c * chunk, base + min((c + 1) * chunk, n_per_view), rect, touched, depth, tiles_x,
                      [&](int64_t i, int4&) { return static_cast<uint32_t>(i - base); }, pair);
}

// Workgroup b takes chunk b % n_chunks of view b / n_chunks. counts:
// [view][chunk][tile of the view].
__global__ void __launch_bounds__(kWideThreads)
chunk_count_kernel(int64_t n_per_view, int n_chunks, int64_t chunk, const int4* __restrict__ rect,
                   const uint32_t* __restrict__ touched, int tiles_x, int n_tiles,
                   uint32_t* __restrict__ counts) {
  extern __shared__ uint32_t h[];
  for (int t = threadIdx.x; t < n_tiles; t += kWideThreads) h[t] = 0u;
  __syncthreads();
  const int64_t view = blockIdx.x / n_chunks, c = blockIdx.x % n_chunks;
  for_chunk<false>(view, n_per_view, c, chunk, rect, touched, nullptr, tiles_x,
                   [&](int t, unsigned long long) { atomicAdd(&h[t], 1u); });
  __syncthreads();
  uint32_t* const out = counts + static_cast<int64_t>(blockIdx.x) * n_tiles;
  for (int t = threadIdx.x; t < n_tiles; t += kWideThreads) out[t] = h[t];
}

// Per tile: exclusive scan of its chunks' counts, in place, and their sum. 64
// tiles per workgroup, a wave per eighth of the chunks, held in registers.
constexpr int kMaxChunks = 256;
__global__ void __launch_bounds__(512)
chunk_scan_kernel(int64_t total_tiles, int n_tiles, int n_chunks, uint32_t* __restrict__ counts,
                  uint32_t* __restrict__ tile_counts) {
  __shared__ uint32_t sum[8][64];
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  const int64_t g = blockIdx.x * 64LL + lane;
  const int per = (n_chunks + 7) >> 3, c0 = part * per, c1 = min(c0 + per, n_chunks);
  const bool live = g < total_tiles;
  const int64_t view = live ? g / n_tiles : 0;
  uint32_t* const at = counts + view * n_chunks * n_tiles + (g - view * n_tiles);
  uint32_t v[kMaxChunks / 8];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kMaxChunks / 8; ++k) {
    v[k] = live && c0 + k < c1 ? at[static_cast<int64_t>(c0 + k) * n_tiles] : 0u;
    s += v[k];
  }
  sum[part][lane] = s;
  __syncthreads();
  uint32_t run = 0;
  for (int p = 0; p < part; ++p) run += sum[p][lane];
#pragma unroll
  for (int k = 0; k < kMaxChunks / 8; ++k) {
    if (live && c0 + k < c1) at[static_cast<int64_t>(c0 + k) * n_tiles] = run;
    run += v[k];
  }
  if (live && part == 7) tile_counts[g] = run;
}

__global__ void __launch_bounds__(kWideThreads)
chunk_scatter_kernel(int64_t n_per_view, int n_chunks, int64_t chunk, const int4* __restrict__ rect,
                     const uint32_t* __restrict__ touched, const float* __restrict__ depth, int tiles_x,
                     int n_tiles, const uint32_t* __restrict__ counts, const uint32_t* __restrict__ offsets,
                     int64_t capacity, unsigned long long* __restrict__ bucket) {
  extern __shared__ uint32_t h[];
  const int64_t view = blockIdx.x / n_chunks, c = blockIdx.x % n_chunks;
  const uint32_t* const before = counts + static_cast<int64_t>(blockIdx.x) * n_tiles;
  for (int t = threadIdx.x; t < n_tiles; t += kWideThreads) h[t] = offsets[view * n_tiles + t] + before[t];
  __syncthreads();
  for_chunk<true>(view, n_per_view, c, chunk, rect, touched, depth, tiles_x, [&](int t, unsigned long long key) {
    const int64_t slot = atomicAdd(&h[t], 1u);
    if (slot < capacity) bucket[slot] = key;
  });
}

// Small scenes: count, scan and scatter in one workgroup and one launch (1,000
// Gaussians on 16 tiles: 4.7 us against 14.5 us in four launches). The records
// of all views are taken side by side, whatever their number (view after view
// cost a memory round trip for each: 64 views of 64 on 16 tiles, 80 us, now 16;
// 1,024 of 16 on 4 tiles, 730 and 27). The limits on records and on records
// times tiles keep it to a few records per thread on a small grid, and to few
// records on a large one (65,536 records in 4,096 one-tile views: 78 us here,
// 36 in chunks).
constexpr int kSmallTiles = 4 * kWideThreads;  // four tiles per thread in the scan
constexpr int64_t kSmallWork = 1 << 16;  // records times tiles of a view
constexpr int64_t kSmallRecords = 16 * kWideThreads;
__global__ void __launch_bounds__(kWideThreads)
bucket_small_kernel(int n, int n_per_view, const int4* __restrict__ rect, const uint32_t* __restrict__ touched,
                    const float* __restrict__ depth, int tiles_x, int tiles_y, int all, int64_t capacity,
                    uint32_t* __restrict__ tile_offsets, uint32_t* __restrict__ total_pairs,
                    unsigned long long* __restrict__ bucket) {
  __shared__ uint32_t h[kSmallTiles];
  __shared__ uint32_t lds16[16];
  for (int t = threadIdx.x; t < kSmallTiles; t += kWideThreads) h[t] = 0u;
  __syncthreads();
  const auto place = [&](int64_t i, int4& r) {  // into the stacked grid of all views
    const int view = static_cast<int>(i) / n_per_view;
    r.y += view * tiles_y;
    r.w += view * tiles_y;
    return static_cast<uint32_t>(static_cast<int>(i) - view * n_per_view);
  };
  for_records<false>(0, n, rect, touched, nullptr, tiles_x, place,
                     [&](int t, unsigned long long) { atomicAdd(&h[t], 1u); });
  __syncthreads();
  const int t0 = 4 * threadIdx.x;
  uint32_t c[4];
  uint32_t s = 0, total;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    c[k] = h[t0 + k];
    s += c[k];
  }
  uint32_t run = wide_scan_exclusive(s, lds16, &total);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    h[t0 + k] = run;
    if (t0 + k < all) tile_offsets[t0 + k] = run;
    run += c[k];
  }
  if (threadIdx.x == 0) {
    tile_offsets[all] = total;
    *total_pairs = total;
  }
  if (capacity == 0) return;
  __syncthreads();
  for_records<true>(0, n, rect, touched, depth, tiles_x, place, [&](int t, unsigned long long key) {
    const int64_t slot = atomicAdd(&h[t], 1u);
    if (slot < capacity) bucket[slot] = key;
  });
}

// ---- bucket by tile: counters in global memory --------------------------------
// For grids whose counters do not fit in LDS, or workspaces without room for
// enough chunks' counts.
__global__ void __launch_bounds__(256)
zero_u32_kernel(uint32_t* __restrict__ a, int64_t n) {
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x) a[i] = 0u;
}

// Each wave takes 64 consecutive projected records and visits them one
// after the other; the covered tiles of the current record are spread over
// the 64 lanes, so a Gaussian that covers a thousand tiles costs sixteen
// lane-rounds instead of a thousand serial iterations of one thread, and no
// per-pair index (and no scan of per-record pair counts) is needed.
// Records come in views of n_per_view (record i is Gaussian i % n_per_view
// seen from view i / n_per_view); view v's tile grid is stacked below view
// v-1's (tile rows v*tiles_y ..), and the key carries the view-local id.
template <bool kScatter>
__global__ void __launch_bounds__(256)
tile_pairs_kernel(int64_t n, int64_t n_per_view, const int4* __restrict__ rect,
                  const uint32_t* __restrict__ touched, const float* __restrict__ depth,
                  int tiles_x, int tiles_y, uint32_t* __restrict__ cnt,
                  const uint32_t* __restrict__ offsets, int64_t capacity,
                  unsigned long long* __restrict__ bucket) {
  const int lane = threadIdx.x & 63;
  const int64_t base = (blockIdx.x * 256LL + threadIdx.x) - lane;  // first Gaussian of this wave
  const int64_t mine = base + lane;
  uint32_t my_cnt = 0;
  int4 my_r = make_int4(0, 0, 0, 0);
  uint32_t my_d = 0;
  int my_row0 = 0;       // first stacked tile row of this record's footprint
  uint32_t my_local = 0;  // view-local Gaussian id
  if (mine < n) {
    my_cnt = touched[mine];
    if (my_cnt) {
      my_r = rect[mine];
      if (kScatter) my_d = __float_as_uint(depth[mine]);
      const int64_t view = mine / n_per_view;
      my_local = static_cast<uint32_t>(mine - view * n_per_view);
      my_row0 = static_cast<int>(view) * tiles_y + my_r.y;
    }
  }
  unsigned long long todo = __ballot(my_cnt != 0);
  while (todo) {
    const int j = __ffsll(static_cast<long long>(todo)) - 1;
    todo &= todo - 1;
    const uint32_t c = __shfl(my_cnt, j, 64);
    const int rx = __shfl(my_r.x, j, 64), rz = __shfl(my_r.z, j, 64);
    const int row0 = __shfl(my_row0, j, 64);
    const int w = rz - rx;
    const unsigned long long key = kScatter
        ? ((static_cast<unsigned long long>(__shfl(my_d, j, 64)) << 32) | __shfl(my_local, j, 64))
        : 0ull;
    for (uint32_t k = lane; k < c; k += 64) {
      const int t = (row0 + static_cast<int>(k) / w) * tiles_x + rx + static_cast<int>(k) % w;
      if (kScatter) {
        const int64_t slot = static_cast<int64_t>(offsets[t]) + atomicAdd(&cnt[t], 1u);
        if (slot < capacity) bucket[slot] = key;
      } else {
        atomicAdd(&cnt[t], 1u);
      }
    }
  }
}

// ---- per-tile sort -------------------------------------------------------------
// Stable scatter of one round of 256 keys (thread order) by an 8-bit digit:
// rank among equal digits within the wave from eight ballots, across waves
// from per-wave digit counts. `run` holds each digit's next output position.
__device__ __forceinline__ void stable_scatter_round(bool valid, unsigned long long key, int shift,
                                                     uint32_t* run, uint32_t (*wcnt)[kRadix],
                                                     unsigned long long* __restrict__ dst) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint32_t digit = valid ? static_cast<uint32_t>(key >> shift) & 0xFFu : 0u;
  unsigned long long eq = __ballot(valid);
  for (int b = 0; b < 8; ++b) {
    const bool bit = (digit >> b) & 1u;
    const unsigned long long m = __ballot(valid && bit);
    eq &= bit ? m : ~m;
  }
  const uint32_t rank = __popcll(eq & ((1ull << lane) - 1ull));
  if (valid && rank == 0) wcnt[wave][digit] = __popcll(eq);
  __syncthreads();
  if (valid) {
    uint32_t pos = run[digit] + rank;
    for (int w = 0; w < wave; ++w) pos += wcnt[w][digit];
    dst[pos] = key;
  }
  __syncthreads();
  run[threadIdx.x] += wcnt[0][threadIdx.x] + wcnt[1][threadIdx.x] + wcnt[2][threadIdx.x] +
                      wcnt[3][threadIdx.x];
  for (int w = 0; w < 4; ++w) wcnt[w][threadIdx.x] = 0;
  __syncthreads();
}

// Bitonic sort of 256 R keys, R per thread: element r * 256 + tid is key[r]
// of thread tid. Steps at a distance of 256 and more stay in the thread's
// registers, below 64 they are exchanges between lanes on the vector ALU
// (DPP moves and row swaps; with lane shuffles through the LDS crossbar and
// whole bitonic stages in LDS, the sort of 16 views of 200k Gaussians took 98
// us, now 44; of longer lists, 500k Gaussians at 960x720, 298 and 142), and only distances 64 and 128 go through LDS.
template <int kCtrl>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(v), kCtrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(v >> 32), kCtrl, 0xF, 0xF, false);
  return (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo);
}

// a, b: the two elements of the lane's pair at lane distance J, in either
// order (the same order in both lanes at 16 and 32, else own first).
template <int J>
__device__ __forceinline__ void lane_pair(uint64_t v, uint64_t& a, uint64_t& b) {
  a = v;
  if constexpr (J == 1) b = dpp_u64<0xB1>(v);        // quad_perm [1,0,3,2]
  else if constexpr (J == 2) b = dpp_u64<0x4E>(v);   // quad_perm [2,3,0,1]
  else if constexpr (J == 4) b = dpp_u64<0x1B>(dpp_u64<0x141>(v));  // half mirror, then quad_perm [3,2,1,0]
  else if constexpr (J == 8) b = dpp_u64<0x128>(v);  // rotation by 8 in 16
  else {
    const uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(v >> 32);
    if constexpr (J == 16) {
      const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
      a = (static_cast<uint64_t>(h[0]) << 32) | l[0];
      b = (static_cast<uint64_t>(h[1]) << 32) | l[1];
    } else {
      const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
      a = (static_cast<uint64_t>(h[0]) << 32) | l[0];
      b = (static_cast<uint64_t>(h[1]) << 32) | l[1];
    }
  }
}

// Lanes whose bit J is 0.
template <int J>
constexpr uint64_t lanes_without() {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l)
    if (!(l & J)) m |= 1ull << l;
  return m;
}

// The smaller of a and b in the lanes of `take_min`, the larger in the others.
__device__ __forceinline__ uint64_t pick(uint64_t a, uint64_t b, uint64_t take_min) {
  constexpr int kUlt = 36;
  const uint64_t less = __builtin_amdgcn_uicmpl(a, b, kUlt);
  return __builtin_amdgcn_inverse_ballot_w64(~(less ^ take_min)) ? a : b;
}

template <int K, int J, int R>
__device__ __forceinline__ void bitonic_step(uint64_t (&key)[R], uint64_t* __restrict__ s_key) {
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (J >= 256) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      constexpr int jr = J / 256;
      if (r & jr) continue;
      const bool up = ((r * 256) & K) == 0;  // K > J: the same for both
      const uint64_t a = key[r], b = key[r + jr];
      const bool swap = (b < a) == up;
      key[r] = swap ? b : a;
      key[r + jr] = swap ? a : b;
    }
  } else if constexpr (J >= 64) {
#pragma unroll
    for (int r = 0; r < R; ++r) s_key[r * 256 + tid] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool up = ((r * 256 + wave * 64) & K) == 0, lower = ((wave * 64) & J) == 0;  // uniform
      key[r] = pick(key[r], s_key[r * 256 + (tid ^ J)], up == lower ? ~0ull : 0ull);
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      uint64_t take_min;
      if constexpr (K < 64) take_min = ~(lanes_without<J>() ^ lanes_without<K>());
      else take_min = ((r * 256 + wave * 64) & K) == 0 ? lanes_without<J>() : ~lanes_without<J>();
      uint64_t a, b;
      lane_pair<J>(key[r], a, b);
      key[r] = pick(a, b, take_min);
    }
  }
  if constexpr (J > 1) bitonic_step<K, J / 2, R>(key, s_key);
}

// Stages K, 2K, .. up to the power of two that holds n keys (the keys past n
// are the largest).
template <int K, int R>
__device__ __forceinline__ void bitonic_stages(int n, uint64_t (&key)[R], uint64_t* __restrict__ s_key) {
  if (K / 2 >= n) return;  // uniform
  bitonic_step<K, K / 2, R>(key, s_key);
  if constexpr (K < 256 * R) bitonic_stages<2 * K, R>(n, key, s_key);
}

template <int R>
__device__ __forceinline__ void sort_registers(int n, int64_t lo, unsigned long long tile_hi,
                                               const unsigned long long* __restrict__ bucket,
                                               uint64_t* __restrict__ s_key, uint32_t* __restrict__ sorted_gid,
                                               unsigned long long* __restrict__ sorted_keys) {
  uint64_t key[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * 256 + static_cast<int>(threadIdx.x);
    key[r] = i < n ? bucket[lo + i] : ~0ull;
  }
  bitonic_stages<2, R>(n, key, s_key);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * 256 + static_cast<int>(threadIdx.x);
    if (i >= n) continue;
    sorted_gid[lo + i] = static_cast<uint32_t>(key[r]);
    if (sorted_keys) sorted_keys[lo + i] = tile_hi | (key[r] >> 32);
  }
}

__global__ void __launch_bounds__(256)
tile_sort_kernel(int n_tiles, const uint32_t* __restrict__ offsets, int64_t capacity,
                 int gid_bits, unsigned long long* __restrict__ bucket,
                 unsigned long long* __restrict__ radix_tmp, uint32_t* __restrict__ sorted_gid,
                 unsigned long long* __restrict__ sorted_keys) {
  __shared__ uint64_t s_key[kSortItems];
  __shared__ uint32_t run[kRadix];
  __shared__ uint32_t wcnt[4][kRadix];
  __shared__ uint32_t lds4[4];
  const int t = blockIdx.x;
  const int64_t lo = std::min<int64_t>(offsets[t], capacity);
  const int64_t hi = std::min<int64_t>(offsets[t + 1], capacity);
  const int n = static_cast<int>(hi - lo);
  if (n <= 0) return;
  const unsigned long long tile_hi = static_cast<unsigned long long>(t) << 32;

  if (n <= kSortItems) {
    if (n <= 256) sort_registers<1>(n, lo, tile_hi, bucket, s_key, sorted_gid, sorted_keys);
    else if (n <= 512) sort_registers<2>(n, lo, tile_hi, bucket, s_key, sorted_gid, sorted_keys);
    else if (n <= 1024) sort_registers<4>(n, lo, tile_hi, bucket, s_key, sorted_gid, sorted_keys);
    else sort_registers<8>(n, lo, tile_hi, bucket, s_key, sorted_gid, sorted_keys);
    return;
  }

  // long bucket: LSD radix sort, one workgroup, ping-pong between the bucket
  // and the radix_tmp segment. Digits cover the id bits (0 .. gid_bits-1) and
  // the depth bits (32 .. 63); bits gid_bits .. 31 are zero in every key.
  unsigned long long* src = bucket + lo;
  unsigned long long* dst = radix_tmp + lo;
  const int gid_passes = (gid_bits + 7) / 8;
  const int passes = gid_passes + 4;
  for (int p = 0; p < passes; ++p) {
    const int shift = p < gid_passes ? 8 * p : 32 + 8 * (p - gid_passes);
    run[threadIdx.x] = 0;
    for (int w = 0; w < 4; ++w) wcnt[w][threadIdx.x] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) atomicAdd(&run[(src[i] >> shift) & 0xFF], 1u);
    __syncthreads();
    const uint32_t c = run[threadIdx.x];
    __syncthreads();
    run[threadIdx.x] = block_scan_exclusive(c, lds4, nullptr);
    __syncthreads();
    for (int base = 0; base < n; base += 256) {
      const int i = base + threadIdx.x;
      const bool valid = i < n;
      stable_scatter_round(valid, valid ? src[i] : 0ull, shift, run, wcnt, dst);
    }
    unsigned long long* tmp = src;
    src = dst;
    dst = tmp;
  }
  for (int i = threadIdx.x; i < n; i += 256) {
    const unsigned long long key = src[i];
    sorted_gid[lo + i] = static_cast<uint32_t>(key);
    if (sorted_keys) sorted_keys[lo + i] = tile_hi | (key >> 32);
  }
}

// Tiles of a view whose counters fit in LDS (64 KB: two workgroups per CU).
constexpr int kLdsTiles = 16384;

// ---- workspace layout --------------------------------------------------------
struct Layout {
  size_t cnt, cursor, part, bucket, radix_tmp, bytes;
};

static size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

static Layout layout(int64_t n_tiles, int64_t capacity) {
  Layout L{};
  size_t o = 0;
  L.cnt = o;     o = align256(o + sizeof(uint32_t) * (n_tiles + 1));
  L.cursor = o;  o = align256(o + sizeof(uint32_t) * (n_tiles + 1));
  L.part = o;    o = align256(o + sizeof(uint32_t) * (scan_parts(n_tiles) + 1));
  L.bucket = o;  o = align256(o + sizeof(uint64_t) * std::max<int64_t>(capacity, 1));
  L.radix_tmp = o; o = align256(o + sizeof(uint64_t) * std::max<int64_t>(capacity, 1));
  L.bytes = o;
  return L;
}

static int bits_for(int64_t n) {
  int b = 0;
  while ((1ll << b) < n) ++b;
  return b;
}

}  // namespace qr

using namespace qr;

extern "C" int qr_bin_sort_workspace_size(int64_t n, int32_t tiles_x, int32_t tiles_y,
                                          int64_t capacity, size_t* bytes) {
  if (!bytes) return fail(QR_ERR_INVALID_ARG, "qr_bin_sort_workspace_size: null result pointer");
  if (n < 0 || capacity < 0 || tiles_x <= 0 || tiles_y <= 0)
    return fail(QR_ERR_INVALID_ARG, "qr_bin_sort_workspace_size: bad sizes");
  *bytes = layout(static_cast<int64_t>(tiles_x) * tiles_y, capacity).bytes;
  return QR_OK;
}

// Bins the records of n_views views (n_per_view each) into the stacked tile
// grid of all views: one launch sequence for the whole batch.
static int bin_sort_impl(const char* name, void* stream, int64_t n_views, int64_t n_per_view,
                         int32_t tiles_x, int32_t tiles_y, const int32_t* tile_rect,
                         const uint32_t* tiles_touched, const float* depth, int64_t capacity,
                         void* workspace, size_t workspace_bytes, uint32_t* sorted_gid,
                         uint64_t* sorted_keys, uint32_t* tile_offsets, uint32_t* total_pairs) {
  if (n_views <= 0 || n_per_view < 0 || capacity < 0) return fail(QR_ERR_INVALID_ARG, "%s: negative size", name);
  if (tiles_x <= 0 || tiles_y <= 0) return fail(QR_ERR_INVALID_ARG, "%s: bad tile grid", name);
  const int64_t n_tiles = static_cast<int64_t>(tiles_x) * tiles_y * n_views;
  if (n_tiles >= (1ll << 31)) return fail(QR_ERR_UNSUPPORTED, "%s: too many tiles", name);
  const int64_t n = n_views * n_per_view;
  if (n_per_view >= (1ll << 32) || n >= (1ll << 40) || capacity >= (1ll << 32) - 1)
    return fail(QR_ERR_UNSUPPORTED, "%s: n and capacity must be below 2^32 - 1", name);
  if (!tile_offsets || !total_pairs || !workspace)
    return fail(QR_ERR_INVALID_ARG, "%s: null output or workspace", name);
  if (n > 0 && (!tile_rect || !tiles_touched || !depth))
    return fail(QR_ERR_INVALID_ARG, "%s: null input pointer", name);
  if (capacity > 0 && !sorted_gid) return fail(QR_ERR_INVALID_ARG, "%s: null sorted_gid", name);
  const Layout L = layout(n_tiles, capacity);
  if (workspace_bytes < L.bytes)
    return fail(QR_ERR_CAPACITY, "%s: workspace needs %zu bytes, got %zu", name, L.bytes,
                workspace_bytes);

  hipStream_t s = as_stream(stream);
  char* ws = static_cast<char*>(workspace);
  auto* cnt = reinterpret_cast<uint32_t*>(ws + L.cnt);
  auto* cursor = reinterpret_cast<uint32_t*>(ws + L.cursor);
  auto* part = reinterpret_cast<uint32_t*>(ws + L.part);
  auto* bucket = reinterpret_cast<unsigned long long*>(ws + L.bucket);
  auto* radix_tmp = reinterpret_cast<unsigned long long*>(ws + L.radix_tmp);

  const int view_tiles = tiles_x * tiles_y;
  const int4* const rect = reinterpret_cast<const int4*>(tile_rect);
  // Chunks of at least 1,024 records (one per thread: with 4,096, 60k records
  // occupy 15 CUs), and no more workgroups than fill the chip (512 of 16
  // waves). Their counts lie where long buckets are sorted later, which bounds
  // their number by the capacity: with room for less than a third of the chunks
  // each workgroup takes too many records one after the other, and the global
  // counters are as fast or faster, as there are few pairs then (1M records,
  // 81 x 61 tiles: room for 2 chunks 268 us in chunks, 24 by global counters;
  // for 45, 52 and 36; for 90, 46 and 48; for 170, 42 and 69).
  const int64_t want = std::max<int64_t>(
      std::min(std::min<int64_t>(ceil_div(n_per_view, kWideThreads), kMaxChunks), ceil_div(512, n_views)), 1);
  const int64_t n_chunks = std::min(want, static_cast<int64_t>(sizeof(uint64_t)) * capacity /
                                              (n_tiles * static_cast<int64_t>(sizeof(uint32_t))));
  if (n > 0 && n_tiles <= kSmallTiles && n <= kSmallRecords && n * view_tiles <= kSmallWork) {
    hipLaunchKernelGGL(bucket_small_kernel, dim3(1), dim3(kWideThreads), 0, s, static_cast<int>(n),
                       static_cast<int>(n_per_view), rect, tiles_touched, depth, tiles_x, tiles_y,
                       static_cast<int>(n_tiles), capacity, tile_offsets, total_pairs, bucket);
  } else if (n > 0 && view_tiles <= kLdsTiles && 3 * n_chunks >= want) {
    const int64_t chunk = ceil_div(n_per_view, n_chunks);
    const unsigned blocks = static_cast<unsigned>(n_views * n_chunks);
    const size_t lds = sizeof(uint32_t) * static_cast<size_t>(view_tiles);
    auto* const counts = reinterpret_cast<uint32_t*>(radix_tmp);
    hipLaunchKernelGGL(chunk_count_kernel, dim3(blocks), dim3(kWideThreads), lds, s, n_per_view,
                       static_cast<int>(n_chunks), chunk, rect, tiles_touched, tiles_x, view_tiles, counts);
    hipLaunchKernelGGL(chunk_scan_kernel, dim3(static_cast<unsigned>(ceil_div(n_tiles, 64))), dim3(512), 0, s, n_tiles,
                       view_tiles, static_cast<int>(n_chunks), counts, cnt);
    scan_exclusive(cnt, tile_offsets, n_tiles, part, total_pairs, s);
    hipLaunchKernelGGL(chunk_scatter_kernel, dim3(blocks), dim3(kWideThreads), lds, s, n_per_view,
                       static_cast<int>(n_chunks), chunk, rect, tiles_touched, depth, tiles_x, view_tiles, counts,
                       tile_offsets, capacity, bucket);
  } else {
    // counters and cursors are adjacent in the layout: one fill clears both
    const int64_t zero_n = static_cast<int64_t>((L.part - L.cnt) / sizeof(uint32_t));
    hipLaunchKernelGGL(zero_u32_kernel, dim3(static_cast<unsigned>(std::min<int64_t>(ceil_div(zero_n, 256), 1024))),
                       dim3(256), 0, s, cnt, zero_n);
    const unsigned gblocks = static_cast<unsigned>(std::max<int64_t>(ceil_div(n, 256), 1));
    const int64_t npv = std::max<int64_t>(n_per_view, 1);
    if (n > 0)
      hipLaunchKernelGGL(tile_pairs_kernel<false>, dim3(gblocks), dim3(256), 0, s, n, npv, rect, tiles_touched, depth,
                         tiles_x, tiles_y, cnt, nullptr, capacity, nullptr);
    scan_exclusive(cnt, tile_offsets, n_tiles, part, total_pairs, s);
    if (n > 0 && capacity > 0)
      hipLaunchKernelGGL(tile_pairs_kernel<true>, dim3(gblocks), dim3(256), 0, s, n, npv, rect, tiles_touched, depth,
                         tiles_x, tiles_y, cursor, tile_offsets, capacity, bucket);
  }
  if (capacity > 0)
    hipLaunchKernelGGL(tile_sort_kernel, dim3(static_cast<unsigned>(n_tiles)), dim3(256), 0, s,
                       static_cast<int>(n_tiles), tile_offsets, capacity, bits_for(n_per_view), bucket,
                       radix_tmp, sorted_gid, reinterpret_cast<unsigned long long*>(sorted_keys));
  return check_launch(name);
}

extern "C" int qr_bin_sort(void* stream, int64_t n, int32_t tiles_x, int32_t tiles_y,
                           const int32_t* tile_rect, const uint32_t* tiles_touched,
                           const float* depth, int64_t capacity, void* workspace,
                           size_t workspace_bytes, uint32_t* sorted_gid, uint64_t* sorted_keys,
                           uint32_t* tile_offsets, uint32_t* total_pairs) {
  if (n < 0) return fail(QR_ERR_INVALID_ARG, "qr_bin_sort: negative size");
  if (n >= (1ll << 32)) return fail(QR_ERR_UNSUPPORTED, "qr_bin_sort: n and capacity must be below 2^32 - 1");
  return bin_sort_impl("qr_bin_sort", stream, 1, n, tiles_x, tiles_y, tile_rect, tiles_touched,
                       depth, capacity, workspace, workspace_bytes, sorted_gid, sorted_keys,
                       tile_offsets, total_pairs);
}

// ---- zero-allocation variant ------------------------------------------------
namespace qr {

// The workspace of qr_bin_sort_noalloc: one copy per GPU, allocated when the
// library's code object is loaded on that GPU and held until the process
// ends. In host code `scratch` only names the symbol; its device address is
// looked up once per device (hipGetSymbolAddress) and only that address is
// passed to kernels.
static __device__ __align__(256) unsigned char scratch[QR_BIN_SORT_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_addr[kMaxDevices];

// Device address of `scratch` on the current device (looked up on the first
// call for each device).
static int scratch_address(const char* name, void** addr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(QR_ERR_HIP, "%s: hipGetDevice: %s", name, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(QR_ERR_UNSUPPORTED, "%s: device index %d beyond %d", name, dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(QR_ERR_HIP, "%s: hipGetSymbolAddress of the scratch array on device %d: %s",
                  name, dev, hipGetErrorString(e));
    g_scratch_addr[dev] = p;
  }
  *addr = g_scratch_addr[dev];
  return QR_OK;
}

}  // namespace qr

extern "C" int qr_bin_sort_noalloc(void* stream, int64_t n, int32_t tiles_x, int32_t tiles_y,
                                   const int32_t* tile_rect, const uint32_t* tiles_touched,
                                   const float* depth, int64_t capacity, uint32_t* sorted_gid,
                                   uint64_t* sorted_keys, uint32_t* tile_offsets,
                                   uint32_t* total_pairs) {
  const char* name = "qr_bin_sort_noalloc";
  if (n < 0 || capacity < 0 || tiles_x <= 0 || tiles_y <= 0)
    return fail(QR_ERR_INVALID_ARG, "%s: bad sizes", name);
  // checked before the layout is computed, so that the sizes below cannot
  // overflow
  if (capacity > static_cast<int64_t>(QR_BIN_SORT_SCRATCH_BYTES) ||
      static_cast<int64_t>(tiles_x) * tiles_y > static_cast<int64_t>(QR_BIN_SORT_SCRATCH_BYTES))
    return fail(QR_ERR_CAPACITY, "%s: capacity %lld pairs over %lld tiles exceeds the %d-byte scratch",
                name, static_cast<long long>(capacity),
                static_cast<long long>(tiles_x) * tiles_y, QR_BIN_SORT_SCRATCH_BYTES);
  const size_t need = layout(static_cast<int64_t>(tiles_x) * tiles_y, capacity).bytes;
  if (need > static_cast<size_t>(QR_BIN_SORT_SCRATCH_BYTES))
    return fail(QR_ERR_CAPACITY,
                "%s: capacity %lld pairs over %lld tiles needs %zu bytes of scratch, the maximum "
                "is %d",
                name, static_cast<long long>(capacity), static_cast<long long>(tiles_x) * tiles_y,
                need, QR_BIN_SORT_SCRATCH_BYTES);
  if (n >= (1ll << 32)) return fail(QR_ERR_UNSUPPORTED, "%s: n must be below 2^32 - 1", name);
  void* ws = nullptr;
  const int rc = scratch_address(name, &ws);
  if (rc != QR_OK) return rc;
  return bin_sort_impl(name, stream, 1, n, tiles_x, tiles_y, tile_rect, tiles_touched, depth,
                       capacity, ws, static_cast<size_t>(QR_BIN_SORT_SCRATCH_BYTES), sorted_gid,
                       sorted_keys, tile_offsets, total_pairs);
}

extern "C" int qr_bin_sort_views(void* stream, int32_t n_views, int64_t n_per_view,
                                 int32_t tiles_x, int32_t tiles_y, const int32_t* tile_rect,
                                 const uint32_t* tiles_touched, const float* depth,
                                 int64_t capacity, void* workspace, size_t workspace_bytes,
                                 uint32_t* sorted_gid, uint64_t* sorted_keys,
                                 uint32_t* tile_offsets, uint32_t* total_pairs) {
  return bin_sort_impl("qr_bin_sort_views", stream, n_views, n_per_view, tiles_x, tiles_y,
                       tile_rect, tiles_touched, depth, capacity, workspace, workspace_bytes,
                       sorted_gid, sorted_keys, tile_offsets, total_pairs);
}
