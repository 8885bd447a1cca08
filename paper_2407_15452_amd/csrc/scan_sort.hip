// Device-wide exclusive scan and a stable LSD radix sort (helpers of CSR construction,
// pair emission, pair sorting and id merging).
#include "common.h"

namespace gs {

static thread_local hipError_t g_last_error = hipSuccess;
void set_last_hip_error(hipError_t e) { g_last_error = e; }

extern "C" int32_t gs_last_hip_error(void) { return (int32_t)g_last_error; }

// ---------------------------------------------------------------------------
// Exclusive scan: tiles of 1024 values.  The tiles' sums first; then every tile is scanned from the sum of the
// tiles before it, which its workgroup adds up itself while there are few (a launch costs more).  Beyond that the
// tile sums are scanned the same way in between.  Offsets of walks, us, up to 1024, 4096 and 16,384 tiles without that: 1.1 M
// walks 21.2, 17.3, 17.3, 4 M 44.3, 41.3, 41.5, 4.2 M 45.9, 45.9, 44.2, 8 M 76.5, 76.3, 78.8, 16 M 146, 146, 181.
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int64_t kScanFewTiles = 4096;

// sum over the workgroup; every lane gets it
__device__ __forceinline__ int64_t block_sum_i64(int64_t v, int64_t* wave_sums) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  if ((threadIdx.x & 63) == 0) wave_sums[threadIdx.x >> 6] = v;
  __syncthreads();
  v = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) v += wave_sums[w];
  return v;
}

__global__ __launch_bounds__(kScanThreads) void scan_sums_i64_kernel(const int64_t* __restrict__ data, int64_t n,
                                                                     int64_t* __restrict__ tile_sums) {
  __shared__ int64_t wave_sums[kScanThreads / 64];
  int64_t local = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = (int64_t)blockIdx.x * kScanTile + k * kScanThreads + threadIdx.x;
    local += (i < n) ? data[i] : 0;
  }
  local = block_sum_i64(local, wave_sums);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = local;
}

// tile_sums: sums of the tiles (scanned == 0) or their exclusive prefix sums
__global__ __launch_bounds__(kScanThreads) void scan_apply_i64_kernel(int64_t* __restrict__ data, int64_t n,
                                                                      const int64_t* __restrict__ tile_sums, int scanned,
                                                                      int64_t* __restrict__ total_out) {
  __shared__ int64_t wave_sums[2][kScanThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int64_t v[kScanItems];
  int64_t local = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = (base + k < n) ? data[base + k] : 0;
    local += v[k];
  }
  int64_t before = 0;
  if (scanned) {
    before = tile_sums[blockIdx.x];
  } else if (blockIdx.x > 0) {
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kScanThreads) before += tile_sums[t];
    before = block_sum_i64(before, wave_sums[1]);
  }
  int64_t incl = local;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) wave_sums[0][wave] = incl;
  __syncthreads();
  int64_t run = before + incl - local;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w)
    if (w < wave) run += wave_sums[0][w];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) data[base + k] = run;
    run += v[k];
  }
  if (total_out != nullptr && blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) *total_out = run;
}

__global__ void zero_one_i64_kernel(int64_t* dst) { *dst = 0; }

size_t scan_scratch_elems(int64_t n) {
  size_t total = 1;
  while (n > 1) {
    n = ceil_div(n, kScanTile);
    total += (size_t)n;
    if (n == 1) break;
  }
  return total + 1;
}

int32_t exclusive_scan_i64(int64_t* data, int64_t n, int64_t* scratch, int64_t* total_out,
                           hipStream_t stream) {
  if (n <= 0) {
    if (total_out) {
      zero_one_i64_kernel<<<1, 1, 0, stream>>>(total_out);
      GS_LAUNCH_CHECK();
    }
    return GS_OK;
  }
  const int64_t tiles = ceil_div(n, kScanTile);
  if (tiles > 1) {
    scan_sums_i64_kernel<<<(unsigned)tiles, kScanThreads, 0, stream>>>(data, n, scratch);
    GS_LAUNCH_CHECK();
    if (tiles > kScanFewTiles) {
      const int32_t rc = exclusive_scan_i64(scratch, tiles, scratch + tiles, nullptr, stream);
      if (rc != GS_OK) return rc;
    }
  }
  scan_apply_i64_kernel<<<(unsigned)tiles, kScanThreads, 0, stream>>>(data, n, scratch, tiles > kScanFewTiles ? 1 : 0, total_out);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

// ---------------------------------------------------------------------------
// Stable least-significant-digit radix sort of (key, value) records.
//
// One pass over a digit: count (per tile and digit), a prefix sum per digit over the tiles, and
// the scatter.  A tile is kSortThreads * ITEMS consecutive records.  The scatter ranks a tile's
// records stably (a wave takes its records 64 at a time in index order: the lanes of equal digit
// find each other by ballots, the first of them advances the wave's counter of that digit),
// brings the tile into digit order in LDS and writes it out from there, so that the records of a
// digit leave as one contiguous run instead of one scattered record per lane.
//
// Bound by memory: a pass reads the keys twice and the values once and writes both once.  Measured
// on 23 million records of 8 + 4 bytes: 200 us per pass (count 63, prefix sums 5, scatter 133; 3.7
// TB/s of the 32 bytes per record), against 640 us with one wave per tile and every lane storing its
// own record (445 us the scatter, 110 us its 64-bit prefix sums); 300,007 records of 4 + 4 bytes: 16
// us per pass against 58.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kDigitBits = 8;
constexpr int kDigits = 1 << kDigitBits;

// keys at or above `limit` sort as `limit` (and keep their value)
template <typename K>
__device__ __forceinline__ uint32_t digit_of(K key, K limit, int shift, uint32_t mask) {
  return (uint32_t)(min(key, limit) >> shift) & mask;
}

template <typename K, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void radix_count_kernel(const K* __restrict__ keys, int64_t n, K limit,
                                                                   int shift, uint32_t mask, int64_t num_tiles,
                                                                   uint32_t* __restrict__ counts) {
  __shared__ uint32_t hist[kSortWaves / 2][kDigits];      // (two waves share a copy)
  uint32_t* flat = &hist[0][0];
  for (int i = threadIdx.x; i < kSortWaves / 2 * kDigits; i += kSortThreads) flat[i] = 0u;
  __syncthreads();
  uint32_t* mine = hist[threadIdx.x >> 7];
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * ITEMS);
  K key[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int64_t i = base + c * kSortThreads + threadIdx.x;
    key[c] = (i < n) ? keys[i] : (K)0;
  }
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (base + c * kSortThreads + threadIdx.x < n) atomicAdd(&mine[digit_of(key[c], limit, shift, mask)], 1u);
  __syncthreads();
  for (uint32_t d = threadIdx.x; d <= mask; d += kSortThreads) {
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves / 2; ++w) sum += hist[w][d];
    counts[(int64_t)d * num_tiles + blockIdx.x] = sum;
  }
}

// inclusive prefix sum over the lanes of a wave
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(v, d, 64);
    if (lane >= d) v += up;
  }
  return v;
}

// block d: exclusive prefix sums of the counts of digit d over the tiles, and their total
__global__ __launch_bounds__(256) void radix_scan_kernel(uint32_t* __restrict__ counts, int64_t num_tiles,
                                                         uint32_t* __restrict__ totals) {
  __shared__ uint32_t wave_sum[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* row = counts + (int64_t)blockIdx.x * num_tiles;
  uint32_t carry = 0;
  int turn = 0;
  for (int64_t base = 0; base < num_tiles; base += 1024, turn ^= 1) {
    const int64_t at = base + (int64_t)threadIdx.x * 4;
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = (at + k < num_tiles) ? row[at + k] : 0u;
    const uint32_t own = v[0] + v[1] + v[2] + v[3];
    const uint32_t incl = wave_inclusive(own, lane);
    if (lane == 63) wave_sum[turn][wave] = incl;
    __syncthreads();
    uint32_t run = carry + incl - own;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w < wave) run += wave_sum[turn][w];
      carry += wave_sum[turn][w];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (at + k < num_tiles) row[at + k] = run;
      run += v[k];
    }
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

template <typename K, typename V, bool kValues, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void radix_scatter_kernel(
    const K* __restrict__ keys, const V* __restrict__ vals, K* __restrict__ keys_out,
    V* __restrict__ vals_out, int64_t n, K limit, int shift, uint32_t mask, int64_t num_tiles,
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ totals) {
  constexpr int kTile = kSortThreads * ITEMS;
  // the tile in digit order: its keys, then its values
  constexpr size_t kRecord = kValues && sizeof(V) > sizeof(K) ? sizeof(V) : sizeof(K);
  __shared__ __align__(16) unsigned char stage_bytes[kTile * kRecord];
  K* stage = reinterpret_cast<K*>(stage_bytes);
  __shared__ uint32_t wave_count[kSortWaves][kDigits];
  __shared__ uint32_t tile_start[kDigits];            // first place of a digit in the tile
  __shared__ uint32_t out_start[kDigits];             // first place of the tile's run of a digit in the output, minus tile_start
  __shared__ uint32_t part[2][kDigits / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t* flat = &wave_count[0][0];
  for (int i = tid; i < kSortWaves * kDigits; i += kSortThreads) flat[i] = 0u;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  const int64_t first = base + (int64_t)wave * (64 * ITEMS) + lane;
  const int live = (int)min((int64_t)kTile, n - base);
  K key[ITEMS];
  V val[ITEMS];
  uint32_t rank[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int64_t i = first + c * 64;
    key[c] = (i < n) ? keys[i] : (K)0;
    if (kValues && i < n) val[c] = vals[i];
  }
  __syncthreads();
  // rank of every record among the wave's records of its digit, in index order
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = first + c * 64 < n;
    const uint32_t d = digit_of(key[c], limit, shift, mask);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kDigitBits; ++b) {
      const bool one = (d >> b) & 1u;
      const uint64_t vote = __ballot(one);
      peers &= one ? vote : ~vote;
    }
    const int leader = peers != 0ull ? __ffsll((unsigned long long)peers) - 1 : lane;
    uint32_t before = 0;
    if (valid && lane == leader) before = atomicAdd(&wave_count[wave][d], (uint32_t)__popcll(peers));
    before = __shfl(before, leader, 64);
    rank[c] = before + (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
  }
  __syncthreads();
  // per digit: the waves' counts become offsets inside the digit's run; digit runs follow each other
  if (tid < kDigits) {
    uint32_t run = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const uint32_t mine = wave_count[w][tid];
      wave_count[w][tid] = run;
      run += mine;
    }
    const uint32_t all = ((uint32_t)tid <= mask) ? totals[tid] : 0u;
    const uint32_t incl = wave_inclusive(run, lane), incl_all = wave_inclusive(all, lane);
    if (lane == 63) { part[0][wave] = incl; part[1][wave] = incl_all; }
    tile_start[tid] = incl - run;
    out_start[tid] = incl_all - all + (((uint32_t)tid <= mask) ? counts[(int64_t)tid * num_tiles + blockIdx.x] : 0u);
  }
  __syncthreads();
  if (tid < kDigits) {
    uint32_t a = 0, b = 0;
#pragma unroll
    for (int w = 0; w < kDigits / 64; ++w)
      if (w < wave) { a += part[0][w]; b += part[1][w]; }
    const uint32_t start = tile_start[tid] + a;
    tile_start[tid] = start;
    out_start[tid] += b - start;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const uint32_t d = digit_of(key[c], limit, shift, mask);
    rank[c] += tile_start[d] + wave_count[wave][d];
    if (first + c * 64 < n) stage[rank[c]] = key[c];
  }
  __syncthreads();
  uint32_t dest[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int at = c * kSortThreads + tid;
    if (at < live) {
      const K k = stage[at];
      dest[c] = out_start[digit_of(k, limit, shift, mask)] + (uint32_t)at;
      keys_out[dest[c]] = k;
    }
  }
  if (kValues) {
    V* vstage = reinterpret_cast<V*>(stage_bytes);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < ITEMS; ++c)
      if (first + c * 64 < n) vstage[rank[c]] = val[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < ITEMS; ++c) {
      const int at = c * kSortThreads + tid;
      if (at < live) vals_out[dest[c]] = vstage[at];
    }
  }
}

template <typename K, typename V, bool kValues, int ITEMS>
static int32_t radix_pass(const K* keys, const V* vals, K* keys_out, V* vals_out, int64_t n, K limit,
                          int shift, int bits, uint32_t* counts, uint32_t* totals, hipStream_t stream) {
  const int64_t tiles = ceil_div(n, kSortThreads * ITEMS);
  const uint32_t mask = (1u << bits) - 1u;
  radix_count_kernel<K, ITEMS><<<(unsigned)tiles, kSortThreads, 0, stream>>>(keys, n, limit, shift, mask, tiles, counts);
  GS_LAUNCH_CHECK();
  radix_scan_kernel<<<1u << bits, 256, 0, stream>>>(counts, tiles, totals);
  GS_LAUNCH_CHECK();
  radix_scatter_kernel<K, V, kValues, ITEMS><<<(unsigned)tiles, kSortThreads, 0, stream>>>(
      keys, vals, keys_out, vals_out, n, limit, shift, mask, tiles, counts, totals);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

// Records per lane: a tile of 8192 records makes runs of 32 records per digit on average (256 bytes
// of 8-byte keys); while that leaves compute units without a tile (256 of them, so below 2^21
// records), tiles of 2048.
constexpr int kSortItemsLarge = 16, kSortItemsSmall = 4;
constexpr int64_t kSortLarge = (int64_t)1 << 21;

// (never less than a shorter sort takes: a caller's workspace for its largest batch serves every batch)
size_t radix_sort_scratch_bytes(int64_t n) {
  const int64_t small = std::max((int64_t)1, std::min(n, kSortLarge - 1));
  const size_t tiles = (size_t)std::max(ceil_div(small, kSortThreads * kSortItemsSmall),
                                   n >= kSortLarge ? ceil_div(n, kSortThreads * kSortItemsLarge) : (int64_t)0);
  return align_up(tiles * kDigits * sizeof(uint32_t)) + align_up(kDigits * sizeof(uint32_t));
}

int radix_sort_passes(int nbits) { return (nbits + kDigitBits - 1) / kDigitBits; }

template <typename K, typename V>
int32_t radix_sort(const K* keys_in, const V* vals_in, K* keys_out, V* vals_out, K* keys_alt, V* vals_alt, int64_t n,
                   K limit, int nbits, void* scratch, hipStream_t stream) {
  if (n <= 0) return GS_OK;
  if (n > (int64_t)UINT32_MAX) return GS_EOVERFLOW;      // (places are 32-bit)
  const bool large = n >= kSortLarge;
  Carver cv(scratch);
  const int64_t tile = kSortThreads * (large ? kSortItemsLarge : kSortItemsSmall);
  uint32_t* counts = cv.take<uint32_t>((size_t)ceil_div(n, tile) * kDigits);
  uint32_t* totals = cv.take<uint32_t>(kDigits);
  auto pass = vals_in != nullptr ? (large ? radix_pass<K, V, true, kSortItemsLarge> : radix_pass<K, V, true, kSortItemsSmall>)
                                 : (large ? radix_pass<K, V, false, kSortItemsLarge> : radix_pass<K, V, false, kSortItemsSmall>);
  const int passes = radix_sort_passes(nbits);
  const int width = (nbits + passes - 1) / passes;
  const K* k_from = keys_in;
  const V* v_from = vals_in;
  for (int p = 0; p < passes; ++p) {
    const bool to_alt = (passes - 1 - p) & 1;              // the last pass ends in the output
    K* k_to = to_alt ? keys_alt : keys_out;
    V* v_to = to_alt ? vals_alt : vals_out;
    const int32_t rc = pass(k_from, v_from, k_to, v_to, n, limit, p * width, std::min(width, nbits - p * width), counts,
                            totals, stream);
    if (rc != GS_OK) return rc;
    k_from = k_to;
    v_from = v_to;
  }
  return GS_OK;
}
template int32_t radix_sort(const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, uint32_t*, uint32_t*, int64_t,
                            uint32_t, int, void*, hipStream_t);
template int32_t radix_sort(const uint32_t*, const uint2*, uint32_t*, uint2*, uint32_t*, uint2*, int64_t, uint32_t,
                            int, void*, hipStream_t);
template int32_t radix_sort(const uint64_t*, const uint32_t*, uint64_t*, uint32_t*, uint64_t*, uint32_t*, int64_t,
                            uint64_t, int, void*, hipStream_t);

}  // namespace gs
