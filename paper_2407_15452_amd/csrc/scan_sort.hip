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
// One pass over a digit: count (per tile and digit), prefix sums per digit over the tiles, and
// the scatter.  A tile is kSortThreads * ITEMS consecutive records.  The scatter ranks a tile's
// records stably (a wave takes its records 64 at a time in index order: the lanes of equal digit
// find each other by ballots, the first of them advances the wave's counter of that digit),
// brings the tile into digit order in LDS and writes it out from there, so that the records of a
// digit leave as one contiguous run instead of one scattered record per lane.
//
// Bound by memory: a pass reads the keys twice and the values once and writes both once, so fewer passes over wider digits
// win as long as the runs of a digit still fill their cache lines.  23 million records of 8 + 4 bytes: 40 bits in four passes
// of 10 (count 42, prefix sums 14, scatter 121 us: 710 us in all) against five of 8 (47, 5 and 130: 908); 20 bits of 11 million
// records of 4 + 8 bytes 218 against 273.  Digits of 11 bits gain nothing: 22 bits of 12 million records in two passes 297 us (scatter 113),
// in three of 8 296 (76).  Counts lie by tile, so that a tile's are written, and read, as one run (by digit: count 58 us
// of 23 million records).  The values are read when the keys have left: 782 against 918 us for the same sort in five passes.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 512;
constexpr int kSortWaves = kSortThreads / 64;

// keys at or above `limit` sort as `limit` (and keep their value)
template <typename K>
__device__ __forceinline__ uint32_t digit_of(K key, K limit, int shift, uint32_t mask) {
  return (uint32_t)(min(key, limit) >> shift) & mask;
}

// The tile of a scattering workgroup: each XCD (workgroups go to the 8 of them in turn) takes one contiguous eighth, so that the runs of a
// digit that share a cache line meet in one L2.  Small tiles of at most 256 digits, whose runs are half a line, go to the XCD where the count kernel
// has just read their keys.  8 + 4 bytes, by eighths / by turns, us: 8 bits, 0.6 million records 12.4 / 10.6, 1 million 12.9 / 11.4; 10 bits, 0.3
// million 9.0 / 9.1, 1.4 million 14.1 / 17.3.
template <int ITEMS, int BITS>
__device__ __forceinline__ int64_t sort_tile(int64_t tiles_per_xcd) {
  if (ITEMS <= 4 && BITS <= 8) return blockIdx.x;
  return (int64_t)(blockIdx.x & 7u) * tiles_per_xcd + (blockIdx.x >> 3);
}

template <typename K, int ITEMS, int BITS>
__global__ __launch_bounds__(kSortThreads) void radix_count_kernel(const K* __restrict__ keys, int64_t n, K limit,
                                                                   int shift, uint32_t mask,
                                                                   uint32_t* __restrict__ counts) {
  constexpr int kD = 1 << BITS;
  constexpr int kCopies = BITS <= 8 ? 4 : 2;              // (the waves share them)
  __shared__ uint32_t hist[kCopies][kD];
  uint32_t* flat = &hist[0][0];
  for (int i = threadIdx.x; i < kCopies * kD; i += kSortThreads) flat[i] = 0u;
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * ITEMS);
  K key[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int64_t i = base + c * kSortThreads + threadIdx.x;
    key[c] = (i < n) ? keys[i] : (K)0;
  }
  __syncthreads();
  uint32_t* mine = hist[(threadIdx.x >> 6) % kCopies];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (base + c * kSortThreads + threadIdx.x < n) atomicAdd(&mine[digit_of(key[c], limit, shift, mask)], 1u);
  __syncthreads();
  uint32_t* row = counts + (int64_t)blockIdx.x * (mask + 1u);
  for (uint32_t d = threadIdx.x; d <= mask; d += kSortThreads) {
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kCopies; ++w) sum += hist[w][d];
    row[d] = sum;
  }
}

// Exclusive prefix sums of the counts of a digit over the tiles, and their total: a workgroup takes kScanDigits digits, a
// lane one digit of a stretch of tiles.
constexpr int kScanDigits = 16, kScanStretches = 1024 / kScanDigits;
__global__ __launch_bounds__(1024) void radix_scan_kernel(uint32_t* __restrict__ counts, int64_t num_tiles, uint32_t digits,
                                                          uint32_t* __restrict__ totals) {
  __shared__ uint32_t sums[kScanStretches][kScanDigits + 1];
  const uint32_t d = blockIdx.x * kScanDigits + (threadIdx.x & (kScanDigits - 1));
  const int s = threadIdx.x / kScanDigits;
  const int64_t per = (num_tiles + kScanStretches - 1) / kScanStretches;
  const int64_t lo = min(num_tiles, s * per), hi = min(num_tiles, lo + per);
  const bool live = d < digits;
  constexpr int kBurst = 16;
  uint32_t v[kBurst];
  auto load = [&](int64_t t) {
#pragma unroll
    for (int u = 0; u < kBurst; ++u) v[u] = (live && t + u < hi) ? counts[(t + u) * digits + d] : 0u;
  };
  uint32_t sum = 0;
  for (int64_t t = lo; t < hi; t += kBurst) {
    load(t);
#pragma unroll
    for (int u = 0; u < kBurst; ++u) sum += v[u];
  }
  sums[s][threadIdx.x & (kScanDigits - 1)] = sum;
  __syncthreads();
  {                                              // wave w: the stretches of digit w
    static_assert(kScanStretches == 64 && kScanDigits == 16, "sixteen waves, a lane per stretch");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t own = sums[lane][w];
    const uint32_t incl = wave_inclusive(own, lane);
    sums[lane][w] = incl - own;
    if (lane == 63 && blockIdx.x * kScanDigits + w < digits) totals[blockIdx.x * kScanDigits + w] = incl;
  }
  __syncthreads();
  uint32_t run = sums[s][threadIdx.x & (kScanDigits - 1)];
  for (int64_t t = lo; t < hi; t += kBurst) {
    if (per > kBurst) load(t);                   // (else still there)
#pragma unroll
    for (int u = 0; u < kBurst; ++u) {
      if (live && t + u < hi) counts[(t + u) * digits + d] = run;
      run += v[u];
    }
  }
}

// The same for few tiles, where a launch takes as long as its chain of reads, sums and writes: a workgroup takes four digits, a lane those of one
// to three tiles.  us, against the kernel above: 256 digits of 40 tiles 3.2 / 4.0, of 290 3.9 / 5.3, of 490 4.5 / 5.3; 1024 digits of 150
// tiles 3.9 / 5.4, of 680 6.3 / 5.4.  With the tiles above, which were slower for a million records and less than counts by digit and tiles in turn: CSR of
// 300,000 edges 122 -> 116 us (115 then).
constexpr int kFewEach = 3, kFewThreads = 256;
constexpr int64_t kFewCounts = 1 << 18;
__global__ __launch_bounds__(kFewThreads) void radix_scan_few_kernel(uint32_t* __restrict__ counts, int num_tiles, uint32_t digits,
                                                                     uint32_t* __restrict__ totals) {
  __shared__ uint4 part[kFewThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t d = blockIdx.x * 4u;
  const int per = (num_tiles + kFewThreads - 1) / kFewThreads, lo = min(num_tiles, (int)threadIdx.x * per), hi = min(num_tiles, lo + per);
  auto plus = [](uint4 a, uint4 b) { return make_uint4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
  uint4 v[kFewEach], own = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int u = 0; u < kFewEach; ++u)
    v[u] = lo + u < hi ? *reinterpret_cast<const uint4*>(counts + (int64_t)(lo + u) * digits + d) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int u = 0; u < kFewEach; ++u) own = plus(own, v[u]);
  const uint4 incl = make_uint4(wave_inclusive(own.x, lane), wave_inclusive(own.y, lane), wave_inclusive(own.z, lane), wave_inclusive(own.w, lane));
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  uint4 run = make_uint4(incl.x - own.x, incl.y - own.y, incl.z - own.z, incl.w - own.w);
#pragma unroll
  for (int w = 0; w < kFewThreads / 64; ++w)
    if (w < wave) run = plus(run, part[w]);
#pragma unroll
  for (int u = 0; u < kFewEach; ++u) {
    if (lo + u < hi) *reinterpret_cast<uint4*>(counts + (int64_t)(lo + u) * digits + d) = run;
    run = plus(run, v[u]);
  }
  if (threadIdx.x == kFewThreads - 1) *reinterpret_cast<uint4*>(totals + d) = run;
}

template <typename K, typename V, bool kValues, int ITEMS, int BITS>
__global__ __launch_bounds__(kSortThreads, 4) void radix_scatter_kernel(
    const K* __restrict__ keys, const V* __restrict__ vals, K* __restrict__ keys_out,
    V* __restrict__ vals_out, int64_t n, K limit, int shift, uint32_t mask, int64_t num_tiles, int64_t tiles_per_xcd,
    const uint32_t* __restrict__ counts, const uint32_t* __restrict__ totals) {
  constexpr int kTile = kSortThreads * ITEMS;
  constexpr int kD = 1 << BITS;
  constexpr int kOwn = kD > kSortThreads ? kD / kSortThreads : 1;       // consecutive digits per lane
  static_assert(kTile <= 65535, "places in a tile have 16 bits");
  // the tile in digit order: its keys, then its values; before that the waves' counters of the digits
  constexpr size_t kRecord = kValues && sizeof(V) > sizeof(K) ? sizeof(V) : sizeof(K);
  constexpr size_t kCounters = sizeof(uint16_t) * kSortWaves * kD;
  constexpr size_t kBytes = kTile * kRecord > kCounters ? kTile * kRecord : kCounters;
  __shared__ __align__(16) unsigned char bytes[kBytes];
  __shared__ uint32_t out_start[kD];                  // first place of the tile's run of a digit in the output, minus its place in the tile
  __shared__ uint32_t part[2][kSortWaves];
  uint32_t* pairs = reinterpret_cast<uint32_t*>(bytes);            // two counters each
  uint16_t* wave_count = reinterpret_cast<uint16_t*>(bytes);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t tile = sort_tile<ITEMS, BITS>(tiles_per_xcd);
  if (tile >= num_tiles) return;
  for (int i = tid; i < kSortWaves * kD / 2; i += kSortThreads) pairs[i] = 0u;
  const int64_t base = tile * kTile;
  const int64_t first = base + (int64_t)wave * (64 * ITEMS) + lane;
  const int live = (int)min((int64_t)kTile, n - base);
  K key[ITEMS];
  V val[ITEMS];
  uint32_t rank[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int64_t i = first + c * 64;
    key[c] = (i < n) ? keys[i] : (K)0;
  }
  uint32_t below_all[kOwn], below_tile[kOwn];
#pragma unroll
  for (int o = 0; o < kOwn; ++o) {
    const uint32_t d = (uint32_t)(tid * kOwn + o);
    below_all[o] = d <= mask ? totals[d] : 0u;
    below_tile[o] = d <= mask ? counts[tile * (mask + 1u) + d] : 0u;
  }
  __syncthreads();
  // rank of every record among the wave's records of its digit, in index order
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const bool valid = first + c * 64 < n;
    const uint32_t d = digit_of(key[c], limit, shift, mask);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const bool one = (d >> b) & 1u;
      const uint64_t vote = __ballot(one);
      peers &= one ? vote : ~vote;
    }
    const int leader = peers != 0ull ? __ffsll((unsigned long long)peers) - 1 : lane;
    const int half = 16 * (int)(d & 1u);
    uint32_t before = 0;
    if (valid && lane == leader) before = atomicAdd(&pairs[(wave * kD + d) >> 1], (uint32_t)__popcll(peers) << half) >> half;
    before = __shfl(before, leader, 64) & 0xffffu;
    rank[c] = before + (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
  }
  __syncthreads();
  // per digit: the waves' counts become places in the tile; digit runs follow each other, in the tile and in the output
  const bool owns = tid * kOwn < kD;
  uint32_t own = 0, all = 0;
  if (owns) {
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      all += below_all[o];
#pragma unroll
      for (int w = 0; w < kSortWaves; ++w) own += wave_count[w * kD + tid * kOwn + o];
    }
  }
  const uint32_t incl = wave_inclusive(own, lane), incl_all = wave_inclusive(all, lane);
  if (lane == 63) { part[0][wave] = incl; part[1][wave] = incl_all; }
  __syncthreads();
  if (owns) {
    uint32_t run = incl - own, run_all = incl_all - all;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w)
      if (w < wave) { run += part[0][w]; run_all += part[1][w]; }
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      out_start[tid * kOwn + o] = run_all + below_tile[o] - run;
      run_all += below_all[o];
#pragma unroll
      for (int w = 0; w < kSortWaves; ++w) {
        const int at = w * kD + tid * kOwn + o;
        const uint32_t mine = wave_count[at];
        wave_count[at] = (uint16_t)run;
        run += mine;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) rank[c] += wave_count[wave * kD + digit_of(key[c], limit, shift, mask)];
  __syncthreads();
  K* stage = reinterpret_cast<K*>(bytes);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (first + c * 64 < n) stage[rank[c]] = key[c];
  if constexpr (kValues)
#pragma unroll
    for (int c = 0; c < ITEMS; ++c) {
      const int64_t i = first + c * 64;
      if (i < n) val[c] = vals[i];
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
  if constexpr (kValues) {
    V* vstage = reinterpret_cast<V*>(bytes);
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

template <typename K, typename V, bool kValues, int ITEMS, int BITS>
static int32_t radix_pass(const K* keys, const V* vals, K* keys_out, V* vals_out, int64_t n, K limit,
                          int shift, int bits, uint32_t* counts, uint32_t* totals, hipStream_t stream) {
  const int64_t tiles = ceil_div(n, kSortThreads * ITEMS), per_xcd = ceil_div(tiles, 8);
  const uint32_t mask = (1u << bits) - 1u;
  radix_count_kernel<K, ITEMS, BITS><<<(unsigned)tiles, kSortThreads, 0, stream>>>(keys, n, limit, shift, mask, counts);
  GS_LAUNCH_CHECK();
  if (tiles <= kFewThreads * kFewEach && tiles << bits <= kFewCounts && bits >= 2) radix_scan_few_kernel<<<(mask + 1u) / 4u, kFewThreads, 0, stream>>>(counts, (int)tiles, mask + 1u, totals);
  else radix_scan_kernel<<<(unsigned)ceil_div(mask + 1, kScanDigits), 1024, 0, stream>>>(counts, tiles, mask + 1u, totals);
  GS_LAUNCH_CHECK();
  radix_scatter_kernel<K, V, kValues, ITEMS, BITS><<<(unsigned)(8 * per_xcd), kSortThreads, 0, stream>>>(
      keys, vals, keys_out, vals_out, n, limit, shift, mask, tiles, per_xcd, counts, totals);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

// Digits of up to 10 bits, that is, as few passes as those take, all of about the same width; of up to 8 for few records, which the
// narrower count table of their one or two tiles serves as well, and where the caller's scratch memory holds no more.
constexpr int kWideBits = 10, kNarrowBits = 8;
constexpr int64_t kWideMin = (int64_t)1 << 13;
// Records per lane.  Long runs per digit want large tiles, which leave compute units idle while there are few records.  Whole sorts, us, with
// 4 / 8 / 16: 20-bit keys of 4 + 8 bytes, 0.7 M records 42 / 45 / 59, 1.5 M 57 / 56 / 64, 3 M 87 / 74 / 82, 5 M 126 / 110 / 117, 8 M
// 201 / 175 / 152; 40-bit keys of 8 + 4 bytes 89 / 91 / 119, 111 / 107 / 122, 171 / 159 / 162, 242 / 229 / 213, 370 / 325 / 302.
constexpr int64_t kMidTiles = (int64_t)3 << 19, kLargeTiles = (int64_t)5 << 20;
constexpr int64_t kLargeTilesNarrow = (int64_t)1 << 21;

static SortPlan sort_plan_of(int64_t n, int nbits, bool wide) {
  SortPlan p;
  const int most = wide ? kWideBits : kNarrowBits;
  p.passes = (nbits + most - 1) / most;
  p.width = (nbits + p.passes - 1) / p.passes;
  if (wide) p.items = n >= kLargeTiles ? 16 : (n >= kMidTiles ? 8 : 4);
  else p.items = n >= kLargeTilesNarrow ? 16 : 4;
  return p;
}
static size_t sort_scratch(int64_t n, const SortPlan& p) {
  return align_up((size_t)ceil_div(std::max((int64_t)1, n), kSortThreads * p.items) * sizeof(uint32_t) << p.width) +
         align_up(sizeof(uint32_t) << p.width);
}

// (for any width of keys; never less than a shorter sort takes: a caller's workspace for its largest batch serves every batch)
size_t radix_sort_scratch_bytes(int64_t n, bool wide) {
  size_t bytes = 0;
  for (const int64_t border : {kWideMin, kMidTiles, kLargeTiles, kLargeTilesNarrow, n + 1}) {
    const int64_t m = std::min(n, border - 1);
    const bool w = wide && m >= kWideMin;
    bytes = std::max(bytes, sort_scratch(m, sort_plan_of(m, w ? kWideBits : kNarrowBits, w)));
  }
  return bytes;
}

SortPlan radix_sort_plan(int64_t n, int nbits, size_t scratch_bytes) {
  const SortPlan wide = sort_plan_of(n, nbits, true);
  return n >= kWideMin && sort_scratch(n, wide) <= scratch_bytes ? wide : sort_plan_of(n, nbits, false);
}

template <typename K, typename V, bool kValues, int ITEMS>
static int32_t radix_pass_of(int bits, const K* keys, const V* vals, K* keys_out, V* vals_out, int64_t n, K limit,
                             int shift, uint32_t* counts, uint32_t* totals, hipStream_t stream) {
  if (bits <= kNarrowBits)
    return radix_pass<K, V, kValues, ITEMS, kNarrowBits>(keys, vals, keys_out, vals_out, n, limit, shift, bits, counts, totals, stream);
  return radix_pass<K, V, kValues, ITEMS, kWideBits>(keys, vals, keys_out, vals_out, n, limit, shift, bits, counts, totals, stream);
}

template <typename K, typename V>
int32_t radix_sort(const SortPlan& plan, const K* keys_in, const V* vals_in, K* keys_out, V* vals_out, K* keys_alt, V* vals_alt,
                   int64_t n, K limit, int nbits, void* scratch, hipStream_t stream) {
  if (n <= 0) return GS_OK;
  if (n > (int64_t)UINT32_MAX) return GS_EOVERFLOW;      // (places are 32-bit)
  Carver cv(scratch);
  uint32_t* counts = cv.take<uint32_t>((size_t)ceil_div(n, kSortThreads * plan.items) << plan.width);
  uint32_t* totals = cv.take<uint32_t>((size_t)1 << plan.width);
  auto pass = plan.items == 16 ? radix_pass_of<K, V, true, 16> : (plan.items == 8 ? radix_pass_of<K, V, true, 8> : radix_pass_of<K, V, true, 4>);
  if constexpr (sizeof(K) == 8) {                          // (64-bit keys alone come without values)
    if (vals_in == nullptr)
      pass = plan.items == 16 ? radix_pass_of<K, V, false, 16> : (plan.items == 8 ? radix_pass_of<K, V, false, 8> : radix_pass_of<K, V, false, 4>);
  }
  const K* k_from = keys_in;
  const V* v_from = vals_in;
  for (int p = 0; p < plan.passes; ++p) {
    const bool to_alt = (plan.passes - 1 - p) & 1;         // the last pass ends in the output
    K* k_to = to_alt ? keys_alt : keys_out;
    V* v_to = to_alt ? vals_alt : vals_out;
    const int32_t rc = pass(std::min(plan.width, nbits - p * plan.width), k_from, v_from, k_to, v_to, n, limit, p * plan.width,
                            counts, totals, stream);
    if (rc != GS_OK) return rc;
    k_from = k_to;
    v_from = v_to;
  }
  return GS_OK;
}
template int32_t radix_sort(const SortPlan&, const uint32_t*, const uint32_t*, uint32_t*, uint32_t*, uint32_t*, uint32_t*, int64_t,
                            uint32_t, int, void*, hipStream_t);
template int32_t radix_sort(const SortPlan&, const uint32_t*, const uint2*, uint32_t*, uint2*, uint32_t*, uint2*, int64_t, uint32_t,
                            int, void*, hipStream_t);
template int32_t radix_sort(const SortPlan&, const uint64_t*, const uint32_t*, uint64_t*, uint32_t*, uint64_t*, uint32_t*, int64_t,
                            uint64_t, int, void*, hipStream_t);


}  // namespace gs
