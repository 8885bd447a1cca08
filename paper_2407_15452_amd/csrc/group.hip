// Grouping of the terms of a large training batch by their row (see sgns.hip): records into the order of their
// rows, the records of a row in any order.
//
// Without stability one pass over memory and one over LDS do what three passes of the radix sort do.  The records are brought into
// a few thousand buckets of consecutive rows (count, prefix sums, scatter; a record's rank in its tile is an LDS atomic's answer), and a
// bucket, of about 6000 records where there are many, fits the registers and the LDS of a workgroup, which counts its
// rows and puts it in order.  12 million records on 4 M rows take 175 us (count 20, prefix sums 14, scatter 76, buckets 62)
// against 296 for the stable sort in three passes; 2.4 million 46 (79 in two), 1.6 million 41 (57).  In a step of walks, which brings 2 million
// staging slots along, 207 (15, 13, 89, 77, and 13 to find no bucket to split).
//
// Two kinds of rows are grouped together: rows of the first kind come as records (row; 8 bytes), rows of the second kind as a list of
// rows with gaps (-1: no record), whose 8 bytes are the place in the list and a constant.  The gaps are left out on the way, so the number of
// records of the second kind need not be known to the host.
//
// Buckets of more records than a workgroup takes (a single row may have any number) are split: the prefix sums enter them in a list,
// in pieces, the bucket kernel adds up the counts of their rows in global memory, and one more launch, which otherwise looks at the length of
// the list and returns, moves their records: every piece sums the counts of its bucket's rows by itself, so that no workgroup waits for what
// another of the same launch has written.  (With the last piece of a bucket summing them in the same launch, the release and acquire around that took 50 to
// 90 us where other workgroups were writing: 4 million records of a batch of walks on 5000 nodes, 64 buckets split, bucket kernel 121 -> 36 us and the
// launch behind it 17 -> 18; without fences 521 -> 437 us the step.)  All 12 million records in one row, 128 fp32 columns: a step of
// 2.84 ms (3.24).
#include "group.h"

namespace gs {

constexpr int kBucketThreads = 1024, kBucketWaves = kBucketThreads / 64;
constexpr int kBucketItems = 9, kBucketItemsMost = 16;         // records per lane: two workgroups, or one, share a compute unit's LDS
constexpr int64_t kBuckets = 2048, kSecondBuckets = 1024;      // most buckets of either kind of rows
// Records per bucket, which leave a bucket of 9216 room for uneven rows; fewer where that keeps compute units busy.
constexpr int64_t kBucketMean = 6000, kBucketMeanLeast = 1024, kBusyBuckets = 256, kBucketMeanMost = 7000;
// Buckets to split: records per lane of a piece, workgroups for the pieces, rows of a bucket whose counters leave room for two of them in a compute unit.
constexpr int kPieceItems = 4, kPiece = kBucketThreads * kPieceItems, kSplitBlocks = 512, kFewRowBits = 12;
// Records of a tile.  us with 2048 / 4096 / 8192: 0.8 M records 35.9 / 36.9 / 41.2, 1.6 M 40.6 / 40.7 / 42.4, 2.4 M 54 / 50 / 54, 3 M
// 65 / 60 / 62, 6 M 108 / 97 / 90; 16,384 instead of 8192 (half the counts): prefix sums of 12 million records 23 -> 15, the scatter the same
constexpr int64_t kMidGroupTiles = (int64_t)3 << 19, kLargeGroupTiles = (int64_t)1 << 22, kLargestGroupTiles = (int64_t)1 << 23;

// ---- into the buckets -----------------------------------------------------------------------
// Tiles [0, first_tiles) hold records of the first kind, the others entries of the list of the second kind.
struct TileOf {
  bool second;
  int64_t base;                  // first record, or first entry of the list
  int live;                      // records or entries
  int row_bits;
  uint32_t digits;               // buckets of the kind
  uint32_t* counts;              // of the tile, per bucket
  uint32_t *totals, *starts;     // of the kind, per bucket: records, and the first of them in the result
};
__device__ __forceinline__ TileOf tile_of(const GroupArgs& a, int64_t tile, int size) {
  TileOf t;
  t.second = tile >= a.first_tiles;
  t.base = (t.second ? tile - a.first_tiles : tile) * size;
  t.live = (int)min((int64_t)size, (t.second ? a.second_n : a.n) - t.base);
  t.row_bits = t.second ? a.second_row_bits : a.row_bits;
  t.digits = t.second ? a.digits - a.buckets : a.buckets;
  t.counts = a.counts + (t.second ? a.first_tiles * a.buckets + (tile - a.first_tiles) * t.digits : tile * t.digits);
  t.totals = a.totals + (t.second ? a.buckets : 0u);
  t.starts = a.starts + (t.second ? a.buckets : 0u);
  return t;
}

template <int kTileThreads, int ITEMS, int DIGITS>
__global__ __launch_bounds__(kTileThreads) void group_count_kernel(GroupArgs a) {
  constexpr int kCopies = DIGITS <= 256 ? 4 : 2;          // (the waves share them)
  __shared__ uint32_t hist[kCopies][DIGITS];
  uint32_t* flat = &hist[0][0];
  for (int i = threadIdx.x; i < kCopies * DIGITS; i += kTileThreads) flat[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x < kGroupCounters) a.counters[threadIdx.x] = 0u;
  const int64_t windows = ((a.n + a.second_n) >> a.seg_shift) + 2, windows_each = (windows + gridDim.x - 1) / gridDim.x;
  for (int64_t w = blockIdx.x * windows_each + threadIdx.x; w < min(windows, (blockIdx.x + 1) * windows_each); w += kTileThreads)
    a.further[w] = make_uint2(kNoGroupRow, 0u);
  const TileOf t = tile_of(a, blockIdx.x, kTileThreads * ITEMS);
  const uint32_t* rows = t.second ? reinterpret_cast<const uint32_t*>(a.second) : a.rows;
  uint32_t row[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int i = c * kTileThreads + threadIdx.x;
    row[c] = i < t.live ? rows[t.base + i] : kNoGroupRow;
  }
  __syncthreads();
  uint32_t* mine = hist[(threadIdx.x >> 6) % kCopies];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (row[c] != kNoGroupRow) atomicAdd(&mine[row[c] >> t.row_bits], 1u);
  __syncthreads();
  for (uint32_t d = threadIdx.x; d < t.digits; d += kTileThreads) {
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kCopies; ++w) sum += hist[w][d];
    t.counts[d] = sum;
  }
}

// Exclusive prefix sums of the counts of a bucket over the tiles, and their total: a workgroup takes kScanDigits buckets, a
// lane one bucket of a stretch of tiles.  Buckets of more than a.most records are entered in the list.
constexpr int kScanDigits = 16, kScanStretches = 1024 / kScanDigits;
__global__ __launch_bounds__(1024) void group_scan_kernel(GroupArgs a) {
  __shared__ uint32_t sums[kScanStretches][kScanDigits + 1];
  __shared__ uint32_t total_s[kScanDigits];
  const bool second = blockIdx.x >= a.first_scans;
  const uint32_t digits = second ? a.digits - a.buckets : a.buckets, first_digit = second ? a.buckets : 0u;
  const uint32_t d0 = (second ? blockIdx.x - a.first_scans : blockIdx.x) * kScanDigits;       // among the kind's buckets
  const uint32_t d = d0 + (threadIdx.x & (kScanDigits - 1));
  uint32_t* counts = a.counts + (second ? a.first_tiles * a.buckets : 0);
  const int64_t tiles = second ? a.tiles - a.first_tiles : a.first_tiles;
  const int s = threadIdx.x / kScanDigits;
  const int64_t per = (tiles + kScanStretches - 1) / kScanStretches;
  const int64_t lo = min(tiles, s * per), hi = min(tiles, lo + per);
  const bool live = d < digits;
  constexpr int kBurst = 8;
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
  {                                              // wave w: the stretches of bucket w
    static_assert(kScanStretches == 64 && kScanDigits == 16, "sixteen waves, a lane per stretch");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t own = sums[lane][w];
    const uint32_t incl = wave_inclusive(own, lane);
    sums[lane][w] = incl - own;
    if (lane == 63) {
      total_s[w] = incl;
      if (d0 + w < digits) a.totals[first_digit + d0 + w] = incl;
    }
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
  {                                              // wave w: bucket w, if it is to be split (those behind the last have no records)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t total = total_s[w];
    if (total <= a.most) return;
    const uint32_t pieces = (total + kPiece - 1) / kPiece;
    const uint32_t rows = 1u << (second ? a.second_row_bits : a.row_bits);
    uint32_t first = 0, rows_at = 0;
    if (lane == 0) {
      first = atomicAdd(a.counters + kGroupPieces, pieces);
      rows_at = atomicAdd(a.counters + kGroupSplitRows, rows);
    }
    first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
    rows_at = (uint32_t)__builtin_amdgcn_readfirstlane((int)rows_at);
    for (uint32_t i = lane; i < pieces; i += 64u) a.pieces[first + i] = make_uint4(first_digit + d0 + (uint32_t)w, rows_at, i, pieces);
    for (uint32_t r = lane; r < rows; r += 64u) a.row_counts[rows_at + r] = a.row_taken[rows_at + r] = 0u;
  }
}

template <int kTileThreads, int ITEMS, int DIGITS>
__global__ __launch_bounds__(kTileThreads, 4) void group_scatter_kernel(GroupArgs a) {
  constexpr int kTile = kTileThreads * ITEMS, kTileWaves = kTileThreads / 64;
  constexpr int kOwn = DIGITS > kTileThreads ? DIGITS / kTileThreads : 1;
  constexpr size_t kBytes = kTile * sizeof(uint2) > sizeof(uint32_t) * DIGITS ? kTile * sizeof(uint2) : sizeof(uint32_t) * DIGITS;
  __shared__ __align__(16) unsigned char bytes[kBytes];          // the buckets' counters, then the tile's rows, then its values
  __shared__ uint32_t out_start[DIGITS];                         // first place of the tile's run of a bucket, minus its place in the tile
  __shared__ uint32_t part[2][kTileWaves];
  uint32_t* count = reinterpret_cast<uint32_t*>(bytes);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // each XCD (workgroups go to the 8 of them in turn) takes one contiguous eighth, so that the runs of a bucket that share a cache
  // line meet in one L2
  const int64_t tile = (int64_t)(blockIdx.x & 7u) * a.tiles_per_xcd + (blockIdx.x >> 3);
  if (tile >= a.tiles) return;
  const TileOf t = tile_of(a, tile, kTile);
  const uint32_t* rows = (t.second ? reinterpret_cast<const uint32_t*>(a.second) : a.rows) + t.base;
  for (int i = tid; i < DIGITS; i += kTileThreads) count[i] = 0u;
  uint32_t row[ITEMS], rank[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) row[c] = c * kTileThreads + tid < t.live ? rows[c * kTileThreads + tid] : kNoGroupRow;
  uint32_t below_all[kOwn], below_tile[kOwn];
#pragma unroll
  for (int o = 0; o < kOwn; ++o) {
    const uint32_t d = (uint32_t)(tid * kOwn + o);
    below_all[o] = d < t.digits ? t.totals[d] : 0u;
    below_tile[o] = d < t.digits ? t.counts[d] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (row[c] != kNoGroupRow) rank[c] = atomicAdd(&count[row[c] >> t.row_bits], 1u);
  __syncthreads();
  const bool owns = tid * kOwn < DIGITS;
  uint32_t mine[kOwn], own = 0, all = 0;
#pragma unroll
  for (int o = 0; o < kOwn; ++o) {
    mine[o] = owns ? count[tid * kOwn + o] : 0u;
    own += mine[o];
    all += below_all[o];
  }
  const uint32_t incl = wave_inclusive(own, lane), incl_all = wave_inclusive(all, lane);
  if (lane == 63) { part[0][wave] = incl; part[1][wave] = incl_all; }
  __syncthreads();
  int live = 0;                                                  // records of the tile
  uint32_t run = incl - own, run_all = incl_all - all + (t.second ? (uint32_t)a.n : 0u);
#pragma unroll
  for (int w = 0; w < kTileWaves; ++w) {
    live += (int)part[0][w];
    if (w < wave) { run += part[0][w]; run_all += part[1][w]; }
  }
  if (owns) {
#pragma unroll
    for (int o = 0; o < kOwn; ++o) {
      count[tid * kOwn + o] = run;
      out_start[tid * kOwn + o] = run_all + below_tile[o] - run;
      if (t.base == 0 && (uint32_t)(tid * kOwn + o) < t.digits) t.starts[tid * kOwn + o] = run_all;
      run += mine[o];
      run_all += below_all[o];
    }
  }
  if (tile == a.first_tiles && tid == kTileThreads - 1) a.counters[kGroupRecords] = run_all + (owns ? 0u : all);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (row[c] != kNoGroupRow) rank[c] += count[row[c] >> t.row_bits];
  __syncthreads();
  uint32_t* stage = reinterpret_cast<uint32_t*>(bytes);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    if (row[c] != kNoGroupRow) stage[rank[c]] = row[c];
    else rank[c] = kNoGroupRow;
  }
  uint2 val[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    if (rank[c] == kNoGroupRow) continue;
    const int i = c * kTileThreads + tid;
    val[c] = t.second ? make_uint2((uint32_t)(t.base + i), a.second_word) : a.vals[t.base + i];
  }
  __syncthreads();
  uint32_t dest[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int at = c * kTileThreads + tid;
    if (at < live) {
      const uint32_t r = stage[at];
      dest[c] = out_start[r >> t.row_bits] + (uint32_t)at;
      a.rows_mid[dest[c]] = r;
    }
  }
  uint2* vstage = reinterpret_cast<uint2*>(bytes);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (rank[c] != kNoGroupRow) vstage[rank[c]] = val[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    const int at = c * kTileThreads + tid;
    if (at < live) a.vals_mid[dest[c]] = vstage[at];
  }
}

// ---- inside the buckets ----------------------------------------------------------------------
struct BucketOf {
  int64_t base;                  // first record
  int row_bits;
  uint32_t first_row;            // of the rows of its kind
  uint32_t key;                  // of the first row
  uint32_t named;                // the first row's mark
};
__device__ __forceinline__ BucketOf bucket_of(const GroupArgs& a, uint32_t b) {
  BucketOf o;
  o.base = (int64_t)a.starts[b];
  const bool second = b >= a.buckets;
  o.row_bits = second ? a.second_row_bits : a.row_bits;
  o.first_row = (second ? b - a.buckets : b) << o.row_bits;
  o.key = o.first_row + (second ? a.second_key : 0u);
  o.named = o.first_row + (second ? a.buckets << a.row_bits : 0u);
  return o;
}

// count[row] += 1 for the live lanes, and how many came before.  Lanes that name one row are served one after the other (17 cycles each), so rows that
// many lanes of the wave name are added once.
__device__ __forceinline__ uint32_t count_row(uint32_t* count, uint32_t row, bool live) {
  constexpr int kMany = 8;
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(live);
  uint32_t add = live ? 1u : 0u, before = 0u;
  int adds = lane;
  while (todo != 0ull) {
    const int l = __builtin_ctzll(todo);
    const bool same = live && row == (uint32_t)__builtin_amdgcn_readlane((int)row, l);
    const unsigned long long peers = __ballot(same);
    if (__popcll(peers) < kMany) break;
    if (same) {
      adds = l;
      add = lane == l ? (uint32_t)__popcll(peers) : 0u;
      before = (uint32_t)__popcll(peers & ((1ull << lane) - 1ull));
    }
    todo &= ~peers;
  }
  uint32_t at = 0u;
  if (add != 0u) at = atomicAdd(&count[row], add);
  return (uint32_t)__shfl((int)at, adds, 64) + before;
}

// counts of rows into exclusive prefix sums, by the whole workgroup
__device__ __forceinline__ void bucket_scan(uint32_t* count, int rows, uint32_t* part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int per = max(1, rows / kBucketThreads), first = (int)threadIdx.x * per;
  uint32_t own = 0;
  if (first < rows)
    for (int o = 0; o < per; ++o) own += count[first + o];
  const uint32_t incl = wave_inclusive(own, lane);
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  if (first < rows) {
    uint32_t run = incl - own;
#pragma unroll
    for (int w = 0; w < kBucketWaves; ++w)
      if (w < wave) run += part[w];
    for (int o = 0; o < per; ++o) {
      const uint32_t c = count[first + o];
      count[first + o] = run;
      run += c;
    }
  }
  __syncthreads();
}

// What the grouping says of the rows of a bucket of `total` records besides their order, from the rows' first places in it: marks, long rows and
// their segments.  A wave takes 64 rows at a time, and of those every pieces-th one (the pieces of a split bucket share them); its lanes clear a long
// row's slot and enter its segments together.
__device__ __forceinline__ void tell_of_rows(const GroupArgs& a, const BucketOf& b, const uint32_t* first, uint32_t total, uint32_t piece,
                                             uint32_t pieces) {
  const uint32_t rows = 1u << b.row_bits;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  for (uint32_t r0 = (wave * pieces + piece) * 64u; r0 < rows; r0 += kBucketThreads * pieces) {
    const uint32_t r = r0 + lane;
    const uint32_t before = r < rows ? first[r] : total, behind = r + 1u < rows ? first[r + 1u] : total;
    if (a.named != nullptr && r < rows) a.named[b.named + r] = behind != before ? 1 : 0;
    const bool is_long = behind - before > 1u << a.seg_shift;
    const uint32_t slot = (uint32_t)((b.base + before) >> a.seg_shift);
    unsigned long long longs = __ballot(is_long);
    if (longs == 0ull) continue;
    uint32_t at = 0;
    if (lane == 0u) at = atomicAdd(a.counters + kGroupLong, (uint32_t)__popcll(longs));
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (is_long) a.long_rows[at + (uint32_t)__popcll(longs & ((1ull << lane) - 1ull))] = make_uint2(b.key + r, slot);
    for (; longs != 0ull; longs &= longs - 1ull) {
      const int l = __builtin_ctzll(longs);
      const int64_t s = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)slot, l);
      for (int x = (int)lane; x < a.dim; x += 64) a.long_acc[s * a.dim + x] = 0;
      const uint32_t row_first = (uint32_t)b.base + (uint32_t)__builtin_amdgcn_readlane((int)before, l);
      const uint32_t records = (uint32_t)__builtin_amdgcn_readlane((int)(behind - before), l);
      for (uint32_t i = (lane + 1u) << a.seg_shift; i < records; i += 64u << a.seg_shift)
        a.further[(row_first + i) >> a.seg_shift] = make_uint2(row_first + i, row_first);
    }
  }
}

// The pieces in the list of buckets to split: the counts of their rows are added up in global memory.
__device__ __forceinline__ void count_pieces(const GroupArgs& a, uint32_t first_piece, uint32_t stride, uint32_t* count) {
  const int tid = threadIdx.x;
  const uint32_t pieces = a.counters[kGroupPieces];
  for (uint32_t j = first_piece; j < pieces; j += stride) {
    const uint4 piece = a.pieces[j];
    const BucketOf b = bucket_of(a, piece.x);
    const int rows = 1 << b.row_bits;
    const uint32_t* piece_rows = a.rows_mid + b.base + (int64_t)piece.z * kPiece;
    const int live = (int)min((uint32_t)kPiece, a.totals[piece.x] - piece.z * (uint32_t)kPiece);
    for (int r = tid; r < rows; r += kBucketThreads) count[r] = 0u;
    uint32_t row[kPieceItems];
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c)
      row[c] = c * kBucketThreads + tid < live ? piece_rows[c * kBucketThreads + tid] & (uint32_t)(rows - 1) : 0u;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c) count_row(count, row[c], c * kBucketThreads + tid < live);
    __syncthreads();
    for (int r = tid; r < rows; r += kBucketThreads)
      if (count[r] != 0u) atomicAdd(a.row_counts + piece.y + r, count[r]);
    __syncthreads();
  }
}

// A workgroup per bucket; those in the list of buckets to split are left to the workgroups behind them.
template <int ITEMS>
__global__ __launch_bounds__(kBucketThreads, ITEMS <= kBucketItems ? 8 : 4) void group_bucket_kernel(GroupArgs a) {
  constexpr int kMost = kBucketThreads * ITEMS;
  static_assert(kMost * sizeof(uint2) >= sizeof(uint32_t) << kBucketRowBits, "the counters lie where the records are put in order");
  __shared__ __align__(16) unsigned char bytes[kMost * sizeof(uint2)];
  __shared__ uint32_t part[kBucketWaves];
  uint32_t* count = reinterpret_cast<uint32_t*>(bytes);
  const int tid = threadIdx.x;
  if (blockIdx.x >= a.digits) {
    count_pieces(a, blockIdx.x - a.digits, gridDim.x - a.digits, count);
    return;
  }
  const uint32_t total = a.totals[blockIdx.x];
  if (total > (uint32_t)kMost) return;
  const int live = (int)total;
  const bool second = blockIdx.x >= a.buckets;
  const int rows = 1 << (second ? a.second_row_bits : a.row_bits);
  const uint32_t mask = (uint32_t)rows - 1u;
  for (int r = tid; r < rows; r += kBucketThreads) count[r] = 0u;
  const BucketOf b = bucket_of(a, blockIdx.x);
  __syncthreads();
  if (total == 0u) {
    if (a.named != nullptr)
      for (int r = tid; r < rows; r += kBucketThreads) a.named[b.named + r] = 0;
    return;
  }
  const uint32_t* my_rows = a.rows_mid + b.base;
  const uint2* my_vals = a.vals_mid + b.base;
  uint32_t* keys_to = a.keys_out + b.base;
  uint2* vals_to = a.vals_out + b.base;
  // a record's row in the bucket, and above it its rank in the row, then its place in the bucket
  static_assert(kMost <= 1 << (32 - kBucketRowBits), "both fit 32 bits");
  constexpr uint32_t kRowMask = (1u << kBucketRowBits) - 1u;
  uint32_t at[ITEMS];
  uint2 val[ITEMS];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) at[c] = my_rows[c * kBucketThreads + tid] & mask;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) val[c] = my_vals[c * kBucketThreads + tid];
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) at[c] |= atomicAdd(&count[at[c]], 1u) << kBucketRowBits;
  __syncthreads();
  bucket_scan(count, rows, part);
  tell_of_rows(a, b, count, total, 0u, 1u);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) at[c] += count[at[c] & kRowMask] << kBucketRowBits;
  __syncthreads();
  uint2* vstage = reinterpret_cast<uint2*>(bytes);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) vstage[at[c] >> kBucketRowBits] = val[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) vals_to[c * kBucketThreads + tid] = vstage[c * kBucketThreads + tid];
  __syncthreads();
  uint32_t* stage = reinterpret_cast<uint32_t*>(bytes);
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) stage[at[c] >> kBucketRowBits] = b.key + (at[c] & kRowMask);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < ITEMS; ++c)
    if (c * kBucketThreads + tid < live) keys_to[c * kBucketThreads + tid] = stage[c * kBucketThreads + tid];
}

// The pieces in the list: a piece takes the next places of its rows and moves its records there.
// ROW_BITS: the most of either kind of buckets.
template <int ROW_BITS>
__global__ __launch_bounds__(kBucketThreads) void group_split_kernel(GroupArgs a) {
  __shared__ uint32_t first[1 << ROW_BITS];                // of a row of the bucket: the records before it,
  __shared__ uint32_t count[1 << ROW_BITS];                // those of this piece, then the place of the first of them
  __shared__ uint32_t part[kBucketWaves];
  const int tid = threadIdx.x;
  const uint32_t pieces = a.counters[kGroupPieces];
  for (uint32_t j = blockIdx.x; j < pieces; j += gridDim.x) {
    const uint4 piece = a.pieces[j];
    const BucketOf b = bucket_of(a, piece.x);
    const int rows = 1 << b.row_bits;
    const uint32_t mask = (uint32_t)rows - 1u, total = a.totals[piece.x];
    const int64_t base = b.base + (int64_t)piece.z * kPiece;
    const int live = (int)min((uint32_t)kPiece, total - piece.z * (uint32_t)kPiece);
    for (int r = tid; r < rows; r += kBucketThreads) {
      first[r] = a.row_counts[piece.y + r];
      count[r] = 0u;
    }
    uint32_t row[kPieceItems], rank[kPieceItems];
    uint2 val[kPieceItems];                                            // (asked for here: between the stores below each would be waited for)
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c)
      row[c] = c * kBucketThreads + tid < live ? a.rows_mid[base + c * kBucketThreads + tid] & mask : 0u;
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c)
      if (c * kBucketThreads + tid < live) val[c] = a.vals_mid[base + c * kBucketThreads + tid];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c)
      rank[c] = count_row(count, row[c], c * kBucketThreads + tid < live);
    bucket_scan(first, rows, part);
    for (int r = tid; r < rows; r += kBucketThreads)
      if (count[r] != 0u) count[r] = first[r] + atomicAdd(a.row_taken + piece.y + r, count[r]);
    tell_of_rows(a, b, first, total, piece.z, piece.w);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kPieceItems; ++c)
      if (c * kBucketThreads + tid < live) {
        const int64_t at = b.base + count[row[c]] + rank[c];
        a.keys_out[at] = b.key + row[c];
        a.vals_out[at] = val[c];
      }
    __syncthreads();
  }
}

// ---- host side -------------------------------------------------------------------------------
struct GroupPlan {
  int row_bits, second_row_bits;
  int64_t buckets, second_buckets;
  int tile;                      // records of a tile
  int bucket_items;              // records per lane of a bucket's workgroup
  int64_t first_tiles, tiles;
};

// the fewest buckets of a power of two of rows that hold about kBucketMean records each
static int row_bits_for(int64_t n, int64_t rows, int64_t most_buckets) {
  const int64_t mean = std::min(kBucketMean, std::max(kBucketMeanLeast, ceil_div(n, kBusyBuckets)));
  int bits = kBucketRowBits;
  while (bits > 0 && ceil_div(n, ceil_div(rows, (int64_t)1 << bits)) > mean &&
         ceil_div(rows, (int64_t)1 << (bits - 1)) <= most_buckets)
    --bits;
  return bits;
}

static GroupPlan plan_group(int64_t n, int64_t second_n, int64_t rows) {
  GroupPlan p;
  p.row_bits = row_bits_for(n, rows, kBuckets);
  p.second_row_bits = row_bits_for(second_n, rows, kSecondBuckets);
  p.buckets = ceil_div(rows, (int64_t)1 << p.row_bits);
  p.second_buckets = ceil_div(rows, (int64_t)1 << p.second_row_bits);
  p.tile = n >= kLargestGroupTiles ? 16384 : (n >= kLargeGroupTiles ? 8192 : (n >= kMidGroupTiles ? 4096 : 2048));
  p.bucket_items = ceil_div(n, p.buckets) > kBucketMeanMost ? kBucketItemsMost : kBucketItems;
  p.first_tiles = ceil_div(n, p.tile);
  p.tiles = p.first_tiles + ceil_div(second_n, p.tile);
  return p;
}

bool can_group(int64_t rows) { return ceil_div(rows, (int64_t)1 << kBucketRowBits) <= kSecondBuckets; }

// Buckets of more records than a workgroup takes, all of which are split, and of more rows than let two workgroups of the splitting launch share a
// compute unit.  Steps, us, grouped / sorted: 16 M rows 30 M records 2992 / 3268, 34 M 3861 / 3666, 72 M 7796 / 7114; 8 M rows 36 M 3651 /
// 3708, 60 M 5922 / 5832; 4 M rows 36 M 3360 / 3526, 120 M 10641 / 10953; 100 k rows 48 M 3882 / 3868.
bool group_crowded(int64_t n, int64_t rows) {
  const int bits = row_bits_for(n, rows, kBuckets);
  return bits > kFewRowBits && ceil_div(n, ceil_div(rows, (int64_t)1 << bits)) > kBucketThreads * kBucketItemsMost;
}

// The most records of a kind that are grouped in buckets of 2^bits rows or more (behind it, there are more buckets of fewer rows); 0: no border.
int64_t group_border(int64_t rows, bool second, int bits) {
  if (bits <= 0 || bits > kBucketRowBits || ceil_div(rows, (int64_t)1 << (bits - 1)) > (second ? kSecondBuckets : kBuckets)) return 0;
  const int64_t buckets = ceil_div(rows, (int64_t)1 << bits);
  return buckets * (buckets >= kBusyBuckets ? kBucketMean : kBucketMeanLeast);
}

// (but for the rows of the buckets to split, which are fewer behind a border, no array is smaller for more records)
void group_take(GroupArgs& a, Carver& cv, int64_t n, int64_t second_n, int64_t rows, int32_t seg_shift, bool marks) {
  const GroupPlan p = plan_group(n, second_n, rows);
  a.digits = (uint32_t)(p.buckets + p.second_buckets);
  size_t counts = 0;                             // (there are fewer tiles where they are larger)
  for (const int64_t m : {n, std::min(n, kMidGroupTiles - 1), std::min(n, kLargeGroupTiles - 1), std::min(n, kLargestGroupTiles - 1)}) {
    const GroupPlan q = plan_group(m, second_n, rows);
    counts = std::max(counts, (size_t)q.first_tiles * (size_t)q.buckets + (size_t)(q.tiles - q.first_tiles) * (size_t)q.second_buckets);
  }
  const size_t records = (size_t)(n + second_n);
  const size_t split = records / (size_t)(kBucketThreads * kBucketItems) + 1;        // (each has more records than that)
  const size_t all_rows = 2 * ((size_t)rows + ((size_t)1 << kBucketRowBits));        // of the buckets of both kinds
  auto split_rows_of = [&](int64_t m, int64_t buckets, int row_bits) {
    return (size_t)std::min(m / (kBucketThreads * kBucketItems) + 1, buckets) << row_bits;
  };
  const size_t split_rows = split_rows_of(n, p.buckets, p.row_bits) + split_rows_of(second_n, p.second_buckets, p.second_row_bits);
  // (the marks are written when the counts have been read for the last time)
  a.counts = cv.take<uint32_t>(marks ? std::max(counts, all_rows / sizeof(uint32_t)) : counts);
  a.named = marks ? reinterpret_cast<uint8_t*>(a.counts) : nullptr;
  a.totals = cv.take<uint32_t>((size_t)(kBuckets + kSecondBuckets));
  a.starts = cv.take<uint32_t>((size_t)(kBuckets + kSecondBuckets));
  a.counters = cv.take<uint32_t>(kGroupCounters);
  a.pieces = cv.take<uint4>(records / kPiece + split);
  a.row_counts = cv.take<uint32_t>(split_rows);
  a.row_taken = cv.take<uint32_t>(split_rows);
  a.long_rows = cv.take<uint2>((records >> seg_shift) + 1);
  a.further = cv.take<uint2>((records >> seg_shift) + 2);
  a.second_named = (uint32_t)(p.buckets << p.row_bits);
}

template <int kTileThreads, int ITEMS, int DIGITS>
static int32_t launch_scatter(const GroupArgs& a, hipStream_t stream) {
  group_count_kernel<kTileThreads, ITEMS, DIGITS><<<(unsigned)a.tiles, kTileThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  group_scan_kernel<<<a.first_scans + (unsigned)ceil_div(a.digits - a.buckets, kScanDigits), 1024, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  group_scatter_kernel<kTileThreads, ITEMS, DIGITS><<<(unsigned)(8 * a.tiles_per_xcd), kTileThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
template <int ITEMS>
static int32_t launch_buckets(const GroupArgs& a, hipStream_t stream) {
  group_bucket_kernel<ITEMS><<<a.digits + kSplitBlocks, kBucketThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  if (std::max(a.row_bits, a.second_row_bits) <= kFewRowBits) group_split_kernel<kFewRowBits><<<kSplitBlocks, kBucketThreads, 0, stream>>>(a);
  else group_split_kernel<kBucketRowBits><<<kSplitBlocks, kBucketThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

int32_t group_rows(GroupArgs a, int64_t rows, hipStream_t stream) {
  const GroupPlan p = plan_group(a.n, a.second_n, rows);
  a.row_bits = p.row_bits;
  a.second_row_bits = p.second_row_bits;
  a.buckets = (uint32_t)p.buckets;
  a.first_tiles = p.first_tiles;
  a.first_scans = (uint32_t)ceil_div(p.buckets, kScanDigits);
  a.tiles = p.tiles;
  a.tiles_per_xcd = ceil_div(p.tiles, 8);
  a.most = (uint32_t)(kBucketThreads * p.bucket_items);
  auto scatter = launch_scatter<512, 4, 256>;
  const int64_t digits = std::max(p.buckets, p.second_buckets);
  if (p.tile == 2048) scatter = digits <= 256 ? scatter : (digits <= 1024 ? launch_scatter<512, 4, 1024> : launch_scatter<512, 4, 2048>);
  else if (p.tile == 4096) scatter = digits <= 256 ? launch_scatter<512, 8, 256> : (digits <= 1024 ? launch_scatter<512, 8, 1024> : launch_scatter<512, 8, 2048>);
  else if (p.tile == 8192) scatter = digits <= 256 ? launch_scatter<512, 16, 256> : (digits <= 1024 ? launch_scatter<512, 16, 1024> : launch_scatter<512, 16, 2048>);
  else scatter = digits <= 1024 ? launch_scatter<1024, 16, 1024> : launch_scatter<1024, 16, 2048>;
  const int32_t rc = scatter(a, stream);
  if (rc != GS_OK) return rc;
  return p.bucket_items == kBucketItems ? launch_buckets<kBucketItems>(a, stream) : launch_buckets<kBucketItemsMost>(a, stream);
}

}  // namespace gs
