// gs_csr_build: edge list -> CSR on the device (GraphScale Sec. 3.1: the
// topology a trainer keeps).  Records (src << id_bits | dst, weight) are sorted
// stably, duplicates are flagged, and the survivors are compacted.
#include "common.h"

namespace gs {

constexpr uint64_t kDroppedKey = ~0ull;

// The weight travels with its key (the sort is stable: among equal keys the one from the lowest
// input index stays first), so nothing is gathered from the edge list afterwards; without weights
// the keys travel alone, because equal keys cannot be told apart.
__global__ void csr_keygen_kernel(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                  const float* __restrict__ w, int64_t cap, int64_t num_nodes, uint32_t flags,
                                  int id_bits, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= cap) return;
  const bool sym = flags & GS_SYMMETRIZE;
  const int64_t i = sym ? (e >> 1) : e;
  int32_t s = src[i], d = dst[i];
  if (sym && (e & 1)) { int32_t t = s; s = d; d = t; }
  const bool ok = s >= 0 && d >= 0 && s < num_nodes && d < num_nodes &&
                  !((flags & GS_DROP_SELF_LOOPS) && s == d);
  keys[e] = ok ? (((uint64_t)(uint32_t)s << id_bits) | (uint64_t)(uint32_t)d) : kDroppedKey;
  if (w != nullptr) vals[e] = __float_as_uint(w[i]);
}

// Compaction: a block takes kCompactTile consecutive records, counts the kept ones (first kernel)
// and, once the counts of the tiles are summed, moves them (second kernel).  In both, a wave takes
// its share 64 records at a time, so the place of a record is its rank among the lanes' votes.  Bound by
// memory: 23 million records of 8 + 4 bytes, 38 us to count (4.8 TB/s) and 90 us to move (5.7 TB/s read and
// written), against 465 + 80 us and a scan of one 64-bit flag per record.
constexpr int kCompactThreads = 256;
constexpr int kCompactWaves = kCompactThreads / 64;
constexpr int kCompactItems = 8;                              // records per lane
constexpr int kCompactTile = kCompactThreads * kCompactItems;

// The wave's records, `first` being the lane's first of them, and which are kept.  All reads are
// issued before any is used (behind the end: the last record again).
__device__ __forceinline__ void csr_keeps(const uint64_t* __restrict__ keys, int64_t first, int64_t cap, bool dedupe,
                                          uint64_t (&key)[kCompactItems], bool (&keep)[kCompactItems]) {
  uint64_t before[kCompactItems];
#pragma unroll
  for (int c = 0; c < kCompactItems; ++c) {
    const int64_t e = min(first + c * 64, cap - 1);
    key[c] = keys[e];
    before[c] = keys[max((int64_t)0, e - 1)];
  }
#pragma unroll
  for (int c = 0; c < kCompactItems; ++c) {
    const int64_t e = first + c * 64;
    keep[c] = e < cap && key[c] != kDroppedKey && !(dedupe && e > 0 && before[c] == key[c]);
  }
}

__global__ __launch_bounds__(kCompactThreads) void csr_count_kernel(const uint64_t* __restrict__ keys, int64_t cap,
                                                                    uint32_t flags, int64_t* __restrict__ tile_counts) {
  __shared__ uint32_t wave_kept[kCompactWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * kCompactTile + wave * (64 * kCompactItems) + lane;
  uint64_t key[kCompactItems];
  bool keep[kCompactItems];
  csr_keeps(keys, first, cap, flags & GS_DEDUPE, key, keep);
  uint32_t kept = 0;
#pragma unroll
  for (int c = 0; c < kCompactItems; ++c) kept += (uint32_t)__popcll(__ballot(keep[c]));
  if (lane == 0) wave_kept[wave] = kept;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t sum = 0;
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) sum += wave_kept[w];
    tile_counts[blockIdx.x] = sum;
  }
}

__global__ __launch_bounds__(kCompactThreads) void csr_compact_kernel(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, const int64_t* __restrict__ tile_first,
    int64_t cap, uint32_t flags, int id_bits, int32_t* __restrict__ nbrs_out, float* __restrict__ w_out,
    int32_t* __restrict__ row_of) {
  __shared__ uint32_t wave_kept[kCompactWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * kCompactTile + wave * (64 * kCompactItems) + lane;
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t place[kCompactItems];                              // among the wave's kept records
  uint64_t key[kCompactItems];
  bool keep[kCompactItems];
  csr_keeps(keys, first, cap, flags & GS_DEDUPE, key, keep);
  uint32_t val[kCompactItems];
  if (vals != nullptr)
#pragma unroll
    for (int c = 0; c < kCompactItems; ++c) val[c] = vals[min(first + c * 64, cap - 1)];
  uint32_t kept = 0;
#pragma unroll
  for (int c = 0; c < kCompactItems; ++c) {
    const uint64_t votes = __ballot(keep[c]);
    place[c] = kept + (uint32_t)__popcll(votes & below);
    kept += (uint32_t)__popcll(votes);
  }
  if (lane == 0) wave_kept[wave] = kept;
  __syncthreads();
  int64_t at = tile_first[blockIdx.x];
#pragma unroll
  for (int w = 0; w < kCompactWaves; ++w)
    if (w < wave) at += wave_kept[w];
#pragma unroll
  for (int c = 0; c < kCompactItems; ++c) {
    if (!keep[c]) continue;
    const int64_t p = at + place[c];
    nbrs_out[p] = (int32_t)(key[c] & ((1ull << id_bits) - 1ull));
    row_of[p] = (int32_t)(key[c] >> id_bits);
    if (vals != nullptr) w_out[p] = __uint_as_float(val[c]);
  }
}

// offsets[v] = number of kept entries whose row is < v  (lower bound in row_of)
template <typename OffT>
__global__ void csr_offsets_kernel(const int32_t* __restrict__ row_of,
                                   const int64_t* __restrict__ num_entries, int64_t num_nodes,
                                   OffT* __restrict__ offsets) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v > num_nodes) return;
  int64_t lo = 0, hi = *num_entries;
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    if ((int64_t)row_of[mid] < v) lo = mid + 1; else hi = mid;
  }
  offsets[v] = (OffT)lo;
}

static int bits_for(int64_t n) {  // bits needed for ids in [0, n)
  int b = 1;
  while (b < 32 && ((int64_t)1 << b) < n) ++b;
  return b;
}

struct CsrPlan {
  uint64_t *keys, *keys_alt;
  uint32_t *vals, *vals_alt;     // weighted graphs only use them
  int64_t *tile_first, *scan_scratch;
  int32_t* row_of;
  void* sort_scratch;            // (in the place of row_of, which is written when the records are sorted)
  size_t sort_bytes;
  size_t bytes;
};

static CsrPlan plan_csr(void* ws, int64_t cap) {
  Carver cv(ws);
  CsrPlan p;
  const size_t c = (size_t)(cap > 0 ? cap : 1);
  const int64_t tiles = ceil_div((int64_t)c, kCompactTile);
  p.keys = cv.take<uint64_t>(c);
  p.keys_alt = cv.take<uint64_t>(c);
  p.vals = cv.take<uint32_t>(c);
  p.vals_alt = cv.take<uint32_t>(c);
  p.tile_first = cv.take<int64_t>((size_t)tiles);
  p.scan_scratch = cv.take<int64_t>(scan_scratch_elems(tiles));
  p.sort_bytes = std::max(c * sizeof(int32_t), radix_sort_scratch_bytes((int64_t)c, true));
  p.sort_scratch = cv.take<char>(p.sort_bytes);
  p.row_of = static_cast<int32_t*>(p.sort_scratch);
  p.bytes = cv.used;
  return p;
}

}  // namespace gs

using namespace gs;

extern "C" size_t gs_csr_build_workspace_bytes(int64_t m, int64_t num_nodes, uint32_t flags) {
  (void)num_nodes;
  if (m < 0) return 0;
  const int64_t cap = (flags & GS_SYMMETRIZE) ? 2 * m : m;
  return plan_csr(nullptr, cap).bytes;
}

extern "C" int32_t gs_csr_build(const int32_t* src, const int32_t* dst, const float* w, int64_t m,
                                int64_t num_nodes, uint32_t flags, int32_t offset_bits,
                                void* offsets_out, int32_t* nbrs_out, float* w_out,
                                int64_t* num_entries_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (m < 0 || num_nodes < 0 || num_nodes > (int64_t)INT32_MAX) return GS_EINVAL;
  if (offset_bits != 32 && offset_bits != 64) return GS_EINVAL;
  if (flags & ~(uint32_t)(GS_SYMMETRIZE | GS_DROP_SELF_LOOPS | GS_DEDUPE)) return GS_EINVAL;
  if (m > 0 && (!src || !dst)) return GS_EINVAL;
  if (!offsets_out || !num_entries_out) return GS_EINVAL;
  if (w != nullptr && w_out == nullptr) return GS_EINVAL;
  if (m > (int64_t)INT32_MAX) return GS_EOVERFLOW;
  const int64_t cap = (flags & GS_SYMMETRIZE) ? 2 * m : m;
  if (offset_bits == 32 && cap > (int64_t)INT32_MAX) return GS_EOVERFLOW;
  if (cap > 0 && !nbrs_out) return GS_EINVAL;
  if (!ws || !aligned(ws, 256)) return GS_EINVAL;
  CsrPlan p = plan_csr(ws, cap);
  if (ws_bytes < p.bytes) return GS_EWORKSPACE;

  const int threads = 256;
  const int64_t tiles = ceil_div(cap, kCompactTile);
  const int nb = bits_for(num_nodes);
  if (cap > 0) {
    // ids take nb bits; dropped records, all of whose bits are set, sort last: their source id is no node's unless
    // the nodes fill the nb bits, and then the key has one bit more.
    // The passes go back and forth between two buffers and end in (keys, vals).
    const int key_bits = 2 * nb + (num_nodes < ((int64_t)1 << nb) ? 0 : 1);
    const SortPlan sort = radix_sort_plan(cap, key_bits, p.sort_bytes);
    const bool odd = sort.passes & 1;
    uint64_t* made = odd ? p.keys_alt : p.keys;
    uint32_t* made_vals = w == nullptr ? nullptr : (odd ? p.vals_alt : p.vals);
    csr_keygen_kernel<<<(unsigned)ceil_div(cap, threads), threads, 0, stream>>>(src, dst, w, cap, num_nodes, flags, nb,
                                                                               made, made_vals);
    GS_LAUNCH_CHECK();
    const int32_t rc = radix_sort<uint64_t>(sort, made, made_vals, p.keys, p.vals, p.keys_alt, p.vals_alt, cap, kDroppedKey,
                                            key_bits, p.sort_scratch, stream);
    if (rc != GS_OK) return rc;
    csr_count_kernel<<<(unsigned)tiles, kCompactThreads, 0, stream>>>(p.keys, cap, flags, p.tile_first);
    GS_LAUNCH_CHECK();
  }
  const int32_t rc = exclusive_scan_i64(p.tile_first, tiles, p.scan_scratch, num_entries_out, stream);
  if (rc != GS_OK) return rc;
  if (cap > 0) {
    csr_compact_kernel<<<(unsigned)tiles, kCompactThreads, 0, stream>>>(
        p.keys, w != nullptr ? p.vals : nullptr, p.tile_first, cap, flags, nb, nbrs_out, w_out, p.row_of);
    GS_LAUNCH_CHECK();
  }
  const unsigned oblocks = (unsigned)ceil_div(num_nodes + 1, threads);
  if (offset_bits == 64)
    csr_offsets_kernel<int64_t><<<oblocks, threads, 0, stream>>>(p.row_of, num_entries_out, num_nodes,
                                                                (int64_t*)offsets_out);
  else
    csr_offsets_kernel<int32_t><<<oblocks, threads, 0, stream>>>(p.row_of, num_entries_out, num_nodes,
                                                                (int32_t*)offsets_out);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
