// gs_make_pairs and gs_sample_negatives (GraphScale Sec. 2.2: skip-gram with
// negative sampling over the walks; Sec. 3.2: the positively and negatively
// sampled nodes of a batch).
#include "common.h"

namespace gs {

__global__ void pairs_count_kernel(const int32_t* __restrict__ walks, int64_t num_walks,
                                   int32_t walk_len, int32_t window, int64_t* __restrict__ counts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= num_walks) return;
  const int32_t len = valid_prefix(walks + i * (int64_t)walk_len, walk_len);
  counts[i] = 2 * window_prefix(len, window);
}

// Pairs of a block's walks, staged in LDS.  The lanes are dealt out in equal groups, one walk per
// group; a lane makes four consecutive pairs of the walk at a time: the closed form gives the
// first, the next three follow from it by stepping the context (and, where its window ends, the
// centre), and the four leave as one 16-byte store per output array (the pairs of a walk start
// anywhere, so the stores are aligned to four bytes only; neighbouring lanes fill whole lines).
// Bound by the 8 bytes written per pair: 29 million pairs of 30,000 walks of 80 nodes in 48 us (4.8
// TB/s); one pair per lane, found by two 64-bit binary searches, took 613 us (arithmetic).
constexpr int kEmitThreads = 256;
constexpr int kEmitLdsInts = 10240;   // staged walks: walks_per_block * walk_len <= this
constexpr int kEmitMaxWalks = 16;     // 16 lanes per walk, and more where fewer walks fit
struct __attribute__((packed, aligned(4))) PairQuad { int32_t v[4]; };

// pairs_before() of a walk prefix of len <= 4096 nodes: fewer than 2^24 pairs, so 32 bits do
__device__ __forceinline__ uint32_t window_prefix32(uint32_t x, uint32_t w) {
  return (x <= w + 1) ? x * (x - 1) / 2 : w * (w + 1) / 2 + (x - w - 1) * w;
}

__device__ __forceinline__ uint32_t pairs_before32(uint32_t a, uint32_t len, uint32_t w, uint32_t f_len) {
  return window_prefix32(a, w) + f_len - window_prefix32(len - a, w);
}

__global__ __launch_bounds__(kEmitThreads) void pairs_emit_kernel(
    const int32_t* __restrict__ walks, int64_t num_walks, int32_t walk_len, int32_t window_arg,
    int walks_per_block, const int64_t* __restrict__ bases, int32_t* __restrict__ centers,
    int32_t* __restrict__ contexts) {
  extern __shared__ int32_t rows[];                          // [walks_per_block][walk_len]
  const int64_t w0 = (int64_t)blockIdx.x * walks_per_block;
  const int here = (int)min((int64_t)walks_per_block, num_walks - w0);
  const int ints = here * walk_len;
  const int32_t* src = walks + w0 * (int64_t)walk_len;
  for (int x = threadIdx.x; x < ints; x += kEmitThreads) rows[x] = src[x];
  __syncthreads();
  const int lanes = kEmitThreads / walks_per_block;
  const int g = threadIdx.x / lanes, l = threadIdx.x - g * lanes;
  if (g >= here) return;
  const int32_t* row = rows + g * walk_len;
  const int32_t len = valid_prefix(row, walk_len);
  const int32_t window = min(window_arg, walk_len);          // (a wider one names no further position)
  const uint32_t f_len = window_prefix32((uint32_t)len, (uint32_t)window);
  const uint32_t count = 2u * f_len;
  // centres at least `window` positions from both ends have 2 * window pairs each; `edge` pairs
  // come before them, and as many after
  const bool interior = len > 2 * window;
  const uint32_t edge = interior ? pairs_before32((uint32_t)window, (uint32_t)len, (uint32_t)window, f_len) : count;
  const float per_center = 1.0f / (float)(2 * window);
  int32_t* c_out = centers + bases[w0 + g];
  int32_t* o_out = contexts + bases[w0 + g];
  for (uint32_t q = 4u * (uint32_t)l; q < count; q += 4u * (uint32_t)lanes) {
    // centre position of pair q: the last a with pairs_before(a) <= q
    uint32_t lo = 0, hi = (uint32_t)len - 1;
    if (interior && q >= edge && q < count - edge) {
      const uint32_t t = q - edge, wide = 2u * (uint32_t)window;
      uint32_t e = (uint32_t)((float)t * per_center);        // t < 2^24: off by one at most
      if (e * wide > t) --e;
      else if ((e + 1u) * wide <= t) ++e;
      lo = hi = (uint32_t)window + e;
    } else if (interior) {
      if (q < edge) hi = (uint32_t)window - 1;
      else lo = (uint32_t)(len - window);
    }
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (pairs_before32(mid, (uint32_t)len, (uint32_t)window, f_len) <= q) lo = mid; else hi = mid - 1;
    }
    int32_t a = (int32_t)lo;
    int32_t o = max(0, a - window) + (int32_t)(q - pairs_before32(lo, (uint32_t)len, (uint32_t)window, f_len));
    if (o >= a) ++o;
    PairQuad c4, o4;
    const int n = (int)min(4u, count - q);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < n) { c4.v[i] = row[a]; o4.v[i] = row[o]; }
      ++o;
      if (o == a) ++o;
      if (o > min(len - 1, a + window)) { ++a; o = max(0, a - window); }
    }
    if (n == 4) {
      *reinterpret_cast<PairQuad*>(c_out + q) = c4;
      *reinterpret_cast<PairQuad*>(o_out + q) = o4;
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if (i < n) { c_out[q + i] = c4.v[i]; o_out[q + i] = o4.v[i]; }
    }
  }
}

__global__ void negatives_kernel(const float* __restrict__ prob, const int32_t* __restrict__ alias,
                                 const uint2* __restrict__ packed,
                                 uint64_t num_nodes, int64_t total, uint64_t pair_base, int32_t k,
                                 uint64_t seed, int32_t* __restrict__ negs) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const uint64_t i = (uint64_t)(e / k);
  const uint32_t j = (uint32_t)(e - (int64_t)i * k);
  const Block4 b = philox_at(seed, pair_base + i, j, 0x80000000u);
  negs[e] = (int32_t)table_draw(prob, alias, packed, num_nodes, b);
}

// One lane per LINE sample: draw an entry, then find the row that holds it
// (the last row whose offset is <= e; empty rows share their offset with the
// next row and are skipped by taking the last one).
template <typename OffT>
__global__ void edges_kernel(const OffT* __restrict__ offsets, int64_t num_nodes,
                             const int32_t* __restrict__ nbrs, uint64_t num_entries,
                             const float* __restrict__ prob, const int32_t* __restrict__ alias,
                             const uint2* __restrict__ packed, int64_t num_samples,
                             uint64_t sample_base, uint64_t seed, int32_t* __restrict__ centers,
                             int32_t* __restrict__ contexts) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= num_samples) return;
  const Block4 b = philox_at(seed, sample_base + (uint64_t)i, 0u, 0x40000000u);
  const int64_t e = table_draw(prob, alias, packed, num_entries, b);
  const int32_t dst = nbrs[e];
  // first t in [1, num_nodes] with offsets[t] > e; offsets[num_nodes] = num_entries > e
  int64_t lo = 1, hi = num_nodes;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)offsets[mid] > e) hi = mid; else lo = mid + 1;
  }
  centers[i] = (int32_t)(lo - 1);
  contexts[i] = dst;
}

struct PairsPlan {
  int64_t *bases, *scan_scratch;
  size_t bytes;
};
static PairsPlan plan_pairs(void* ws, int64_t num_walks) {
  Carver cv(ws);
  PairsPlan p;
  const size_t n = (size_t)(num_walks > 0 ? num_walks : 1);
  p.bases = cv.take<int64_t>(n);
  p.scan_scratch = cv.take<int64_t>(scan_scratch_elems((int64_t)n));
  p.bytes = cv.used;
  return p;
}

}  // namespace gs

using namespace gs;

extern "C" size_t gs_make_pairs_workspace_bytes(int64_t num_walks) {
  if (num_walks < 0) return 0;
  return plan_pairs(nullptr, num_walks).bytes;
}

extern "C" int32_t gs_make_pairs(const int32_t* walks, int64_t num_walks, int32_t walk_len,
                                 int32_t window, int32_t* centers_out, int32_t* contexts_out,
                                 int64_t* num_pairs_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (num_walks < 0 || walk_len < 1 || walk_len > 4096 || window < 1 || !num_pairs_out)
    return GS_EINVAL;
  if (num_walks > 0 && !walks) return GS_EINVAL;
  if (!ws || !aligned(ws, 256)) return GS_EINVAL;
  PairsPlan p = plan_pairs(ws, num_walks);
  if (ws_bytes < p.bytes) return GS_EWORKSPACE;
  const bool may_emit = walk_len > 1;
  if (num_walks > 0 && may_emit && (!centers_out || !contexts_out)) return GS_EINVAL;
  if (num_walks > 0) {
    pairs_count_kernel<<<(unsigned)ceil_div(num_walks, 256), 256, 0, stream>>>(walks, num_walks, walk_len,
                                                                             window, p.bases);
    GS_LAUNCH_CHECK();
  }
  int32_t rc = exclusive_scan_i64(p.bases, num_walks, p.scan_scratch, num_pairs_out, stream);
  if (rc != GS_OK) return rc;
  if (num_walks > 0 && may_emit) {
    int wpb = kEmitMaxWalks;                       // a power of two: the lanes divide evenly
    while (wpb > 1 && wpb * walk_len > kEmitLdsInts) wpb >>= 1;
    pairs_emit_kernel<<<(unsigned)ceil_div(num_walks, wpb), kEmitThreads, (size_t)wpb * walk_len * sizeof(int32_t),
                        stream>>>(walks, num_walks, walk_len, window, wpb, p.bases, centers_out, contexts_out);
    GS_LAUNCH_CHECK();
  }
  return GS_OK;
}

extern "C" size_t gs_pair_offsets_workspace_bytes(int64_t num_walks) {
  if (num_walks < 0) return 0;
  Carver cv(nullptr);
  cv.take<int64_t>(scan_scratch_elems(num_walks > 0 ? num_walks : 1));
  return cv.used;
}

extern "C" int32_t gs_pair_offsets(const int32_t* walks, int64_t num_walks, int32_t walk_len,
                                   int32_t window, int64_t* offsets_out, void* ws, size_t ws_bytes,
                                   void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (num_walks < 0 || walk_len < 1 || walk_len > 4096 || window < 1 || !offsets_out) return GS_EINVAL;
  if (num_walks > 0 && !walks) return GS_EINVAL;
  if (!ws || !aligned(ws, 256)) return GS_EINVAL;
  if (ws_bytes < gs_pair_offsets_workspace_bytes(num_walks)) return GS_EWORKSPACE;
  if (num_walks > 0) {
    pairs_count_kernel<<<(unsigned)ceil_div(num_walks, 256), 256, 0, stream>>>(walks, num_walks, walk_len,
                                                                             window, offsets_out);
    GS_LAUNCH_CHECK();
  }
  // exclusive sums in place; the total goes to the entry after the last walk
  return exclusive_scan_i64(offsets_out, num_walks, static_cast<int64_t*>(ws), offsets_out + num_walks,
                            stream);
}

extern "C" int32_t gs_sample_negatives(const gs_alias* noise, int64_t num_nodes, int64_t num_pairs,
                                       uint64_t pair_index_base, int32_t k, uint64_t seed,
                                       int32_t* negs_out, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (num_nodes < 1 || num_nodes > (int64_t)INT32_MAX || num_pairs < 0 || k < 0) return GS_EINVAL;
  if (num_pairs > 0 && k > 0 && !negs_out) return GS_EINVAL;
  const bool weighted = noise != nullptr && noise->prob != nullptr;
  if (weighted && !noise->alias) return GS_EINVAL;
  const int64_t total = num_pairs * (int64_t)k;
  if (total == 0) return GS_OK;
  if (ceil_div(total, 256) > (int64_t)INT32_MAX) return GS_EOVERFLOW;
  negatives_kernel<<<(unsigned)ceil_div(total, 256), 256, 0, stream>>>(
      weighted ? noise->prob : nullptr, weighted ? noise->alias : nullptr,
      weighted ? reinterpret_cast<const uint2*>(noise->packed) : nullptr, (uint64_t)num_nodes, total,
      pair_index_base, k, seed, negs_out);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

extern "C" int32_t gs_sample_edges(const gs_csr* g, const gs_alias* edge_alias, int64_t num_samples,
                                   uint64_t sample_index_base, uint64_t seed, int32_t* centers_out,
                                   int32_t* contexts_out, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!g || g->num_nodes < 1 || g->num_nodes > (int64_t)INT32_MAX || g->num_entries < 1 ||
      !g->offsets || !g->nbrs || num_samples < 0)
    return GS_EINVAL;
  if (g->offset_bits != 32 && g->offset_bits != 64) return GS_EINVAL;
  if (num_samples > 0 && (!centers_out || !contexts_out)) return GS_EINVAL;
  const bool weighted = edge_alias != nullptr && edge_alias->prob != nullptr;
  if (weighted && !edge_alias->alias) return GS_EINVAL;
  if (num_samples == 0) return GS_OK;
  if (ceil_div(num_samples, 256) > (int64_t)INT32_MAX) return GS_EOVERFLOW;
  const float* prob = weighted ? edge_alias->prob : nullptr;
  const int32_t* alias = weighted ? edge_alias->alias : nullptr;
  const uint2* packed = weighted ? reinterpret_cast<const uint2*>(edge_alias->packed) : nullptr;
  const unsigned blocks = (unsigned)ceil_div(num_samples, 256);
  if (g->offset_bits == 32)
    edges_kernel<int32_t><<<blocks, 256, 0, stream>>>(
        static_cast<const int32_t*>(g->offsets), g->num_nodes, g->nbrs, (uint64_t)g->num_entries, prob,
        alias, packed, num_samples, sample_index_base, seed, centers_out, contexts_out);
  else
    edges_kernel<int64_t><<<blocks, 256, 0, stream>>>(
        static_cast<const int64_t*>(g->offsets), g->num_nodes, g->nbrs, (uint64_t)g->num_entries, prob,
        alias, packed, num_samples, sample_index_base, seed, centers_out, contexts_out);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
