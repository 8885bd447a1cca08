// gs_sgns_step: one SGNS training iteration (GraphScale Sec. 3.2: fetch the
// rows the batch names, loss and sparse gradient on them, write them back, with
// the barrier of "Synchronization": all reads see the pre-iteration tables).
//
// The batch-synchronous rule is kept by splitting the iteration at kernel
// boundaries, and no atomic ever touches an embedding table: float atomics run
// at ~1/5 of the plain read-modify-write rate on this chip (and do not exist
// for a "round once" bf16 update), so contributions are first brought together
// per destination row and every touched row is written exactly once, as
// round(old + delta).
//
// Destination rows of both tables share one key space: key r < N is row r of
// the context table (its terms are the (pair, j) logits that name it), key N + c
// is row c of the input table (its terms are the staged gradients of the runs
// of equal centres).  A key has a counter slot: the key itself, or, when the
// graph is much larger than the batch, its place in a table of the batch's keys
// (so that nothing cleared, scanned or hit at random has the size of the graph).
//
//   clear      counters 0, key tables empty
//   forward    read-only on both tables: logits, g = dLoss/dx, loss, the
//              centre-row gradient of every run of equal centres staged in a
//              slot, and rank = cnt[slot of key]++ for every term and every
//              used staging slot (optionally the pairs themselves from the walk
//              buffer and the negatives from their counters)
//   scan       off = exclusive prefix sum of cnt
//   place      sorted[off[key] + rank] = (key, source row, coefficient, rank):
//              (context row, centre, -lr * g) or (N + centre, slot, -lr)
//   update     once over the context-table keys (source rows: the input table,
//              still unmodified), then once over the input-table keys (source
//              rows: the staged gradients): delta = sum coef * source row.  A
//              whole wave works on one row at a time.  The terms of a key are cut
//              into segments of 256 positions (64 in small batches); a row of one
//              segment is written once, as round(old + delta); the segments of a
//              longer row are added into a side buffer
//   finish     table[row] = round(old + side buffer) for the longer rows; one
//              extra block sums the per-block loss partials in a fixed order
//
// Small batches take two launches instead (forward, and one kernel for the rest): see
// sgns_small_update_kernel.  Large ones write their terms as records that are grouped by row instead of counting and
// placing them: see sgns_sorted_update_kernel.
//
// delta is accumulated exactly: every product coef * element is rounded once to
// a multiple of 2^-36 (one fp64 fused multiply-add against 1.5 * 2^52, whose
// result bits hold the integer) and the 64-bit integers are added.  Integer
// addition is associative, so the result does not depend on the order in which
// the terms of a row arrive (ranks come from atomics), on the places the keys
// get in their table, or on how a long row is split: the same call gives the
// same bits every time.
//
// Forward: a row is handled by 16 lanes holding 16-byte pieces (256 contiguous
// bytes per load instruction); a wave works on four rows at once and a dot
// product is a 16-lane DPP reduction.  No matrix cores: 0.3 flop per byte moved.
//
// The other entry points of this file run the same kernels with a few switches
// (SgnsArgs / SgnsExtras): the momentum and Adam steps apply the whole optimizer
// where a row of the batch is written, and one pass over the tables does the rows
// outside the batch (momentum with a small batch and small tables: the two
// launches between two dense passes); the fused step
// draws the negatives in the forward kernel; the one-table step (first-order
// LINE) reads the input rows in the update kernel from copies the forward kernel
// kept, because that kernel then writes rows of the table it would read.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "group.h"

namespace gs {

constexpr int kSgnsThreads = 256;
constexpr int kGroupLanes = 16;
constexpr int kGroupsPerBlock = kSgnsThreads / kGroupLanes;
constexpr size_t kCompactFactor = 16;  // keys per batch entry beyond which the key space is compacted
constexpr int64_t kStageMaxBlocks = 8192;   // launch of the input-table pass (its waves stride over the slices)
constexpr int kStageSlice = 8;     // staged gradients per 16-lane group in the input-table pass: they are
                                   // few (one per run of equal centres), so short slices keep the chip busy
// Terms of one key are cut into segments of 2^seg_shift positions, each summed by one wave;
// rows with more than one segment go through the side buffer (slot = position of the row's
// first term >> seg_shift).  Long segments keep the side-buffer traffic low; small batches take
// short ones, so that the few waves of a launch do not wait for one that sums a long segment.
constexpr int kSegShiftLarge = 8, kSegShiftSmall = 6;
constexpr int kLongRowBlocks = 512;   // launch over the list of long rows
constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 16;
constexpr int kScanTile = kScanThreads * kScanPerThread;
constexpr int64_t kFewTiles = 4096;   // up to this many scan tiles, blocks add up the earlier tile sums themselves
// Exact accumulation of the row sums: a product x = coef * element becomes the integer
// round(x * 2^36), read off the low bits of the fp64 value x * 2^36 + kFixMagic
// (one fused multiply-add; valid while |x| * 2^36 < 2^51, i.e. |x| < 32768).
constexpr double kFixScale = 68719476736.0;                  // 2^36
constexpr double kFixInvScale = 1.0 / 68719476736.0;
constexpr double kFixMagic = 6755399441055744.0;             // 1.5 * 2^52
constexpr unsigned long long kFixMagicBits = 0x4338000000000000ull;
constexpr float kFixPeak = 16384.0f;   // products at or beyond this magnitude are reported (NaN loss)
constexpr int kHotBits = 8;                      // block-local rank counters in forward
constexpr int kHotSlots = 1 << kHotBits;
constexpr uint32_t kRankPending = 0x80000000u;   // rank still relative to the block (ranks < 2^31)
constexpr uint32_t kNoRow = 0xffffffffu;         // no key: keys are below 2 * num_nodes <= 2^32 - 2


struct Term {      // one contribution to a destination row
  uint32_t row;    // key: context-table row r, or num_nodes + c for input-table row c
  int32_t center;  // source row: row of the input table (one-table mode: slot of its copy in
                   // `snap`), or the staging slot for an input-table key
  float coef;      // -lr * g, or -lr for a staged gradient
  uint32_t pos;    // position of this term among the terms of its key
};

// The optimizer behind the sparse update (a template argument of the kernels that write rows).  With
// delta D, the exact sum of a row's terms (computed with step -1, so D is the row's gradient):
//   kPlain     row = round(row + D)
//   kMomentum  m = round(round(mu * m) + D), w = round(w - lr * m)
//   kAdam      m = round(round(beta1 * m) + (1 - beta1) * D), v = round(round(beta2 * v) + (1 - beta2) * D * D),
//              w = round(w - adam_move(m, v))
// The rows that the batch does not name get the same with D = 0, in a pass over whole tables that
// leaves the others alone.
enum : int { kPlain, kMomentum, kAdam };
struct OptRates {
  float decay1, decay2;     // mu, or beta1 and beta2
  float c1, c2;             // Adam: 1 - beta1, 1 - beta2
  float lr;                 // of the model update (Adam: lr / (1 - beta1^t))
  float root_c2, eps;
};

struct SgnsArgs {
  void* w_in;               // tables the logits are computed from
  void* w_out;
  void* dst_in;             // tables that receive round(old + delta): the same two for plain
  void* dst_out;            // SGD, the momentum tables for the momentum step
  float* sq_in;             // Adam only (else null): the second-moment tables (fp32)
  float* sq_out;
  OptRates opt;             // momentum and Adam: the rates of the optimizer
  // negatives drawn inside the step (draw_negs != 0): entry (i, j) is the draw of
  // gs_sample_negatives for pair index neg_pair_base + i, written to negs_draw
  // (which `negs` then points to) for the later kernels
  int32_t draw_negs;
  const float* noise_prob;
  const int32_t* noise_alias;
  const uint2* noise_packed;
  uint64_t neg_seed;
  uint64_t neg_pair_base;
  int32_t* negs_draw;
  // pairs made inside the step (walks != null): pair i of the batch is pair first_pair + i of
  // the canonical pair sequence of walks[0 .. num_walks) (walk, then centre position, then
  // offset: the order of gs_make_pairs); pair_offsets[w] = number of pairs of the walks before
  // w, pair_offsets[num_walks] = all of them.  The forward kernel writes the ids it derives to
  // gen_centers / gen_contexts (which `centers` / `contexts` then point to) for the later kernels
  const int32_t* walks;
  const int64_t* pair_offsets;
  int64_t num_walks;
  int64_t first_pair;
  int32_t walk_len, window;
  int32_t* gen_centers;
  int32_t* gen_contexts;
  // one table on both sides (first-order LINE; else null): the update kernel writes rows of
  // the table while input rows are still needed, so the forward kernel keeps a copy of every
  // input row it loads (one per run of equal centres, at the run's staging slot) and notes
  // the slot of every pair (for the place kernel; a sorted record holds it); the update kernel
  // reads the copies
  void* snap;               // [num_pairs][dim], storage type of the table
  int32_t* pair_slot;       // [num_pairs]
  const int32_t* centers;
  const int32_t* contexts;
  const int32_t* negs;
  int64_t num_pairs;
  int64_t num_nodes;
  int64_t num_terms;        // num_pairs * (k + 1): positions [0, num_terms) of `sorted` hold the
                            // context-table keys, the positions after them the input-table keys
  int64_t long_slots;       // ((num_terms + num_pairs) >> seg_shift) + 1
  int32_t seg_shift;        // log2 of the segment length
  int32_t chunk_pairs;      // consecutive pairs per 16-lane group in forward (<= 16)
  int32_t slice_terms;      // sorted terms per 16-lane group in update
  int32_t k;
  uint32_t per_k1;          // t / (k + 1) = t * per_k1 >> 16 for t < 16 * 61 (k is at most 60)
  int32_t dim;
  float lr;
  float* g;                 // [num_terms]
  uint32_t* rank;           // [num_terms]
  uint32_t* cnt;            // [cnt_last + 1] counters, indexed by the slot of a key; after scan: offsets,
                            // and entry cnt_last holds the number of positions in use
  int64_t cnt_last;
  // Counter slots.  The context-table keys take the slots [0, in_base), the input-table keys
  // the slots from in_base on, so that in `sorted` every context-table key comes before every
  // input-table key.  A kind of key is either counted per vertex (bits == 0: slot = vertex) or,
  // when the graph is much larger than the batch, through an open-addressing table of
  // 1 << bits places holding the keys of the batch (slot = the key's place).  The batch has
  // few input-table keys (one per run of equal centres), so those go through a table sooner.
  uint32_t* key_table;      // [table_places = (out_bits ? 1 << out_bits : 0) + (in_bits ? 1 << in_bits : 0)],
                            // kNoRow = free
  int64_t table_places;
  int32_t out_bits, in_bits;
  uint32_t in_base;
  uint32_t* tile_sums;      // scan scratch
  Term* sorted;             // [num_terms + num_pairs]; large batches: the input-table terms only
  int64_t stage_base;       // position of the first input-table term in `sorted`
  int64_t stage_long_base;  // first side-buffer slot of the input-table rows
  uint32_t* term_key;       // large batches: [num_terms] row of the context table and
  uint2* term_src;          // (source row, coefficient) of every term; after the sort: in order of the rows
  const uint32_t* num_records;   // grouped batches: records of both kinds of rows,
  const uint2* long_rows;        // (key, side-buffer slot) of the long rows
  const uint32_t* num_long_rows;
  const uint8_t* named;          // optimizers on grouped batches: which rows of the context table the batch names, and from named_in on of
  uint32_t named_in;             // the input table; else null
  long long* long_acc;      // [long_slots][dim] exact sums of the long rows
  int32_t* stage_center;    // [num_pairs], -1 = unused slot
  uint32_t* stage_rank;     // [num_pairs] rank of the slot among the slots of its centre
  float* stage_delta;       // [num_pairs][dim], natural element order
  double* loss_partials;    // [forward blocks]
  int64_t forward_blocks;
  int64_t forward_blocks_per_xcd;
  double* loss_out;
  uint32_t* bad_ids;        // set when a centre / context / negative id is not a row of the tables,
                            // or a product left the range of the exact accumulation
};

// Ids come from device memory the host cannot inspect.  An id outside
// [0, num_nodes) is read as row 0 everywhere (so no access leaves the tables)
// and flagged; the call then reports a NaN loss.
__device__ __forceinline__ int32_t checked_row(const SgnsArgs& a, int32_t id) {
  if ((uint32_t)id < (uint32_t)a.num_nodes) return id;
  *a.bad_ids = 1u;
  return 0;
}

// ---- small device helpers ---------------------------------------------------------
// sum over the 16 lanes of a DPP row; every lane gets the total
__device__ __forceinline__ float row_sum16(float x) {
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));  // row_half_mirror
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));  // row_mirror
  return x;
}

// every table type other than float is one of the 16-bit formats (bf16_t, f16_t)
template <typename T>
using if_16bit = std::enable_if_t<!std::is_same<T, float>::value, int>;

// Register image of a row: VPL float4 per lane.  Register v of lane l holds the
// elements [4q, 4q+4) with q = natural_q(v, l):
//   fp32 rows   one float4 per 16-byte load,  q = v*16 + l
//   16-bit rows two float4 per 16-byte load (8 elements), q = 2*((v/2)*16 + l) + (v&1)
template <typename T>
__device__ __forceinline__ int natural_q(int v, int l16) {
  return 2 * ((v >> 1) * kGroupLanes + l16) + (v & 1);
}
template <>
__device__ __forceinline__ int natural_q<float>(int v, int l16) { return v * kGroupLanes + l16; }

template <int VPL>
__device__ __forceinline__ void zero(float4 (&a)[VPL]) {
#pragma unroll
  for (int v = 0; v < VPL; ++v) a[v] = make_float4(0.f, 0.f, 0.f, 0.f);
}

template <int VPL>
__device__ __forceinline__ float dot_partial(const float4 (&a)[VPL], const float4 (&b)[VPL]) {
  float s = 0.f;
#pragma unroll
  for (int v = 0; v < VPL; ++v)
    s += a[v].x * b[v].x + a[v].y * b[v].y + a[v].z * b[v].z + a[v].w * b[v].w;
  return s;
}

template <int VPL>
__device__ __forceinline__ void axpy(float4 (&acc)[VPL], float c, const float4 (&x)[VPL]) {
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    acc[v].x += c * x[v].x; acc[v].y += c * x[v].y;
    acc[v].z += c * x[v].z; acc[v].w += c * x[v].w;
  }
}

// A row as it was loaded, kept in as few registers as its storage type needs:
// fp32 rows VPL float4, 16-bit rows VPL/2 uint4 (widened element by element where
// they are used).  Rows that wait in registers for their turn are held this way,
// so a 16-bit group keeps twice as many of them in flight.
template <typename T, int VPL>
struct RawRow { uint4 r[VPL / 2]; };
template <int VPL>
struct RawRow<float, VPL> { float4 r[VPL]; };

template <int VPL>
__device__ __forceinline__ void load_raw(const float* __restrict__ table, int64_t row, int dim, int l16,
                                         RawRow<float, VPL>& x) {
  const float4* p = reinterpret_cast<const float4*>(table + row * (int64_t)dim);
  const int dim4 = dim >> 2;
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int q = v * kGroupLanes + l16;
    x.r[v] = (q < dim4) ? p[q] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}
// (16-bit rows: lanes behind the end of the row read its last piece again, see the forward kernel.)
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ void load_raw(const T* __restrict__ table, int64_t row, int dim, int l16,
                                         RawRow<T, VPL>& x) {
  static_assert(VPL % 2 == 0, "16-bit rows are held as pairs of float4");
  const uint4* p = reinterpret_cast<const uint4*>(table + row * (int64_t)dim);
  const int last = (dim >> 3) - 1;
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) x.r[w] = p[min(w * kGroupLanes + l16, last)];
}

// zeros in the place of the pieces behind the end of the row
template <int VPL>
__device__ __forceinline__ const RawRow<float, VPL>& inside_row(const RawRow<float, VPL>& x, int, int) { return x; }
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ RawRow<T, VPL> inside_row(const RawRow<T, VPL>& x, int dim, int l16) {
  RawRow<T, VPL> y;
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) {
    const bool in = w * kGroupLanes + l16 < (dim >> 3);
    y.r[w] = make_uint4(in ? x.r[w].x : 0u, in ? x.r[w].y : 0u, in ? x.r[w].z : 0u, in ? x.r[w].w : 0u);
  }
  return y;
}

// an input row, widened, and as it is stored; zeros behind its end, where an infinity of the last piece would meet the zeros of inside_row
template <int VPL>
__device__ __forceinline__ void load_center(const float* __restrict__ table, int64_t row, int dim, int l16, RawRow<float, VPL>& x, float4 (&u)[VPL]) {
  load_raw<VPL>(table, row, dim, l16, x);
#pragma unroll
  for (int v = 0; v < VPL; ++v) u[v] = x.r[v];
}
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ void load_center(const T* __restrict__ table, int64_t row, int dim, int l16, RawRow<T, VPL>& x, float4 (&u)[VPL]) {
  load_raw<VPL>(table, row, dim, l16, x);
  x = inside_row<VPL>(x, dim, l16);
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) {
    const uint4 q = x.r[w];
    u[2 * w] = make_float4(T::lo(q.x), T::hi(q.x), T::lo(q.y), T::hi(q.y));
    u[2 * w + 1] = make_float4(T::lo(q.z), T::hi(q.z), T::lo(q.w), T::hi(q.w));
  }
}

template <int VPL>
__device__ __forceinline__ void store_raw(float* __restrict__ table, int64_t row, int dim, int l16,
                                          const RawRow<float, VPL>& x) {
  float4* p = reinterpret_cast<float4*>(table + row * (int64_t)dim);
  const int dim4 = dim >> 2;
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int q = v * kGroupLanes + l16;
    if (q < dim4) p[q] = x.r[v];
  }
}
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ void store_raw(T* __restrict__ table, int64_t row, int dim, int l16,
                                          const RawRow<T, VPL>& x) {
  uint4* p = reinterpret_cast<uint4*>(table + row * (int64_t)dim);
  const int chunks = dim >> 3;
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) {
    const int c = w * kGroupLanes + l16;
    if (c < chunks) p[c] = x.r[w];
  }
}

// Between two uses of a raw 16-bit row: makes the compiler widen it again at the
// second use instead of keeping the widened copy (twice the registers) alive.
template <int VPL>
__device__ __forceinline__ void rewiden_later(RawRow<float, VPL>&) {}
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ void rewiden_later(RawRow<T, VPL>& x) {
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w)
    asm volatile("" : "+v"(x.r[w].x), "+v"(x.r[w].y), "+v"(x.r[w].z), "+v"(x.r[w].w));
}

template <int VPL>
__device__ __forceinline__ float dot_partial(const float4 (&a)[VPL], const RawRow<float, VPL>& b) {
  return dot_partial<VPL>(a, b.r);
}
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ float dot_partial(const float4 (&a)[VPL], const RawRow<T, VPL>& b) {
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) {
    const uint4 x = b.r[w];
    s += a[2 * w].x * T::lo(x.x) + a[2 * w].y * T::hi(x.x) + a[2 * w].z * T::lo(x.y) +
         a[2 * w].w * T::hi(x.y);
    s += a[2 * w + 1].x * T::lo(x.z) + a[2 * w + 1].y * T::hi(x.z) + a[2 * w + 1].z * T::lo(x.w) +
         a[2 * w + 1].w * T::hi(x.w);
  }
  return s;
}

template <int VPL>
__device__ __forceinline__ void axpy(float4 (&acc)[VPL], float c, const RawRow<float, VPL>& x) {
  axpy<VPL>(acc, c, x.r);
}
template <int VPL, typename T, if_16bit<T> = 0>
__device__ __forceinline__ void axpy(float4 (&acc)[VPL], float c, const RawRow<T, VPL>& b) {
#pragma unroll
  for (int w = 0; w < VPL / 2; ++w) {
    const uint4 x = b.r[w];
    acc[2 * w].x += c * T::lo(x.x); acc[2 * w].y += c * T::hi(x.x);
    acc[2 * w].z += c * T::lo(x.y); acc[2 * w].w += c * T::hi(x.y);
    acc[2 * w + 1].x += c * T::lo(x.z); acc[2 * w + 1].y += c * T::hi(x.z);
    acc[2 * w + 1].z += c * T::lo(x.w); acc[2 * w + 1].w += c * T::hi(x.w);
  }
}

// loss and dLoss/dx of one term from its logit: one expf, one log1pf, one divide
__device__ __forceinline__ void term_grad(float x, bool positive, float& g, float& loss) {
  const float e = expf(-fabsf(x));
  const float inv = 1.0f / (1.0f + e);
  const float sig = (x >= 0.0f) ? inv : e * inv;           // sigmoid(x)
  const float sig_m1 = (x >= 0.0f) ? -e * inv : -inv;      // sigmoid(x) - 1
  const float z = positive ? -x : x;
  loss = fmaxf(z, 0.0f) + log1pf(e);                       // softplus(z), |z| = |x|
  g = positive ? sig_m1 : sig;
}

// Blocks are handed to the 8 XCDs round-robin; this maps them so that each XCD
// works on one contiguous eighth of the batch: neighbouring chunks share
// centre and context rows, which then stay in that XCD's L2.  Performance only:
// any block-to-XCD assignment gives the same result.
__device__ __forceinline__ int64_t xcd_contiguous_block(int64_t bid, int64_t per_xcd) {
  return (bid & 7) * per_xcd + (bid >> 3);
}

// Counter slot of a key.  With the compacted key space the forward kernel enters the keys
// (claim_slot: first come, first served, linear probing; the table has at least twice as
// many places as the batch can hold keys) and the place kernel looks them up (find_slot).
// Which slot a key gets depends on the order of arrival, and with it the order of the rows in
// `sorted`; the results do not (exact sums).
struct KeyRegion {
  uint32_t slot_base;   // first counter slot of this kind of key
  uint32_t vertex;      // the key's vertex
  uint32_t* table;      // the kind's table (bits != 0)
  int bits;
};
__device__ __forceinline__ KeyRegion key_region(const SgnsArgs& a, uint32_t key) {
  const bool input_key = key >= (uint32_t)a.num_nodes;
  KeyRegion r;
  r.slot_base = input_key ? a.in_base : 0u;
  r.vertex = input_key ? key - (uint32_t)a.num_nodes : key;
  r.bits = input_key ? a.in_bits : a.out_bits;
  r.table = a.key_table + ((input_key && a.out_bits != 0) ? (1u << a.out_bits) : 0u);
  return r;
}
__device__ __forceinline__ uint32_t claim_slot(const SgnsArgs& a, uint32_t key) {
  const KeyRegion r = key_region(a, key);
  if (r.bits == 0) return r.slot_base + r.vertex;
  const uint32_t mask = (1u << r.bits) - 1u;
  const uint32_t home = (key * 2654435761u) >> (32 - r.bits);
  uint32_t h = home;
  // (the probe count is bounded so that the loop ends whatever the memory holds; a table
  // without a free place cannot arise from a batch the plan was made for, and is reported)
  for (uint32_t probes = 0; probes <= mask; ++probes) {
    uint32_t seen = __hip_atomic_load(r.table + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (seen == kNoRow) seen = atomicCAS(r.table + h, kNoRow, key);
    if (seen == kNoRow || seen == key) return r.slot_base + h;
    h = (h + 1u) & mask;
  }
  *a.bad_ids = 1u;
  return r.slot_base + home;
}
__device__ __forceinline__ uint32_t find_slot(const SgnsArgs& a, uint32_t key) {
  const KeyRegion r = key_region(a, key);
  if (r.bits == 0) return r.slot_base + r.vertex;
  const uint32_t mask = (1u << r.bits) - 1u;
  const uint32_t home = (key * 2654435761u) >> (32 - r.bits);
  uint32_t h = home;
  // every key of the batch was entered by the forward kernel
  for (uint32_t probes = 0; probes <= mask; ++probes) {
    if (r.table[h] == key) return r.slot_base + h;
    h = (h + 1u) & mask;
  }
  *a.bad_ids = 1u;
  return r.slot_base + home;
}

// ---- clear / fill ---------------------------------------------------------------------
// everything a call starts from: counters 0, no bad id seen (16 bytes per lane; the counter
// array is padded to a multiple of four entries)
__global__ void sgns_clear_kernel(uint4* __restrict__ cnt4, int64_t n4, uint4* __restrict__ table4,
                                  int64_t m4, uint32_t* __restrict__ flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *flag = 0u;
  if (i < n4) cnt4[i] = make_uint4(0u, 0u, 0u, 0u);
  if (i < m4) table4[i] = make_uint4(kNoRow, kNoRow, kNoRow, kNoRow);
}

// ---- forward ------------------------------------------------------------------------------
enum : int { kByCounter, kBySort, kGrouped, kInLds };
// whether an earlier kernel has cleared the flag of bad ids (else the block's loss partial reports them)
constexpr bool has_flag(int group) { return group == kByCounter || group == kBySort; }
// Staged centre-row gradient of one run of equal centres, in natural element
// order.  Slot numbers are fixed by position (first pair of the chunk + flush
// number), so no counter is shared between groups; unused slots of a chunk are
// marked with centre -1.
template <typename T, int VPL, int kGroup>
__device__ __forceinline__ void stage_flush(const SgnsArgs& a, int64_t slot, int32_t center, int l16,
                                            const float4 (&du)[VPL]) {
  if (l16 == 0) {
    a.stage_center[slot] = center;
    if constexpr (has_flag(kGroup)) a.stage_rank[slot] = atomicAdd(a.cnt + claim_slot(a, (uint32_t)a.num_nodes + (uint32_t)center), 1u);
  }
  float4* out = reinterpret_cast<float4*>(a.stage_delta + slot * (int64_t)a.dim);
  const int dim4 = a.dim >> 2;
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int q = natural_q<T>(v, l16);
    if (q < dim4) out[q] = du[v];
  }
}

// largest magnitude among the elements a lane holds of a row
template <int VPL>
__device__ __forceinline__ float row_peak(const float4 (&r)[VPL]) {
  float m = 0.f;
#pragma unroll
  for (int v = 0; v < VPL; ++v)
    m = fmaxf(fmaxf(m, fmaxf(fabsf(r[v].x), fabsf(r[v].y))), fmaxf(fabsf(r[v].z), fabsf(r[v].w)));
  return m;
}

// kGroup: how the terms of a row come together afterwards.
//   kByCounter  every term takes a rank from its row's counter (for the place kernel)
//   kBySort     every term is written as a record for the sort; only staging slots are counted
//   kGrouped    every term is written as a record for the grouping, which takes the staging slots as well:
//               nothing is counted, and a bad id or an out-of-range product turns the block's loss partial into
//               NaN (there is no flag that an earlier kernel would have cleared)
//   kInLds      the step of a small batch, whose update kernel groups the terms itself: the same
// kWaves: waves per SIMD that the registers have to leave room for (0: no say); see launch_forward.
template <typename T, int VPL, int RB, int kGroup, int kThreads, int kWaves = 0>
__global__ __launch_bounds__(kThreads, kWaves) void sgns_forward_kernel(SgnsArgs a) {
  constexpr int kGroups = kThreads / kGroupLanes;
  extern __shared__ int32_t idx_s[];              // per group: centres[chunk], rows[chunk][K+1]
  __shared__ float loss_s[kGroups];
  // Rank counters of rows that many terms hit at once are same-address atomics in
  // memory, which serialise.  Each block therefore counts up to kHotSlots rows
  // locally first (whichever rows reach a slot of this small LDS table first):
  // a term of such a row takes a block-local rank, the block adds its total to
  // the row's global counter once, and the ranks are completed afterwards.
  __shared__ int32_t hot_key[kGroup == kByCounter ? kHotSlots : 1];
  __shared__ uint32_t hot_cnt[kGroup == kByCounter ? kHotSlots : 1];
  __shared__ uint32_t hot_base[kGroup == kByCounter ? kHotSlots : 1];
  bool bad = false;
  auto row_of = [&](int32_t id) -> int32_t {
    if constexpr (has_flag(kGroup)) return checked_row(a, id);
    if ((uint32_t)id < (uint32_t)a.num_nodes) return id;
    bad = true;
    return 0;
  };
  auto report = [&]() {
    if constexpr (has_flag(kGroup)) *a.bad_ids = 1u;
    else bad = true;
  };
  const T* __restrict__ w_in = static_cast<const T*>(a.w_in);
  const T* __restrict__ w_out = static_cast<const T*>(a.w_out);
  const int l16 = threadIdx.x & (kGroupLanes - 1);
  const int group_in_block = threadIdx.x / kGroupLanes;
  const int64_t block = xcd_contiguous_block(blockIdx.x, a.forward_blocks_per_xcd);
  const int K = a.k, K1 = a.k + 1;
  const int64_t group = block * kGroups + group_in_block;
  const int64_t first = group * a.chunk_pairs;
  const bool block_live = block < a.forward_blocks;
  const int64_t last = block_live ? min(first + a.chunk_pairs, a.num_pairs) : first;
  const int count = (int)max((int64_t)0, last - first);

  int32_t* cen_s = idx_s + group_in_block * (a.chunk_pairs * (K1 + 1));
  int32_t* rows_s = cen_s + a.chunk_pairs;
  if constexpr (kGroup == kByCounter)
    for (int h = threadIdx.x; h < kHotSlots; h += kThreads) { hot_key[h] = -1; hot_cnt[h] = 0u; }
  if (a.walks != nullptr) {
    if (l16 < count) {                      // lane p derives pair p of the chunk from its walk
      int32_t c = 0, o = 0;
      const int64_t gp = a.first_pair + first + l16;
      if (gp < a.pair_offsets[a.num_walks]) {
        int64_t lo = 0, hi = a.num_walks - 1;     // last walk w with pair_offsets[w] <= gp
        while (lo < hi) {
          const int64_t mid = (lo + hi + 1) >> 1;
          if (a.pair_offsets[mid] <= gp) lo = mid; else hi = mid - 1;
        }
        const int32_t* row = a.walks + lo * (int64_t)a.walk_len;
        const int64_t len = valid_prefix(row, a.walk_len);
        int64_t at, other;
        pair_positions(gp - a.pair_offsets[lo], len, a.window, at, other);
        if (at >= 0 && at < len && other >= 0 && other < len) {
          c = row[at];
          o = row[other];
        } else {
          report();                         // pair_offsets does not belong to these walks
        }
      } else {
        report();                           // the walks do not hold that many pairs
      }
      a.gen_centers[first + l16] = c;
      a.gen_contexts[first + l16] = o;
      cen_s[l16] = row_of(c);
      rows_s[l16 * K1] = row_of(o);
    }
  } else if (l16 < count) {
    cen_s[l16] = row_of(a.centers[first + l16]);
  }
  const int terms = count * K1;
  if constexpr (kGroup == kInLds) {         // (two pairs per group, so most lanes have one term: 256 to 4096 pairs are 0.5 % slower with the loop below)
    for (int t = l16; t < terms; t += kGroupLanes) {
      const int p = t / K1, j = t - p * K1;
      int32_t row;
      if (j == 0) {
        if (a.walks != nullptr) continue;   // set above
        row = row_of(a.contexts[first + p]);
      } else if (a.draw_negs) {
        const Block4 b = philox_at(a.neg_seed, a.neg_pair_base + (uint64_t)(first + p), (uint32_t)(j - 1),
                                   0x80000000u);
        row = (int32_t)table_draw(a.noise_prob, a.noise_alias, a.noise_packed, (uint64_t)a.num_nodes, b);
        a.negs_draw[(first + p) * (int64_t)K + (j - 1)] = row;
      } else {
        row = row_of(a.negs[(first + p) * (int64_t)K + (j - 1)]);
      }
      rows_s[t] = row;
    }
  } else {
    constexpr int kIds = 4;                 // ids in flight per lane
    for (int t0 = l16; t0 < terms; t0 += kIds * kGroupLanes) {
      int32_t id[kIds];
#pragma unroll
      for (int c = 0; c < kIds; ++c) {
        const int t = t0 + c * kGroupLanes;
        id[c] = 0;
        if (t >= terms) continue;
        const int p = (int)((uint32_t)t * a.per_k1 >> 16), j = t - p * K1;
        if (j == 0) {
          if (a.walks == nullptr) id[c] = a.contexts[first + p];
        } else if (a.draw_negs) {
          const Block4 b = philox_at(a.neg_seed, a.neg_pair_base + (uint64_t)(first + p), (uint32_t)(j - 1),
                                     0x80000000u);
          id[c] = (int32_t)table_draw(a.noise_prob, a.noise_alias, a.noise_packed, (uint64_t)a.num_nodes, b);
          a.negs_draw[(first + p) * (int64_t)K + (j - 1)] = id[c];
        } else {
          id[c] = a.negs[(first + p) * (int64_t)K + (j - 1)];
        }
      }
#pragma unroll
      for (int c = 0; c < kIds; ++c) {
        const int t = t0 + c * kGroupLanes;
        if (t >= terms || (a.walks != nullptr && t % K1 == 0)) continue;    // (a walk's pairs: set above)
        rows_s[t] = row_of(id[c]);
      }
    }
  }
  __syncthreads();

  // 16-bit rows: no branch lies between the reads of a block of rows and nothing else is written into their registers, so that all of
  // them are under way together; with zeros for the lanes behind the end of a row the compiler moved half of the rows to other registers and
  // waited for each before it asked for the next (fp32 rows stay where they are read to, and up to 400 columns that do not fill the
  // lanes are 5 % faster with the branches).  1 M pairs of 256 bf16 columns, 11 M terms: 1020 -> 823 us; 300,000 pairs of 200 fp16 columns, 2.4 M
  // terms: 213 -> 184.  (Lanes behind the end add up what the last piece does, in du too, which is not stored from there; reads behind the last
  // term of a pair are of its row again.)
  const bool full = a.dim == VPL * 64;         // every lane has a piece of the row
  float4 u[VPL], du[VPL];
  zero<VPL>(u);
  zero<VPL>(du);
  int32_t cur_c = -1;
  int flushes = 0;
  float loss = 0.f;
  // The update kernels add products coef * element exactly while these stay below 32768:
  // coef is -lr * g with |g| <= 1 times an element of an input row, or -lr times an element
  // of a staged gradient.  Both kinds of rows pass through this kernel, which checks them.
  float peak = 0.f;
  // The rank of the lane's last term, and the place of that term's id, which it takes one block of terms later: reads and
  // atomics return in order, so a rank is asked for behind the rows of its block and not waited for before the next.
  // (In front of them where they are short: 16-bit rows of up to 128 columns are 0.6 % faster so on average over 8500 to 500,000 pairs,
  // 200 to 400 columns up to 2 % slower.)
  constexpr bool kRankFirst = sizeof(T) == 2 && VPL <= 2;
  uint32_t held = 0u;
  int held_at = -1;

  for (int p = 0; p < count; ++p) {
    const int32_t c = cen_s[p];
    if (c != cur_c) {
      if (cur_c >= 0) {
        peak = fmaxf(peak, row_peak<VPL>(du));
        stage_flush<T, VPL, kGroup>(a, first + flushes++, cur_c, l16, du);
      }
      RawRow<T, VPL> keep;
      load_center<VPL>(w_in, c, a.dim, l16, keep, u);
      peak = fmaxf(peak, row_peak<VPL>(u));
      // one-table mode: keep the row as it is now
      if (a.snap != nullptr) store_raw<VPL>(static_cast<T*>(a.snap), first + flushes, a.dim, l16, keep);
      zero<VPL>(du);
      cur_c = c;
    }
    if (a.snap != nullptr && l16 == 0) a.pair_slot[first + p] = (int32_t)(first + flushes);
    const int64_t e0 = (first + p) * (int64_t)K1;
    const int32_t* prow = rows_s + p * K1;
    for (int j0 = 0; j0 <= K; j0 += RB) {
      // lane b of the group owns term j0 + b of this block of RB terms
      const int my_j = j0 + l16;
      const bool mine = l16 < RB && my_j <= K;
      if constexpr (kGroup == kByCounter && kRankFirst) {
        if (held_at >= 0) rows_s[held_at] = (int32_t)held;
        held_at = -1;
        if (mine) {
          const int32_t row = prow[my_j];
          const uint32_t h = ((uint32_t)row * 2654435761u) >> (32 - kHotBits);
          const int32_t seen = atomicCAS(&hot_key[h], -1, row);
          if (seen == -1 || seen == row) held = kRankPending | (atomicAdd(&hot_cnt[h], 1u) << kHotBits) | h;
          else held = atomicAdd(a.cnt + claim_slot(a, (uint32_t)row), 1u);
          held_at = p * K1 + my_j;
        }
      }
      RawRow<T, VPL> vv[RB];
#pragma unroll
      for (int b = 0; b < RB; ++b)
        if (sizeof(T) == 2 || j0 + b <= K) load_raw<VPL>(w_out, prow[sizeof(T) == 2 ? min(j0 + b, K) : j0 + b], a.dim, l16, vv[b]);
      if constexpr (kGroup == kByCounter && !kRankFirst) {   // (the same; as one function it costs the wide rows registers: 4 %)
        if (held_at >= 0) rows_s[held_at] = (int32_t)held;
        held_at = -1;
        if (mine) {
          const int32_t row = prow[my_j];
          const uint32_t h = ((uint32_t)row * 2654435761u) >> (32 - kHotBits);
          const int32_t seen = atomicCAS(&hot_key[h], -1, row);
          if (seen == -1 || seen == row) held = kRankPending | (atomicAdd(&hot_cnt[h], 1u) << kHotBits) | h;
          else held = atomicAdd(a.cnt + claim_slot(a, (uint32_t)row), 1u);
          held_at = p * K1 + my_j;
        }
      }
      float x_mine = 0.f;
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        if (j0 + b <= K) {
          const float x = row_sum16(sizeof(T) == 4 || full ? dot_partial<VPL>(u, vv[b]) : dot_partial<VPL>(u, inside_row<VPL>(vv[b], a.dim, l16)));
          if (l16 == b) x_mine = x;
        }
      }
#pragma unroll
      for (int b = 0; b < RB; ++b) rewiden_later<VPL>(vv[b]);
      float g_mine = 0.f, l_mine = 0.f;
      if (mine) term_grad(x_mine, my_j == 0, g_mine, l_mine);
      loss += l_mine;
#pragma unroll
      for (int b = 0; b < RB; ++b)
        if (j0 + b <= K) axpy<VPL>(du, __shfl(g_mine, b, kGroupLanes), vv[b]);
      if (mine) {
        if constexpr (kGroup == kBySort || kGroup == kGrouped) {
          const int32_t src = a.snap != nullptr ? (int32_t)(first + flushes) : c;
          a.term_key[e0 + my_j] = (uint32_t)prow[my_j];
          a.term_src[e0 + my_j] = make_uint2((uint32_t)src, __float_as_uint(-a.lr * g_mine));
        } else {
          a.g[e0 + my_j] = g_mine;
        }
      }
    }
  }
  if (cur_c >= 0) {
    peak = fmaxf(peak, row_peak<VPL>(du));
    stage_flush<T, VPL, kGroup>(a, first + flushes++, cur_c, l16, du);
  }
  if (l16 >= flushes && l16 < count) a.stage_center[first + l16] = -1;
  if (!(peak * fabsf(a.lr) < kFixPeak)) report();   // (also taken for NaN)
  if (!has_flag(kGroup) && bad) loss = __uint_as_float(0x7fc00000u);

  loss = row_sum16(loss);
  if (l16 == 0) loss_s[group_in_block] = loss;
  if (kGroup == kByCounter && held_at >= 0) rows_s[held_at] = (int32_t)held;
  __syncthreads();
  if constexpr (kGroup == kByCounter) {
    // one global update per locally counted row, then complete the pending ranks
    for (int h = threadIdx.x; h < kHotSlots; h += kThreads)
      if (hot_key[h] >= 0) hot_base[h] = atomicAdd(a.cnt + claim_slot(a, (uint32_t)hot_key[h]), hot_cnt[h]);
    __syncthreads();
    for (int t = l16; t < terms; t += kGroupLanes) {
      const uint32_t rk = (uint32_t)rows_s[t];
      a.rank[first * (int64_t)K1 + t] =
          (rk & kRankPending) ? hot_base[rk & (kHotSlots - 1)] + ((rk & ~kRankPending) >> kHotBits) : rk;
    }
  }
  if (threadIdx.x == 0 && block_live) {
    double s = 0.0;
#pragma unroll
    for (int gidx = 0; gidx < kGroups; ++gidx) s += (double)loss_s[gidx];
    a.loss_partials[block] = s;
  }
}

// ---- exclusive scan of cnt[0..n) (uint32), three kernels ---------------------
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const uint32_t* __restrict__ data,
                                                                   int64_t n,
                                                                   uint32_t* __restrict__ tile_sums) {
  __shared__ uint32_t s[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint32_t acc = 0;
#pragma unroll
  for (int k = 0; k < kScanPerThread; ++k) {
    const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (i < n) acc += data[i];
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) t += s[w];
    tile_sums[blockIdx.x] = t;
  }
}

// single block: exclusive scan of the tile sums in place
__global__ __launch_bounds__(1024) void scan_tiles_kernel(uint32_t* __restrict__ tile_sums,
                                                          int64_t tiles) {
  __shared__ uint32_t wave_tot[16];
  __shared__ uint32_t carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t base = 0; base < tiles; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const uint32_t v = (i < tiles) ? tile_sums[i] : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = carry_s, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w < wave) before += wave_tot[w];
      all += wave_tot[w];
    }
    if (i < tiles) tile_sums[i] = before + incl - v;
    __syncthreads();
    if (threadIdx.x == 0) carry_s += all;
    __syncthreads();
  }
}

// tile_offsets: exclusive prefix sums of the tile sums (raw_sums == 0), or the tile sums
// themselves (raw_sums != 0: each block adds up the sums of the tiles before it, which is
// cheaper than a kernel of its own while there are few tiles)
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(uint32_t* __restrict__ data, int64_t n,
                                                                  const uint32_t* __restrict__ tile_offsets,
                                                                  int raw_sums) {
  __shared__ uint32_t wave_tot[kScanThreads / 64];
  __shared__ uint32_t before_s[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t tile_base;
  if (raw_sums) {
    uint32_t part = 0;
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) part += tile_offsets[i];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) part += __shfl_xor(part, d, 64);
    if (lane == 0) before_s[wave] = part;
    __syncthreads();
    tile_base = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) tile_base += before_s[w];
  } else {
    tile_base = tile_offsets[blockIdx.x];
  }
  // thread t owns kScanPerThread consecutive values
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
  uint32_t v[kScanPerThread];
  uint32_t local = 0;
  const bool whole = base + kScanPerThread <= n;   // 64 aligned bytes: four 16-byte accesses
  if (whole) {
    const uint4* p4 = reinterpret_cast<const uint4*>(data + base);
#pragma unroll
    for (int k4 = 0; k4 < kScanPerThread / 4; ++k4) {
      const uint4 x = p4[k4];
      v[4 * k4] = x.x; v[4 * k4 + 1] = x.y;
      v[4 * k4 + 2] = x.z; v[4 * k4 + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) v[k] = (base + k < n) ? data[base + k] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kScanPerThread; ++k) local += v[k];
  uint32_t incl = local;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t run = tile_base + incl - local;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w)
    if (w < wave) run += wave_tot[w];
  if (whole) {
    uint4* p4 = reinterpret_cast<uint4*>(data + base);
#pragma unroll
    for (int k4 = 0; k4 < kScanPerThread / 4; ++k4) {
      uint4 x;
      x.x = run; run += v[4 * k4];
      x.y = run; run += v[4 * k4 + 1];
      x.z = run; run += v[4 * k4 + 2];
      x.w = run; run += v[4 * k4 + 3];
      p4[k4] = x;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kScanPerThread; ++k) {
      if (base + k < n) data[base + k] = run;
      run += v[k];
    }
  }
}

// The whole scan in one block, for the few counters of a small batch (one kernel instead of
// two on a path that is bound by its number of dependent kernels): a thread sums its stretch
// of consecutive entries, the block scans the sums, the thread writes its stretch.  Entries
// move 16 bytes at a time, eight independent loads in flight per thread: `data` is 16-byte
// aligned and allocated up to a multiple of four entries; the padding is read (it holds
// zeros) and written.
constexpr int64_t kScanSmallMax = 24 << 10;      // (20,000 entries 7 us, 100,000 47; the two kernels 10 to 11)
__global__ __launch_bounds__(1024) void scan_small_kernel(uint32_t* __restrict__ data, int64_t n) {
  __shared__ uint32_t wave_tot[16];
  constexpr int kBurst = 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint4* __restrict__ d4 = (uint4*)data;
  const int64_t n4 = (n + 3) / 4;
  const int per = (int)((n4 + 1023) / 1024);
  const int64_t lo = min(n4, (int64_t)threadIdx.x * per);
  const int mine = (int)(min(n4, lo + per) - lo);
  uint32_t local = 0;
  for (int c = 0; c < mine; c += kBurst) {
    uint4 v[kBurst];
#pragma unroll
    for (int u = 0; u < kBurst; ++u) v[u] = (c + u < mine) ? d4[lo + c + u] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < kBurst; ++u) local += v[u].x + v[u].y + v[u].z + v[u].w;
  }
  uint32_t incl = local;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t run = incl - local;
#pragma unroll
  for (int w = 0; w < 16; ++w)
    if (w < wave) run += wave_tot[w];
  for (int c = 0; c < mine; c += kBurst) {
    uint4 v[kBurst];
#pragma unroll
    for (int u = 0; u < kBurst; ++u) v[u] = (c + u < mine) ? d4[lo + c + u] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < kBurst; ++u) {
      uint4 o;
      o.x = run;
      o.y = o.x + v[u].x;
      o.z = o.y + v[u].y;
      o.w = o.z + v[u].z;
      run = o.w + v[u].w;
      if (c + u < mine) d4[lo + c + u] = o;
    }
  }
}

// ---- place: scatter the terms into key-major order ------------------------------
// Entries [0, num_terms) are the (pair, j) terms, entries num_terms + s the staging slots.
// The entry with position 2^seg_shift (it exists exactly in the rows of more than one
// segment) also clears the row's slot of the side buffer.
// (Large batches, whose terms are sorted: first_entry = num_terms, the staging slots alone.)
__global__ __launch_bounds__(256) void sgns_place_kernel(SgnsArgs a, int64_t first_entry) {
  const int64_t e = first_entry + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.num_terms + a.num_pairs) return;
  Term t;
  uint32_t rk;
  if (e < a.num_terms) {
    const int K1 = a.k + 1;
    const int64_t i = e / K1;
    const int j = (int)(e - i * K1);
    t.row = (uint32_t)checked_row(a, (j == 0) ? a.contexts[i] : a.negs[i * (int64_t)a.k + (j - 1)]);
    t.center = (a.pair_slot != nullptr) ? a.pair_slot[i] : checked_row(a, a.centers[i]);
    t.coef = -a.lr * a.g[e];
    rk = a.rank[e];
  } else {
    const int64_t slot = e - a.num_terms;
    const int32_t c = a.stage_center[slot];
    if (c < 0) return;
    t.row = (uint32_t)a.num_nodes + (uint32_t)c;
    t.center = (int32_t)slot;
    t.coef = -a.lr;
    rk = a.stage_rank[slot];
  }
  const uint32_t begin = a.cnt[find_slot(a, t.row)];
  t.pos = rk;
  a.sorted[begin + rk] = t;
  if (rk == (1u << a.seg_shift)) {
    const int64_t long_base = e < a.num_terms ? 0 : a.stage_long_base;
    long long* acc = a.long_acc + (long_base + (int64_t)(begin >> a.seg_shift)) * a.dim;
    for (int x = 0; x < a.dim; ++x) acc[x] = 0;
  }
}

// ---- update: one pass over the key-major terms of one table ----------------------------
// Here a whole wave works on one row at a time: the fields of a term are broadcast
// from the lane that holds it into scalar registers, so every branch (row change,
// long row, end of slice) is uniform and the per-row epilogue runs once per row.
// Lane l holds, for p < PPL, piece p*64 + l of a row; a piece is WPP 32-bit words of the
// table's storage type (4, 8 or 16 bytes: 256, 512 or 1024 contiguous bytes per load
// instruction), i.e. EPP = WPP (fp32) or 2 * WPP (16-bit) consecutive elements.
//
// Exact row sums: acc holds the sum of the result bits of fma(element, coef * 2^36,
// kFixMagic), i.e. terms * kFixMagicBits + the sum of the rounded products (mod 2^64).
__device__ __forceinline__ void fix_add(unsigned long long& acc, double c, float x) {
  acc += (unsigned long long)__double_as_longlong(__builtin_fma((double)x, c, kFixMagic));
}

template <typename T>
struct Words { static constexpr int kPerWord = 2; };     // elements in a 32-bit word of a table
template <>
struct Words<float> { static constexpr int kPerWord = 1; };

// one piece of WORDS 32-bit words, in a single load / store instruction
template <int WORDS>
__device__ __forceinline__ void load_words(const uint32_t* __restrict__ p, uint32_t (&w)[WORDS]) {
  if constexpr (WORDS == 1) {
    w[0] = *p;
  } else if constexpr (WORDS == 2) {
    const uint2 x = *reinterpret_cast<const uint2*>(p);
    w[0] = x.x; w[1] = x.y;
  } else {
    static_assert(WORDS % 4 == 0, "pieces are 4, 8 or a multiple of 16 bytes");
#pragma unroll
    for (int i = 0; i < WORDS / 4; ++i) {
      const uint4 x = reinterpret_cast<const uint4*>(p)[i];
      w[4 * i] = x.x; w[4 * i + 1] = x.y; w[4 * i + 2] = x.z; w[4 * i + 3] = x.w;
    }
  }
}
template <int WORDS>
__device__ __forceinline__ void store_words(uint32_t* __restrict__ p, const uint32_t (&w)[WORDS]) {
  if constexpr (WORDS == 1) {
    *p = w[0];
  } else if constexpr (WORDS == 2) {
    *reinterpret_cast<uint2*>(p) = make_uint2(w[0], w[1]);
  } else {
#pragma unroll
    for (int i = 0; i < WORDS / 4; ++i)
      reinterpret_cast<uint4*>(p)[i] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
  }
}

// element i of a piece held as words of storage type T, widened exactly
template <typename T, int WORDS>
__device__ __forceinline__ float piece_elem(const uint32_t (&w)[WORDS], int i) {
  if constexpr (std::is_same<T, float>::value) return __uint_as_float(w[i]);
  else return (i & 1) ? T::hi(w[i >> 1]) : T::lo(w[i >> 1]);
}

// elements back into words of storage type T (16-bit: rounded)
template <typename T, int WORDS>
__device__ __forceinline__ void pack_piece(const float* x, uint32_t (&w)[WORDS]) {
#pragma unroll
  for (int i = 0; i < WORDS; ++i) {
    if constexpr (std::is_same<T, float>::value) w[i] = __float_as_uint(x[i]);
    else w[i] = pack16<T>(x[2 * i], x[2 * i + 1]);
  }
}

// x as a table of type T holds it
template <typename T>
__device__ __forceinline__ float as_stored(float x) {
  if constexpr (std::is_same<T, float>::value) return x;
  else return T::lo(T::round(x));
}

// one element of the optimizers' rows (d = 0 for the rows outside the batch); w comes back unrounded
template <typename T>
__device__ __forceinline__ void momentum_elem(const OptRates& o, float& m, float& w, double d) {
  m = as_stored<T>(m * o.decay1);
  m = as_stored<T>((float)((double)m + d));
  w = w - o.lr * m;
}
__device__ __forceinline__ float adam_move(float m, float v, float step, float root_c2, float eps) {
  return step * m / (sqrtf(v) / root_c2 + eps);
}
__device__ __forceinline__ void adam_elem(const OptRates& o, float& m, float& v, float& w, double d) {
  m *= o.decay1;
  v *= o.decay2;
  m = (float)((double)m + (double)o.c1 * d);
  v = (float)((double)v + (double)o.c2 * d * d);
  w -= adam_move(m, v, o.lr, o.root_c2, o.eps);
}

// the exact sum as a double: net integer (terms * magic bits taken off) times 2^-36
__device__ __forceinline__ double fix_value(unsigned long long acc) {
  return (double)(long long)acc * kFixInvScale;
}

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// first position >= p (and < limit) whose term starts a segment, else limit; wave-uniform
__device__ __forceinline__ int64_t next_segment_start(const Term* __restrict__ sorted, int64_t p,
                                                      int64_t limit, int lane, uint32_t seg_mask) {
  while (p < limit) {
    const bool start = p + lane >= limit || (sorted[p + lane].pos & seg_mask) == 0u;
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(start);
    if (mask != 0ull) return min(limit, p + (int64_t)__builtin_ctzll(mask));
    p += 64;
  }
  return limit;
}

// What one wave does with the positions [begin, end) of key-major terms: begin and end are the
// starts of segments (or the end of the terms).  kStage = false: context-table keys, source rows
// from the input table; kStage = true: input-table keys, source rows = staged gradients (fp32,
// natural element order).  kSegments = false: every key is one segment.  kSorted: the terms are the
// sorted records (term_key, term_src), which do not hold their positions: these follow from
// where the keys change, and from first_row, the first position of the row that `begin` lies in.
template <typename T, int WPP, int PPL, int UB, int kOpt, bool kStage, bool kSegments, bool kSorted = false>
__device__ __forceinline__ void update_range(const SgnsArgs& a, const Term* __restrict__ sorted, int64_t begin,
                                             int64_t end, int64_t pos_hi, int lane, int64_t first_row = 0) {
  static_assert(kOpt != kAdam || std::is_same<T, float>::value, "second-moment tables are fp32");
  constexpr int EPP = WPP * Words<T>::kPerWord;          // elements per piece
  constexpr int EPL = EPP * PPL;                         // elements per lane
  constexpr int SW = kStage ? EPP : WPP;                 // 32-bit words of a source piece
  // source rows: the input table, or the copies the forward kernel kept (one-table mode, small
  // batches), or the staged gradients
  const uint32_t* __restrict__ src_base = reinterpret_cast<const uint32_t*>(
      kStage ? static_cast<const void*>(a.stage_delta) : (a.snap != nullptr ? a.snap : a.w_in));
  uint32_t* dst_base = reinterpret_cast<uint32_t*>(kStage ? a.dst_in : a.dst_out);
  uint32_t* sq_base = reinterpret_cast<uint32_t*>(kStage ? a.sq_in : a.sq_out);
  uint32_t* model_base = reinterpret_cast<uint32_t*>(kStage ? a.w_in : a.w_out);   // momentum and Adam
  const uint32_t key_base = kStage ? (uint32_t)a.num_nodes : 0u;
  const int64_t src_row_words = kStage ? (int64_t)a.dim : (int64_t)a.dim / Words<T>::kPerWord;
  const int64_t dst_row_words = (int64_t)a.dim / Words<T>::kPerWord;
  const uint32_t seg_mask = kSegments ? (1u << a.seg_shift) - 1u : ~0u;
  bool piece_ok[PPL];                                    // piece p of this lane lies inside the row
#pragma unroll
  for (int p = 0; p < PPL; ++p) piece_ok[p] = (p * 64 + lane) * EPP < a.dim;

  unsigned long long acc[EPL];
  uint32_t old[PPL][WPP];
  uint32_t old_w[kOpt != kPlain ? PPL : 1][WPP], old_v[kOpt == kAdam ? PPL : 1][WPP];
#pragma unroll
  for (int x = 0; x < EPL; ++x) acc[x] = 0;
#pragma unroll
  for (int p = 0; p < PPL; ++p)
#pragma unroll
    for (int w = 0; w < WPP; ++w) {
      old[p][w] = 0u;
      if constexpr (kOpt != kPlain) old_w[p][w] = 0u;
      if constexpr (kOpt == kAdam) old_v[p][w] = 0u;
    }
  uint32_t cur_row = kNoRow;       // key of the segment being summed (table row: cur_row - key_base)
  uint32_t cur_seg = 0;            // its number within the key (pos >> seg_shift of its terms)
  int64_t seg_first = 0;           // position of its first term
  uint32_t cur_terms = 0;          // terms added into acc since it was cleared

  // takes the magic bits of the terms off (their low word is zero): acc becomes the net sum
  auto settle = [&]() {
    const unsigned long long off = (unsigned long long)(cur_terms * (uint32_t)(kFixMagicBits >> 32)) << 32;
#pragma unroll
    for (int x = 0; x < EPL; ++x) acc[x] -= off;
  };
  auto flush_long = [&]() {
    const int64_t row_first = seg_first - ((int64_t)cur_seg << a.seg_shift);
    unsigned long long* dst = reinterpret_cast<unsigned long long*>(a.long_acc) +
                              ((row_first >> a.seg_shift) + (kStage && !kSorted ? a.stage_long_base : 0)) * a.dim;
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      if (piece_ok[p]) {
#pragma unroll
        for (int i = 0; i < EPP; ++i) atomicAdd(dst + (p * 64 + lane) * EPP + i, acc[p * EPP + i]);
      }
    }
  };
  // new = round(old + d) for the elements of one piece, packed back into storage words
  auto write_piece = [&](uint32_t* row_words, int p, const uint32_t (&was)[WPP], const double* d) {
    uint32_t out[WPP];
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
      for (int i = 0; i < WPP; ++i)
        out[i] = __float_as_uint((float)((double)__uint_as_float(was[i]) + d[i]));
    } else {
#pragma unroll
      for (int i = 0; i < WPP; ++i)
        out[i] = pack16<T>((float)((double)T::lo(was[i]) + d[2 * i]),
                           (float)((double)T::hi(was[i]) + d[2 * i + 1]));
    }
    store_words<WPP>(row_words + (int64_t)(p * 64 + lane) * WPP, out);
  };
  // continues: the next term belongs to the same key (the row has a further segment)
  auto flush = [&](bool continues) {
    settle();
    if constexpr (kSegments) {
      if (cur_seg > 0 || continues) {
        flush_long();
        return;
      }
    }
    const int64_t r = (int64_t)(cur_row - key_base);
    uint32_t* row_words = dst_base + r * dst_row_words;
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      if (!piece_ok[p]) continue;
      double d[EPP];
#pragma unroll
      for (int i = 0; i < EPP; ++i) d[i] = fix_value(acc[p * EPP + i]);
      if constexpr (kOpt == kPlain) {
        write_piece(row_words, p, old[p], d);
      } else {
        const int64_t at = r * dst_row_words + (int64_t)(p * 64 + lane) * WPP;
        float m[EPP], w[EPP];
#pragma unroll
        for (int i = 0; i < EPP; ++i) { m[i] = piece_elem<T, WPP>(old[p], i); w[i] = piece_elem<T, WPP>(old_w[p], i); }
        if constexpr (kOpt == kMomentum) {
#pragma unroll
          for (int i = 0; i < EPP; ++i) momentum_elem<T>(a.opt, m[i], w[i], d[i]);
        } else {
          uint32_t v_out[WPP];
#pragma unroll
          for (int i = 0; i < EPP; ++i) {
            float v = __uint_as_float(old_v[p][i]);
            adam_elem(a.opt, m[i], v, w[i], d[i]);
            v_out[i] = __float_as_uint(v);
          }
          store_words<WPP>(sq_base + at, v_out);
        }
        uint32_t m_out[WPP], w_out[WPP];
        pack_piece<T, WPP>(m, m_out);
        pack_piece<T, WPP>(w, w_out);
        store_words<WPP>(dst_base + at, m_out);
        store_words<WPP>(model_base + at, w_out);
      }
    }
  };

  uint32_t last_key = kNoRow;      // sorted records: key of the term before the 64 at hand
  for (int64_t q = begin; q < end; q += 64) {
    Term t;
    t.row = kNoRow; t.center = 0; t.coef = 0.f; t.pos = 0;
    const int n = (int)min((int64_t)64, end - q);
    if constexpr (kSorted) {
      if (lane < n) {
        t.row = a.term_key[q + lane];
        const uint2 src = a.term_src[q + lane];
        t.center = (int32_t)src.x;
        t.coef = __uint_as_float(src.y);
      }
      uint32_t before = (uint32_t)__shfl_up((int)t.row, 1, 64);
      if (lane == 0) before = (q == begin) ? t.row : last_key;
      const unsigned long long changes = __builtin_amdgcn_ballot_w64(lane < n && t.row != before);
      const unsigned long long upto = changes & ((2ull << lane) - 1ull);
      const int64_t run_first = upto != 0ull ? q + 63 - __builtin_clzll(upto) : first_row;
      t.pos = (uint32_t)(q + lane - run_first);
      if (changes != 0ull) first_row = q + 63 - __builtin_clzll(changes);
      last_key = (uint32_t)__builtin_amdgcn_readlane((int)t.row, n - 1);
    } else {
      if (lane < n) t = sorted[q + lane];
    }
#pragma unroll 1
    for (int b0 = 0; b0 < n; b0 += UB) {
      uint32_t u[UB][PPL][SW];
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (b0 + b < n) {
          const int64_t src = (int64_t)__builtin_amdgcn_readlane(t.center, b0 + b);
          const uint32_t* row_words = src_base + src * src_row_words;
#pragma unroll
          for (int p = 0; p < PPL; ++p) {
            if (piece_ok[p]) {
              load_words<SW>(row_words + (int64_t)(p * 64 + lane) * SW, u[b][p]);
            } else {
#pragma unroll
              for (int w = 0; w < SW; ++w) u[b][p][w] = 0u;
            }
          }
        }
      }
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (b0 + b < n) {
          const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)t.pos, b0 + b);
          if ((pos & seg_mask) == 0u) {                  // a segment starts here
            const uint32_t row = (uint32_t)__builtin_amdgcn_readlane((int)t.row, b0 + b);
            if (cur_row != kNoRow) flush(row == cur_row);
            cur_row = row;
            if constexpr (kSegments) {
              cur_seg = pos >> a.seg_shift;
              seg_first = q + b0 + b;
            }
            cur_terms = 0;
#pragma unroll
            for (int x = 0; x < EPL; ++x) acc[x] = 0;
            if (pos == 0u) {
              const uint32_t* row_words = dst_base + (int64_t)(cur_row - key_base) * dst_row_words;
#pragma unroll
              for (int p = 0; p < PPL; ++p) {
                if (!piece_ok[p]) continue;
                const int64_t in_row = (int64_t)(p * 64 + lane) * WPP;
                load_words<WPP>(row_words + in_row, old[p]);
                if constexpr (kOpt != kPlain)
                  load_words<WPP>(model_base + (int64_t)(cur_row - key_base) * dst_row_words + in_row, old_w[p]);
                if constexpr (kOpt == kAdam)
                  load_words<WPP>(sq_base + (int64_t)(cur_row - key_base) * dst_row_words + in_row, old_v[p]);
              }
            }
          }
          const double c =
              (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(t.coef), b0 + b)) *
              kFixScale;
#pragma unroll
          for (int p = 0; p < PPL; ++p)
#pragma unroll
            for (int i = 0; i < EPP; ++i) {
              const float x = kStage ? __uint_as_float(u[b][p][i]) : piece_elem<T, SW>(u[b][p], i);
              fix_add(acc[p * EPP + i], c, x);
            }
          ++cur_terms;
        }
      }
    }
  }
  // last pending segment: the row goes on if the term after the range has the same key
  if (cur_row != kNoRow)
    flush(kSegments && end < pos_hi && uniform_u32(kSorted ? a.term_key[end] : sorted[end].row) == cur_row);
}

// Ownership: the terms of a key are cut into segments of S = 2^seg_shift consecutive
// positions (pos = 0..S-1, S..2S-1, ...); a wave handles the segments whose first term lies
// in its slice, reading on past the slice's end to finish the last one.  A row of at most S
// terms is one segment: it is written once, as round(old + sum).  The partial sums of a row
// with more segments meet in the side buffer at slot (position of the row's first term) >>
// seg_shift, which no two such rows can share because each spans more than S positions.
// Context-table keys take the positions [0, num_terms), input-table keys the positions after them.
template <typename T, int WPP, int PPL, int UB, int kOpt, bool kStage>
__global__ __launch_bounds__(kSgnsThreads) void sgns_update_kernel(SgnsArgs a) {
  constexpr int kWaves = kSgnsThreads / 64;
  const int64_t pos_lo = kStage ? a.stage_base : 0;
  // (scalars that come out of memory are made wave-uniform explicitly: loop bounds and the
  // lane numbers of the broadcasts must live in scalar registers)
  const int64_t pos_hi = kStage ? (int64_t)uniform_u32(a.cnt[a.cnt_last]) : a.num_terms;
  const int lane = threadIdx.x & 63;
  const int64_t first_wave = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int slice = kStage ? kStageSlice : a.slice_terms;
  const Term* __restrict__ sorted = a.sorted;
  const uint32_t seg_mask = (1u << a.seg_shift) - 1u;
  // a wave takes the slices first_wave, first_wave + (waves of the launch), ...: the launch of
  // the input-table pass is sized for the few slots a batch normally uses, not for one per pair
  for (int64_t wave = first_wave;; wave += (int64_t)gridDim.x * kWaves) {
    const int64_t slice_begin = pos_lo + wave * slice;
    if (slice_begin >= pos_hi) break;
    const int64_t slice_end = min(slice_begin + slice, pos_hi);
    // what lies before `begin` is an earlier wave's; up to `end`: finish the segment we started (the 64 positions
    // behind either end, which almost always decide, are read together)
    const uint32_t behind_begin = slice_begin + lane < pos_hi ? sorted[slice_begin + lane].pos & seg_mask : 0u;
    const uint32_t behind_end = slice_end + lane < pos_hi ? sorted[slice_end + lane].pos & seg_mask : 0u;
    auto segment_start = [&](int64_t p, uint32_t behind) {
      const unsigned long long starts = __builtin_amdgcn_ballot_w64(behind == 0u);
      return starts != 0ull ? min(pos_hi, p + (int64_t)__builtin_ctzll(starts)) : next_segment_start(sorted, p + 64, pos_hi, lane, seg_mask);
    };
    const int64_t begin = segment_start(slice_begin, behind_begin);
    const int64_t end = segment_start(slice_end, behind_end);
    update_range<T, WPP, PPL, UB, kOpt, kStage, true>(a, sorted, begin, end, pos_hi, lane);
  }
}

// element-wise row helpers for the finishing kernel (natural order)
__device__ __forceinline__ float elem_load(const float* row, int e) { return row[e]; }
template <typename T, if_16bit<T> = 0>
__device__ __forceinline__ float elem_load(const T* row, int e) { return T::lo((uint32_t)row[e].bits); }
__device__ __forceinline__ void elem_store(float* row, int e, float v) { row[e] = v; }
template <typename T, if_16bit<T> = 0>
__device__ __forceinline__ void elem_store(T* row, int e, float v) { row[e].bits = (uint16_t)T::round(v); }

// ---- finish: table[row] = round(old + side buffer) for the long rows ------------------------
// one long row, by 16 lanes
template <typename T, int kOpt>
__device__ __forceinline__ void finish_row(const SgnsArgs& a, bool input_row, int64_t row, const unsigned long long* src, int l16) {
  T* dst = static_cast<T*>(input_row ? a.dst_in : a.dst_out) + row * (int64_t)a.dim;
  if constexpr (kOpt != kPlain) {
    T* model = static_cast<T*>(input_row ? a.w_in : a.w_out) + row * (int64_t)a.dim;
    for (int e = l16; e < a.dim; e += kGroupLanes) {
      float m = elem_load(dst, e), w = elem_load(model, e);
      if constexpr (kOpt == kMomentum) {
        momentum_elem<T>(a.opt, m, w, fix_value(src[e]));
      } else {
        float* sq = (input_row ? a.sq_in : a.sq_out) + row * (int64_t)a.dim + e;
        float v = *sq;
        adam_elem(a.opt, m, v, w, fix_value(src[e]));
        *sq = v;
      }
      elem_store(dst, e, m);
      elem_store(model, e, w);
    }
    return;
  }
  for (int e = l16; e < a.dim; e += kGroupLanes)
    elem_store(dst, e, (float)((double)elem_load(dst, e) + fix_value(src[e])));
}

// the per-block loss partials, in a fixed order, by one workgroup
__device__ __forceinline__ double sum_of_losses(const SgnsArgs& a) {
  __shared__ double sum_s[kSgnsThreads];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < a.forward_blocks; i += kSgnsThreads) acc += a.loss_partials[i];
  sum_s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kSgnsThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sum_s[threadIdx.x] += sum_s[threadIdx.x + w];
    __syncthreads();
  }
  return sum_s[0];
}

// Side-buffer slot s belongs to the long row (more than one segment of S = 2^seg_shift terms)
// whose first term lies in [s * S, (s+1) * S): that row then also owns the last position of
// the window.  The last block of the launch adds up the per-block
// loss partials instead (in a fixed order, so the loss is reproducible); a bad id
// or an out-of-range product seen by an earlier kernel turns it into NaN.
// which: 0 = long rows of both tables and the loss; 1 = context-table keys only, no loss;
// 2 = input-table keys and the loss.  With one table on both sides a row can be long under
// both of its keys, and its two read-modify-writes must not overlap: the context-table keys
// are then finished before the input-table keys are summed.
template <typename T, int kOpt>
__global__ __launch_bounds__(kSgnsThreads) void sgns_finish_kernel(SgnsArgs a, int which) {
  if (blockIdx.x == gridDim.x - 1) {
    if (which == 1) return;
    const double sum = sum_of_losses(a);
    if (threadIdx.x == 0)
      *a.loss_out = (*a.bad_ids != 0u) ? __longlong_as_double(0x7ff8000000000000ll) : sum;
    return;
  }
  const int l16 = threadIdx.x & (kGroupLanes - 1);
  const int64_t s = ((int64_t)blockIdx.x * kSgnsThreads + threadIdx.x) / kGroupLanes;
  const int64_t last_pos = ((s + 1) << a.seg_shift) - 1;
  const int64_t total = (int64_t)a.cnt[a.cnt_last];
  if (last_pos >= total) return;
  const Term t = a.sorted[last_pos];
  const int64_t first_pos = last_pos - (int64_t)t.pos;
  if ((first_pos >> a.seg_shift) != s) return;
  // long: the row has a term at position S
  const int64_t second = first_pos + ((int64_t)1 << a.seg_shift);
  if (second >= total || a.sorted[second].row != t.row) return;
  const bool input_row = (int64_t)t.row >= a.num_nodes;
  if (which != 0 && input_row != (which == 2)) return;
  const int64_t row = input_row ? (int64_t)t.row - a.num_nodes : (int64_t)t.row;
  const unsigned long long* src = reinterpret_cast<const unsigned long long*>(a.long_acc) +
                                  (s + (input_row ? a.stage_long_base : 0)) * (int64_t)a.dim;
  finish_row<T, kOpt>(a, input_row, row, src, l16);
}

// The same for grouped batches, whose long rows are in a list (which: as above; a bad id or an out-of-range product has made a
// partial NaN).
template <typename T, int kOpt>
__global__ __launch_bounds__(kSgnsThreads) void sgns_long_rows_kernel(SgnsArgs a, int which) {
  if (blockIdx.x == gridDim.x - 1) {
    if (which == 1) return;
    const double sum = sum_of_losses(a);
    if (threadIdx.x == 0) *a.loss_out = sum;
    return;
  }
  const int l16 = threadIdx.x & (kGroupLanes - 1);
  const uint32_t rows = *a.num_long_rows;
  for (uint32_t i = (blockIdx.x * kSgnsThreads + threadIdx.x) / kGroupLanes; i < rows; i += (gridDim.x - 1) * kGroupsPerBlock) {
    const uint2 r = a.long_rows[i];
    const bool input_row = (int64_t)r.x >= a.num_nodes;
    if (which != 0 && input_row != (which == 2)) continue;
    const unsigned long long* src = reinterpret_cast<const unsigned long long*>(a.long_acc) + (int64_t)r.y * a.dim;
    finish_row<T, kOpt>(a, input_row, input_row ? (int64_t)r.x - a.num_nodes : (int64_t)r.x, src, l16);
  }
}

// ---- large batches: the terms as records in the order of their rows --------------------------
// With many terms the counters cost more than bringing records together: a random atomic per term in the forward
// kernel, and in the place kernel a random read and a random 16-byte write per term, all of them whole
// cache lines.  The forward kernel writes each term as a record (row; source row, coefficient)
// instead, and the update kernels read the records as they lie in the order of their rows.
//   Up to 2^24 rows: grouped (group.hip), the records of both tables at once; the staging slots are the list with gaps.  Nothing is
//   cleared, counted per row or scanned; the grouping also says which rows have more than one segment and, for the optimizers, which rows
//   have any records.  12 million terms, 128 fp32 columns, 4 M nodes: a step takes 2256 us (2579 with the counters, 2411 with the
//   records of the context table through the stable sort in three passes); 65,536 pairs, 64 columns on 10 k nodes 90 (104 with the counters).
//   More rows: the radix sort brings the records of the context table into order; the few input-table terms keep their counters.

// First position >= p (p < hi; at most hi) that starts a segment of its row, and the row's first position, among the records [lo, hi).  keys: those of
// the 64 positions from p - 1 on (kNoRow outside); here and next: the entries of p's window and of the one behind it.  The caller loads them, so
// that the loads of both ends of a slice are under way together.  A row's first segment starts where the keys change; where its further ones
// do, whoever brought the records together has written down.  (Searching for the row's first record instead, 64 reads of 64 cache lines, several times, at
// both ends of every slice in a long row: 7.3 M terms of walks on 5000 nodes, 20 columns 322 us for the context table, now 306; 1.2 M with one negative,
// 104 columns 103 and, for the input table, 47, now 96 and 45; 12 M on 4 M nodes, 128 columns 964 and 72, now 962 and 71.)
__device__ __forceinline__ int64_t sorted_segment_start(const SgnsArgs& a, int64_t p, int lane, uint32_t keys, uint2 here, uint2 next,
                                                        int64_t hi, int64_t& first_row) {
  const int64_t none = (int64_t)1 << 62;
  int64_t further = none;                                            // a further segment of p's row
  if (uniform_u32(here.x) != kNoRow && (int64_t)uniform_u32(here.x) >= p) {
    further = (int64_t)uniform_u32(here.x);
    first_row = (int64_t)uniform_u32(here.y);
  } else if (uniform_u32(next.x) != kNoRow) {
    further = (int64_t)uniform_u32(next.x);
    first_row = (int64_t)uniform_u32(next.y);
  }
  for (int64_t q = p;; q += 63) {
    if (q > further) return further;
    if (q != p) keys = q - 1 + lane < hi ? a.term_key[q - 1 + lane] : kNoRow;
    const uint32_t before = (uint32_t)__shfl_up((int)keys, 1, 64);   // (by every lane: lane 1 wants lane 0's)
    const unsigned long long changes = __builtin_amdgcn_ballot_w64(keys != before) & ~1ull;
    if (changes == 0ull) continue;                                   // (a segment has at most 2^seg_shift records, and behind hi there is none)
    const int64_t row = q - 1 + __builtin_ctzll(changes);
    if (further < row) return further;
    first_row = row;
    return row;
  }
}

// kStage: the records of the input-table rows, which follow those of the context table (grouped batches); their number is on
// the device, so the launch is sized for the few that a batch normally has and its waves stride over the slices.  further (behind SgnsArgs: one more
// field in there costs the forward kernel of narrow rows 12 %): entry w tells of the records [w << seg_shift, (w + 1) << seg_shift) the one that starts
// a segment of a row other than its first, and the row's first record; else kNoRow.
template <typename T, int WPP, int PPL, int UB, int kOpt, bool kStage>
__global__ __launch_bounds__(kSgnsThreads) void sgns_sorted_update_kernel(SgnsArgs a, const uint2* __restrict__ further) {
  const uint32_t* __restrict__ keys = a.term_key;
  const int lane = threadIdx.x & 63;
  const int64_t first_wave = (int64_t)blockIdx.x * (kSgnsThreads / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t lo = kStage ? a.num_terms : 0, hi = kStage ? (int64_t)uniform_u32(*a.num_records) : a.num_terms;
  const int64_t slice = kStage ? kStageSlice : a.slice_terms;
  for (int64_t wave = first_wave;; wave += (int64_t)gridDim.x * (kSgnsThreads / 64)) {
    const int64_t p0 = lo + wave * slice;
    if (p0 >= hi) return;
    const int64_t p1 = min(p0 + slice, hi);
    auto key_at = [&](int64_t p) { return p >= lo && p < hi ? keys[p] : kNoRow; };
    const uint32_t keys0 = key_at(p0 - 1 + lane), keys1 = key_at(p1 - 1 + lane);
    const uint2 here0 = further[p0 >> a.seg_shift], next0 = further[(p0 >> a.seg_shift) + 1];
    const uint2 here1 = further[p1 >> a.seg_shift], next1 = further[(p1 >> a.seg_shift) + 1];
    int64_t first_row, unused;
    const int64_t begin = sorted_segment_start(a, p0, lane, keys0, here0, next0, hi, first_row);
    const int64_t end = p1 < hi ? sorted_segment_start(a, p1, lane, keys1, here1, next1, hi, unused) : hi;
    update_range<T, WPP, PPL, UB, kOpt, kStage, true, true>(a, nullptr, begin, end, hi, lane, first_row);
    if constexpr (!kStage) return;               // (one slice per wave)
  }
}

// The long rows (more than one segment) of the sorted terms, 16 lanes per side-buffer slot: slot s
// belongs to the row whose first term lies in positions [s * S, (s + 1) * S), if that row goes on for more
// than S terms.  kZero: clears the slot, and writes down where a further segment of a row starts in those positions; else table[row] =
// round(old + slot).
template <typename T, bool kZero>
__global__ __launch_bounds__(kSgnsThreads) void sgns_sorted_long_kernel(SgnsArgs a, uint2* __restrict__ further) {
  const uint32_t* __restrict__ keys = a.term_key;
  const int l16 = threadIdx.x & (kGroupLanes - 1);
  const int64_t s = ((int64_t)blockIdx.x * kSgnsThreads + threadIdx.x) / kGroupLanes;
  const int64_t low = s << a.seg_shift, after = (s + 1) << a.seg_shift;
  if constexpr (kZero) {
    if (s > a.stage_long_base) return;
    uint2 start_and_row = make_uint2(kNoRow, 0u);
    if (low > 0 && low < a.num_terms && keys[low - 1] == keys[low]) {
      // the row goes back: if it has more than S records, half a segment away on one side or the other are some of them
      const uint32_t key = keys[low];
      const int64_t half = (int64_t)1 << (a.seg_shift - 1);
      if ((low >= half && keys[low - half] == key) || (low + half < a.num_terms && keys[low + half] == key)) {
        int64_t hi = low - 1, step = half;                             // (keys[hi] == key)
        int64_t lo = max((int64_t)0, hi - step);
        while (lo > 0 && keys[lo] == key) {
          hi = lo;
          step *= 2;
          lo = max((int64_t)0, hi - step);
        }
        while (lo < hi) {
          const int64_t mid = (lo + hi) >> 1;
          if (keys[mid] < key) lo = mid + 1; else hi = mid;
        }
        const int64_t segment = (int64_t)1 << a.seg_shift;
        const int64_t start = lo + ((low - lo + segment - 1) & ~(segment - 1));
        if (start < a.num_terms && keys[start] == key) start_and_row = make_uint2((uint32_t)start, (uint32_t)lo);
      }
    }
    if (l16 == 0) further[s] = start_and_row;
  }
  if (after >= a.num_terms) return;
  const uint32_t key = keys[after];
  if (keys[after - 1] != key) return;
  int64_t lo = low, hi = after - 1;                      // first position of the row in the window
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < key) lo = mid + 1; else hi = mid;
  }
  if (lo == low && lo > 0 && keys[lo - 1] == key) return;                  // started in an earlier window
  const int64_t second = lo + ((int64_t)1 << a.seg_shift);
  if (second >= a.num_terms || keys[second] != key) return;
  unsigned long long* acc = reinterpret_cast<unsigned long long*>(a.long_acc) + s * (int64_t)a.dim;
  if constexpr (kZero) {
    for (int e = l16; e < a.dim; e += kGroupLanes) acc[e] = 0ull;
  } else {
    T* dst = static_cast<T*>(a.dst_out) + (int64_t)key * a.dim;
    for (int e = l16; e < a.dim; e += kGroupLanes)
      elem_store(dst, e, (float)((double)elem_load(dst, e) + fix_value(acc[e])));
  }
}

// ---- small batches: the whole step in two launches -----------------------------------------
// Bound by latency: the kernels above are a chain of seven dependent launches, each a few microseconds
// for a batch of a few thousand pairs (2048 pairs, 5 negatives, 128 columns on 1 M nodes: 82 us; the
// two launches here: 25 us, 9 in the forward kernel and 17 in the update kernel).  Here the forward kernel counts nothing, and one kernel of
// kSmallBlocks workgroups does the rest: a workgroup owns the keys whose hash names it, reads all
// ids of the batch (they fit the L2), counts its keys in an LDS table, brings its terms together
// in LDS and sums and writes its rows.  Both kinds of keys are handled at once, because the source
// rows of the context-table keys are the copies the forward kernel kept, not the input table.
// Rows of more than kSmallRow terms are summed by the whole workgroup, which picks their terms from
// the ids as it goes.  Should the keys of a workgroup not fit its table or its terms their place in
// LDS (ids that share a hash, rows of just under kSmallRow terms), it sums all its rows that way.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int kSmallBlockBits = 8, kSmallBlocks = 1 << kSmallBlockBits;
constexpr int kSmallSlotBits = 10, kSmallSlots = 1 << kSmallSlotBits;
constexpr int kSmallTerms = 2048;
constexpr uint32_t kSmallRow = 64;
constexpr int kSmallMaxDim = 512;
constexpr int kSmallMaxRowBytes = 1024;
constexpr int kSmallChunkPairs = 2;              // consecutive pairs per 16-lane group in forward
constexpr int kSmallForwardThreads = 64;
static_assert(kSmallThreads == kSmallSlots, "the prefix sum takes one slot per lane");

// entry e of the batch: contexts, then negatives, then staging slots; its key (kNoRow: none)
__device__ __forceinline__ uint32_t small_key(const SgnsArgs& a, uint32_t e, uint32_t pairs, uint32_t terms) {
  if (e < terms) {
    const int32_t id = e < pairs ? a.contexts[e] : a.negs[e - pairs];
    return (uint32_t)id < (uint32_t)a.num_nodes ? (uint32_t)id : 0u;
  }
  if (e >= terms + pairs) return kNoRow;
  const int32_t c = a.stage_center[e - terms];
  return c < 0 ? kNoRow : (uint32_t)a.num_nodes + (uint32_t)c;
}
// its source row and coefficient
__device__ __forceinline__ void small_source(const SgnsArgs& a, uint32_t e, uint32_t pairs, uint32_t terms,
                                             int32_t& center, float& coef) {
  if (e >= terms) {
    center = (int32_t)(e - terms);
    coef = -a.lr;
    return;
  }
  const uint32_t k = (uint32_t)a.k;
  const uint32_t i = e < pairs ? e : (e - pairs) / k;
  const uint32_t j = e < pairs ? 0u : e - pairs - i * k + 1u;
  center = a.pair_slot[i];
  coef = -a.lr * a.g[i * (k + 1u) + j];
}
__device__ __forceinline__ uint32_t small_hash(uint32_t key) { return key * 2654435761u; }
__device__ __forceinline__ bool small_owns(uint32_t key) {
  return key != kNoRow && (small_hash(key) >> (32 - kSmallBlockBits)) == blockIdx.x;
}
__device__ __forceinline__ uint32_t small_home(uint32_t key) {
  return (small_hash(key) >> (32 - kSmallBlockBits - kSmallSlotBits)) & (uint32_t)(kSmallSlots - 1);
}

// The row of `key`, summed by the whole workgroup: every wave picks the key's entries out of its
// share of the ids, 64 at a time, and adds their source rows; the waves' sums meet in row_acc.
template <typename T, int WPP, int UB, bool kStage>
__device__ void small_long_row(const SgnsArgs& a, uint32_t key, uint32_t pairs, uint32_t terms,
                               unsigned long long* row_acc, uint32_t* found) {
  constexpr int EPP = WPP * Words<T>::kPerWord;
  constexpr int SW = kStage ? EPP : WPP;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t entries = terms + pairs;
  const uint32_t* __restrict__ src_base = static_cast<const uint32_t*>(kStage ? static_cast<const void*>(a.stage_delta) : a.snap);
  const int64_t src_row_words = kStage ? (int64_t)a.dim : (int64_t)a.dim / Words<T>::kPerWord;
  const bool piece_ok = lane * EPP < a.dim;
  if (tid < a.dim) row_acc[tid] = 0ull;
  __syncthreads();
  unsigned long long acc[EPP];
#pragma unroll
  for (int i = 0; i < EPP; ++i) acc[i] = 0ull;
  uint32_t summed = 0;
  auto add = [&](int n) {                                 // the first n entries of `found`
    int32_t center = 0;
    float coef = 0.f;
    if (lane < n) small_source(a, found[lane], pairs, terms, center, coef);
#pragma unroll 1
    for (int b0 = 0; b0 < n; b0 += UB) {
      uint32_t u[UB][SW];
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (b0 + b < n) {
          const uint32_t* row_words = src_base + (int64_t)__builtin_amdgcn_readlane(center, b0 + b) * src_row_words;
          if (piece_ok) load_words<SW>(row_words + (int64_t)lane * SW, u[b]);
          else
#pragma unroll
            for (int w = 0; w < SW; ++w) u[b][w] = 0u;
        }
      }
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (b0 + b < n) {
          const double c = (double)__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(coef), b0 + b)) * kFixScale;
#pragma unroll
          for (int i = 0; i < EPP; ++i)
            fix_add(acc[i], c, kStage ? __uint_as_float(u[b][i]) : piece_elem<T, SW>(u[b], i));
        }
      }
    }
    summed += (uint32_t)n;
  };
  int held = 0;
  for (uint32_t e0 = wave * 64u; e0 < entries; e0 += kSmallThreads) {
    const bool match = small_key(a, e0 + (uint32_t)lane, pairs, terms) == key;
    const uint64_t votes = __ballot(match);
    if (votes == 0ull) continue;
    if (match) found[held + __popcll(votes & ((1ull << lane) - 1ull))] = e0 + (uint32_t)lane;
    held += __popcll(votes);
    wave_fence();
    if (held >= 64) {
      add(64);
      held -= 64;
      const uint32_t rest = found[64 + lane];
      wave_fence();
      if (lane < held) found[lane] = rest;
      wave_fence();
    }
  }
  if (held > 0) add(held);
  if (summed > 0 && piece_ok) {
    const unsigned long long off = (unsigned long long)(summed * (uint32_t)(kFixMagicBits >> 32)) << 32;
#pragma unroll
    for (int i = 0; i < EPP; ++i) atomicAdd(row_acc + lane * EPP + i, acc[i] - off);
  }
  __syncthreads();
  if (tid < a.dim) {
    T* row = static_cast<T*>(kStage ? a.dst_in : a.dst_out) + (int64_t)(kStage ? key - (uint32_t)a.num_nodes : key) * a.dim;
    elem_store(row, tid, (float)((double)elem_load(row, tid) + fix_value(row_acc[tid])));
  }
  __syncthreads();
}

template <typename T, int WPP, int UB>
__global__ __launch_bounds__(kSmallThreads) void sgns_small_update_kernel(SgnsArgs a) {
  __shared__ uint32_t keys[kSmallSlots], cnt[kSmallSlots], off[kSmallSlots];
  __shared__ uint32_t long_keys[kSmallSlots];
  __shared__ __align__(16) Term terms_s[kSmallTerms];     // (the loss block keeps doubles here)
  __shared__ uint2 owned[kSmallTerms];                    // entry; slot and position among the terms of its key
  __shared__ unsigned long long row_acc[kSmallMaxDim];
  __shared__ uint32_t found[kSmallWaves][128];
  __shared__ uint32_t wave_tot[2][kSmallWaves];
  __shared__ uint32_t n_long, n_owned, failed, next_key;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (blockIdx.x == kSmallBlocks) {                       // the loss: partials added in a fixed order
    double* sum_s = reinterpret_cast<double*>(terms_s);
    double sum = 0.0;
    for (int64_t i = tid; i < a.forward_blocks; i += kSmallThreads) sum += a.loss_partials[i];
    sum_s[tid] = sum;
    __syncthreads();
    for (int w = kSmallThreads / 2; w > 0; w >>= 1) {
      if (tid < w) sum_s[tid] += sum_s[tid + w];
      __syncthreads();
    }
    if (tid == 0) *a.loss_out = sum_s[0];
    return;
  }
  const uint32_t pairs = (uint32_t)a.num_pairs, terms = (uint32_t)a.num_terms, entries = terms + pairs;
  const uint32_t nodes = (uint32_t)a.num_nodes;
  keys[tid] = kNoRow;
  cnt[tid] = 0u;
  if (tid == 0) { n_long = 0u; n_owned = 0u; failed = 0u; }
  __syncthreads();

  constexpr int kBatch = 8;                               // ids in flight per lane
  for (uint32_t e0 = 0; e0 < entries; e0 += kBatch * kSmallThreads) {
    uint32_t key[kBatch];
#pragma unroll
    for (int c = 0; c < kBatch; ++c) key[c] = small_key(a, e0 + c * kSmallThreads + tid, pairs, terms);
#pragma unroll
    for (int c = 0; c < kBatch; ++c) {
      if (!small_owns(key[c])) continue;
      uint32_t at = small_home(key[c]);
      int probes = 0;
      for (; probes < kSmallSlots; ++probes, at = (at + 1u) & (kSmallSlots - 1)) {
        const uint32_t seen = atomicCAS(&keys[at], kNoRow, key[c]);
        if (seen == kNoRow || seen == key[c]) break;
      }
      if (probes == kSmallSlots) { failed = 1u; continue; }
      const uint32_t pos = atomicAdd(&cnt[at], 1u);
      if (pos >= kSmallRow) continue;                     // (a long row: its terms are picked later)
      const uint32_t i = atomicAdd(&n_owned, 1u);
      if (i < (uint32_t)kSmallTerms) owned[i] = make_uint2(e0 + c * kSmallThreads + tid, (at << 8) | pos);
    }
  }
  __syncthreads();
  // places: the short context rows first, then the short input rows
  uint32_t n_out = 0, n_in = 0;
  {
    const uint32_t c = cnt[tid], key = keys[tid];
    const bool is_short = c <= kSmallRow;
    const uint32_t c_out = is_short && key < nodes ? c : 0u, c_in = is_short && key >= nodes ? c : 0u;
    if (!is_short) long_keys[atomicAdd(&n_long, 1u)] = key;
    uint32_t i_out = c_out, i_in = c_in;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t u0 = __shfl_up(i_out, d, 64), u1 = __shfl_up(i_in, d, 64);
      if (lane >= d) { i_out += u0; i_in += u1; }
    }
    if (lane == 63) { wave_tot[0][wave] = i_out; wave_tot[1][wave] = i_in; }
    __syncthreads();
    uint32_t b_out = 0, b_in = 0;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) {
      if (w < wave) { b_out += wave_tot[0][w]; b_in += wave_tot[1][w]; }
      n_out += wave_tot[0][w];
      n_in += wave_tot[1][w];
    }
    off[tid] = !is_short ? kNoRow : (key < nodes ? b_out + i_out - c_out : n_out + b_in + i_in - c_in);
    __syncthreads();
  }
  n_out = uniform_u32(n_out);
  n_in = uniform_u32(n_in);
  uint32_t* my_found = found[wave];
  if (failed != 0u || n_owned > (uint32_t)kSmallTerms) {
    // does not fit: every key of this workgroup on its own, in ascending order
    for (uint32_t lowest = 0;;) {
      if (tid == 0) next_key = kNoRow;
      __syncthreads();
      uint32_t best = kNoRow;
      for (uint32_t e = tid; e < entries; e += kSmallThreads) {
        const uint32_t key = small_key(a, e, pairs, terms);
        if (key >= lowest && key < best && small_owns(key)) best = key;
      }
      if (best != kNoRow) atomicMin(&next_key, best);
      __syncthreads();
      const uint32_t key = uniform_u32(next_key);
      if (key == kNoRow) return;
      if (key < nodes) small_long_row<T, WPP, UB, false>(a, key, pairs, terms, row_acc, my_found);
      else small_long_row<T, WPP, UB, true>(a, key, pairs, terms, row_acc, my_found);
      lowest = key + 1u;
    }
  }
  for (uint32_t i = tid; i < n_owned; i += kSmallThreads) {
    const uint2 o = owned[i];
    const uint32_t at = o.y >> 8;
    if (off[at] == kNoRow) continue;
    Term t;
    t.row = keys[at];
    t.pos = o.y & 255u;
    small_source(a, o.x, pairs, terms, t.center, t.coef);
    terms_s[off[at] + t.pos] = t;
  }
  __syncthreads();
  const uint32_t s_out = min(64u, (n_out + kSmallWaves - 1) / kSmallWaves), s_in = min(64u, (n_in + kSmallWaves - 1) / kSmallWaves);
  for (uint32_t at = (uint32_t)wave * s_out; at < n_out; at += kSmallWaves * s_out) {
    const int64_t begin = next_segment_start(terms_s, at, n_out, lane, ~0u);
    const int64_t end = next_segment_start(terms_s, min(at + s_out, n_out), n_out, lane, ~0u);
    update_range<T, WPP, 1, UB, kPlain, false, false>(a, terms_s, begin, end, n_out, lane);
  }
  const uint32_t n_all = n_out + n_in;
  for (uint32_t at = n_out + (uint32_t)wave * s_in; at < n_all; at += kSmallWaves * s_in) {
    const int64_t begin = next_segment_start(terms_s, at, n_all, lane, ~0u);
    const int64_t end = next_segment_start(terms_s, min(at + s_in, n_all), n_all, lane, ~0u);
    update_range<T, WPP, 1, UB, kPlain, true, false>(a, terms_s, begin, end, n_all, lane);
  }
  const uint32_t longs = uniform_u32(n_long);
  for (uint32_t l = 0; l < longs; ++l) {
    const uint32_t key = uniform_u32(long_keys[l]);
    if (key < nodes) small_long_row<T, WPP, UB, false>(a, key, pairs, terms, row_acc, my_found);
    else small_long_row<T, WPP, UB, true>(a, key, pairs, terms, row_acc, my_found);
  }
}

// ---- host side -----------------------------------------------------------------------------
// Work per 16-lane group: large batches fill the chip many times over, so long runs per
// group amortise the row loads of a run of equal centres; small batches are cut finer so
// that every compute unit gets work and the dependent loads of a group stay few.
static int chunk_pairs_for(int64_t num_pairs) {
  return num_pairs >= (1 << 20) ? 16 : (num_pairs >= (1 << 18) ? 8 : 4);
}
static int slice_terms_for(int64_t num_pairs) {
  return num_pairs >= (1 << 20) ? 128 : (num_pairs >= (1 << 18) ? 64 : 32);
}
static int seg_shift_for(int64_t num_pairs) {
  return num_pairs >= (1 << 18) ? kSegShiftLarge : kSegShiftSmall;
}
static int64_t forward_blocks_for(int64_t num_pairs) {
  return ceil_div(ceil_div(num_pairs, chunk_pairs_for(num_pairs)), kGroupsPerBlock);
}

struct SgnsPlan {
  double* loss_partials;
  float* g;
  uint32_t* rank;
  uint32_t* cnt;
  int64_t cnt_last;         // counters are cnt[0 .. cnt_last]
  uint32_t* key_table;      // tables of the batch's keys (null: none)
  int64_t table_places;
  int32_t out_bits, in_bits;
  uint32_t in_base;
  uint32_t* tile_sums;
  uint32_t* bad_ids;
  Term* sorted;
  long long* long_acc;
  int32_t* stage_center;
  uint32_t* stage_rank;
  float* stage_delta;
  int64_t long_slots;
  int32_t seg_shift;
  bool small = false;       // the two-launch step of a small batch, which keeps copies of the input rows
  void* snap = nullptr;
  int32_t* pair_slot = nullptr;
  bool by_sort = false;     // the context-table terms as sorted records (large batches on very many rows)
  bool grouped = false;     // records of both tables, grouped by row (large batches)
  GroupArgs group = {};
  uint32_t* term_key[2] = {nullptr, nullptr};      // [0] holds the sorted ones
  uint2* term_src[2] = {nullptr, nullptr};
  void* sort_scratch = nullptr;
  size_t sort_bytes = 0;
  int64_t stage_base = 0, stage_long_base = 0;
  size_t bytes;
};

// force_compact: always count over the table of the batch's keys, whatever the graph's size,
// so that the workspace depends on (num_pairs, k, dim) only
static SgnsPlan plan_sgns(void* ws, int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim,
                          bool force_compact = false) {
  Carver cv(ws);
  SgnsPlan p;
  const size_t b = (size_t)(num_pairs > 0 ? num_pairs : 1);
  const size_t terms = b * (size_t)(k + 1);
  const size_t keys = 2 * (size_t)(num_nodes > 0 ? num_nodes : 1);
  // A counter per key while the keys are few.  For graphs much larger than the batch (the
  // paper's own batches of 512 to 2048 source nodes on graphs of 10^8 and more vertices) the
  // counters go over the places of a table of the keys the batch holds (at most one per term
  // and per pair): everything that is cleared, scanned or hit at random in a call then has
  // the size of the batch, not of the graph.
  // (a table has at least twice as many places as there can be keys of its kind)
  const size_t nodes = keys / 2;
  const bool compact = force_compact || keys > kCompactFactor * (terms + b);
  int in_bits = 8, out_bits = 8;
  while (((size_t)1 << out_bits) < 2 * terms) ++out_bits;
  while (((size_t)1 << in_bits) < 2 * b) ++in_bits;
  p.out_bits = compact ? out_bits : 0;
  p.in_bits = (compact || ((size_t)1 << in_bits) < nodes) ? in_bits : 0;
  const size_t out_slots = p.out_bits ? (size_t)1 << p.out_bits : nodes;
  const size_t in_slots = p.in_bits ? (size_t)1 << p.in_bits : nodes;
  p.in_base = (uint32_t)out_slots;
  p.table_places = (int64_t)((p.out_bits ? (size_t)1 << p.out_bits : 0) + (p.in_bits ? (size_t)1 << p.in_bits : 0));
  p.cnt_last = (int64_t)(out_slots + in_slots);
  p.seg_shift = seg_shift_for((int64_t)b);
  p.long_slots = (int64_t)((terms + b) >> p.seg_shift) + 1;
  p.stage_base = (int64_t)terms;
  p.loss_partials = cv.take<double>((size_t)forward_blocks_for((int64_t)b));
  p.g = cv.take<float>(terms);
  p.rank = cv.take<uint32_t>(terms);
  p.cnt = cv.take<uint32_t>((size_t)p.cnt_last + 1 + 3);                   // cleared 16 bytes at a time
  p.key_table = p.table_places > 0 ? cv.take<uint32_t>((size_t)p.table_places) : nullptr;
  p.tile_sums = cv.take<uint32_t>((size_t)ceil_div(p.cnt_last + 1, kScanTile));
  p.bad_ids = cv.take<uint32_t>(1);
  p.sorted = cv.take<Term>(terms + b);
  p.long_acc = cv.take<long long>((size_t)p.long_slots * (size_t)dim);
  p.stage_center = cv.take<int32_t>(b);
  p.stage_rank = cv.take<uint32_t>(b);
  p.stage_delta = cv.take<float>(b * (size_t)dim);
  p.bytes = cv.used;
  return p;
}

// Batches of at least this many terms on more rows than can be grouped take the sorted records.  Times of the counters over those
// of the records (in four passes of 8 bits; three of 9 are faster): 4.8 M terms on 18 M rows 1.02 to 1.14, 16 M terms 1.06 to 1.16; 25 M rows of 256
// bf16 columns, 22 M terms 8697 / 7879 us; 100 M rows of 128 fp32 columns, 24 M terms 11866 / 10166 us.  On fewer rows the records are grouped; in a workspace
// that has no room for that but for the sorted ones, which take up to 3 % less, these still beat the counters (2 M pairs, 128 fp32 columns, 4 M
// nodes 2411 / 2579 us).  Few rows with busy counters: from fewer terms on (batches of walks, counters over records: 65,536 rows and less,
// 2.0 M terms 0.99 to 1.23; 100 k rows, 4.8 M terms 0.90 to 1.07, 8 M 1.02 to 1.21).
constexpr int64_t kSortedMinTerms = (int64_t)9 << 19, kSortedMinTermsFewRows = (int64_t)3 << 21, kSortedFewRows = (int64_t)1 << 17;
constexpr int64_t kSortedMinTermsFewest = (int64_t)1 << 20, kSortedFewestRows = (int64_t)1 << 16;
// Sorted terms per wave of the update: the ends of a slice cost four loads of keys (256 against 128 terms:
// 2407 / 2425 us for 12 million terms on 4 M rows), and a short batch has to make enough waves.
static int sorted_slice_for(int64_t num_terms) { return num_terms >= ((int64_t)1 << 22) ? 256 : 128; }

static int bits_for_rows(int64_t num_nodes) {
  int b = 1;
  while (((int64_t)1 << b) < num_nodes) ++b;
  return b;
}

// wide: with room for the fewest passes of the sort
static SgnsPlan plan_sorted(void* ws, int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim, bool wide) {
  Carver cv(ws);
  SgnsPlan p = {};
  const size_t b = (size_t)num_pairs, terms = b * (size_t)(k + 1), nodes = (size_t)num_nodes;
  p.by_sort = true;
  // counters of the input-table keys alone, as in plan_sgns
  int in_bits = 8;
  while (((size_t)1 << in_bits) < 2 * b) ++in_bits;
  p.in_bits = ((size_t)1 << in_bits) < nodes ? in_bits : 0;
  p.cnt_last = (int64_t)(p.in_bits ? (size_t)1 << p.in_bits : nodes);
  p.table_places = p.in_bits ? (int64_t)1 << p.in_bits : 0;
  p.seg_shift = seg_shift_for(num_pairs);
  p.stage_long_base = (int64_t)(terms >> p.seg_shift) + 1;
  p.long_slots = (int64_t)(b >> p.seg_shift) + 1;            // of the input-table rows
  p.loss_partials = cv.take<double>((size_t)forward_blocks_for(num_pairs));
  for (int i = 0; i < 2; ++i) {
    p.term_key[i] = cv.take<uint32_t>(terms);
    p.term_src[i] = cv.take<uint2>(terms);
  }
  // (behind the sort, its scratch memory holds `further`)
  p.sort_bytes = std::max(radix_sort_scratch_bytes((int64_t)terms, wide), ((terms >> p.seg_shift) + 2) * sizeof(uint2));
  p.sort_scratch = cv.take<char>(p.sort_bytes);
  p.cnt = cv.take<uint32_t>((size_t)p.cnt_last + 1 + 3);                   // cleared 16 bytes at a time
  p.key_table = p.table_places > 0 ? cv.take<uint32_t>((size_t)p.table_places) : nullptr;
  p.tile_sums = cv.take<uint32_t>((size_t)ceil_div(p.cnt_last + 1, kScanTile));
  p.bad_ids = cv.take<uint32_t>(1);
  p.sorted = cv.take<Term>(b);
  p.long_acc = cv.take<long long>((size_t)(p.stage_long_base + p.long_slots) * (size_t)dim);
  p.stage_center = cv.take<int32_t>(b);
  p.stage_rank = cv.take<uint32_t>(b);
  p.stage_delta = cv.take<float>(b * (size_t)dim);
  p.bytes = cv.used;
  return p;
}

// Records of both kinds of rows, grouped.
static SgnsPlan plan_grouped(void* ws, int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim) {
  Carver cv(ws);
  SgnsPlan p = {};
  const size_t b = (size_t)num_pairs, terms = b * (size_t)(k + 1);
  p.grouped = true;
  p.seg_shift = seg_shift_for(num_pairs);
  p.long_slots = (int64_t)((terms + b) >> p.seg_shift) + 1;
  p.loss_partials = cv.take<double>((size_t)forward_blocks_for(num_pairs));
  for (int i = 0; i < 2; ++i) {
    p.term_key[i] = cv.take<uint32_t>(terms + b);
    p.term_src[i] = cv.take<uint2>(terms + b);
  }
  group_take(p.group, cv, (int64_t)terms, num_pairs, num_nodes, p.seg_shift, true);
  p.long_acc = cv.take<long long>((size_t)p.long_slots * (size_t)dim);
  p.stage_center = cv.take<int32_t>(b);
  p.stage_delta = cv.take<float>(b * (size_t)dim);
  p.bytes = cv.used;
  return p;
}
// Batches of at least this many terms are grouped: fewer on few rows, whose counters are busy.  Times of the counters over those of the
// records, 755 batches of walks and negatives (windows of 2 to 10) and of LINE on R-MAT graphs, momentum and Adam among them, 16 to 256 columns (least and most
// of them; with one negative, with more):
//   5 k and 10 k rows    0.33 M terms 1.06 to 1.13, 1.04 to 1.12; 0.5 M 1.00 to 1.24, 1.08 to 1.24; 1.2 M 0.98 to 1.16, 1.03 to 1.28; 3 M and more 1.15 to 1.46
//   20 k to 2^16         0.33 M 0.99 to 1.12, 1.01 to 1.13; 0.5 M 0.97 to 1.13, 1.01 to 1.18; 1.2 M 0.96 to 1.07, 1.01 to 1.27; 3 M 1.09 to 1.38
//   2^16 to 100 k        0.4 M 0.94 to 1.05, 0.94 to 1.06; 0.66 M 1.01 to 1.08, 0.98 to 1.11; 1.2 M 1.00, 1.01 to 1.12; 3 M 1.05 to 1.31
//   300 k                0.4 M 0.96 to 1.00, 0.99 to 1.08; 0.66 M 1.03, 0.99 to 1.12; 1.2 M 0.97 to 1.11, 0.99 to 1.09; 3 M 1.07 to 1.19
//   1 M and 2 M          0.4 M 1.00 to 1.09, 0.92 to 1.06; 0.66 M 1.11 to 1.29, 0.98 to 1.19; 1.2 M 1.01 to 1.10, 1.07 to 1.15; 3 M 1.09 to 1.39
// (Below 0.98 of those that are grouped: five of 607, four of them of one negative on rows of 32 to 48 bytes.)
constexpr int64_t kGroupedMinTerms = (int64_t)5 << 17, kGroupedMinTermsFewRows = (int64_t)5 << 16, kGroupedFewRows = (int64_t)1 << 16;
static bool grouped_batch(int64_t num_pairs, int64_t num_nodes, int32_t k) {
  return num_pairs * (int64_t)(k + 1) >= (num_nodes <= kGroupedFewRows ? kGroupedMinTermsFewRows : kGroupedMinTerms) && can_group(num_nodes);
}
// Records per wave of the update (us with 32 / 64 / 128 / 256): 0.4 M terms on 10 k rows of 64 columns 108 / 99 / 102 / 117, on 1 M rows of 128 151 /
// 156 / 166 / 209, 1.6 M 387 / 376 / 383 / 406, 2.4 M 591 / 563 / 554 / 555, 6 M 1210 / 1127 / 1095 / 1100, 12 M 2472 / 2345 / 2282 / 2256
static int grouped_slice_for(int64_t num_terms) {
  return num_terms >= ((int64_t)1 << 23) ? 256 : (num_terms >= ((int64_t)1 << 21) ? 128 : 64);
}

static bool sorted_batch(int64_t num_pairs, int64_t num_nodes, int32_t k) {
  const int64_t terms = num_pairs * (int64_t)(k + 1);
  if (num_nodes <= kSortedFewestRows) return terms >= (k >= 2 ? kSortedMinTermsFewest : 2 * kSortedMinTermsFewest);
  return terms >= (num_nodes <= kSortedFewRows ? kSortedMinTermsFewRows : kSortedMinTerms);
}

// Batches of at most this many ids (contexts, negatives, centres) take the two-launch step: every
// workgroup of its update kernel reads all of them, so its time grows with the ids (about 0.8 us
// per 1000) while that of the seven launches hardly does.  Measured, seven launches against two, with
// 5 negatives and 128 fp32 columns on 1 M nodes: 2048 pairs (14 k ids) 82 / 25 us, 6000 (42 k) 81 /
// 46, 12,000 (84 k) 89 / 105; 64 columns on 10 k nodes: 4096 (29 k) 50 / 38, 6000 53 / 46, 8192 (57 k)
// 54 / 59; 10 negatives, 256 bf16 columns on 500 k nodes: 4096 (49 k) 123 / 64, 8192 (98 k) 117 / 125.
constexpr int64_t kSmallMaxEntries = 3 << 14;
// A row is summed by one workgroup (about 14 ns a term with 128 fp32 columns, in fp64 instructions), and one of
// more than kSmallRow terms costs a look at all ids as well, so the step must not be taken by batches with long
// rows.  The ids are on the device; of a skewed graph the most frequent one has a share of about one
// in sqrt(num_nodes), which leaves such batches of at most sqrt(2^17 * num_nodes) ids.  Seven launches against
// two, R-MAT graphs, walks, k = 5 and 128 columns: 10,000 nodes, 35 k ids 63 / 56 us, 42 k 63 / 74; 5000 nodes, 28 k 58
// / 49, 35 k 59 / 63; 20,000 nodes, 49 k 75 / 70; and ids drawn with a density of 1 / sqrt(id): 3000 nodes, 14 k 52
// / 42, 28 k 53 / 66; 1000 nodes, 7 k 51 / 30, 14 k 52 / 47, 28 k 53 / 61.  Where it still loses: a tenth of
// all ids the same one (10,000 nodes, 14 k ids 62 / 66; 1 M nodes, 49 k ids 85 / 123).
constexpr int kSmallShareShift = 17;

static bool small_batch(int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim, int32_t dtype) {
  const int64_t ids = num_pairs * (int64_t)(k + 2);
  return ids <= kSmallMaxEntries && ids * ids <= (num_nodes << kSmallShareShift) &&
         dim * (dtype == GS_F32 ? 4 : 2) <= kSmallMaxRowBytes;
}
static int64_t small_forward_blocks(int64_t num_pairs) {
  return ceil_div(ceil_div(num_pairs, kSmallChunkPairs), kSmallForwardThreads / kGroupLanes);
}

static SgnsPlan plan_small(void* ws, int64_t num_pairs, int32_t k, int32_t dim, int32_t dtype) {
  Carver cv(ws);
  SgnsPlan p = {};
  const size_t b = (size_t)(num_pairs > 0 ? num_pairs : 1);
  p.small = true;
  p.loss_partials = cv.take<double>((size_t)small_forward_blocks((int64_t)b));
  p.g = cv.take<float>(b * (size_t)(k + 1));
  p.stage_center = cv.take<int32_t>(b);
  p.stage_delta = cv.take<float>(b * (size_t)dim);
  p.snap = cv.take<char>(b * (size_t)dim * (dtype == GS_F32 ? 4 : 2));
  p.pair_slot = cv.take<int32_t>(b);
  p.bytes = cv.used;
  return p;
}

// The plan of a step in a workspace of ws_bytes, of which the call's own arrays take `extra` bytes
// behind the plan; false: too small.  Every call needs room for the counters' plan, whatever its
// batch takes; with more room, the two-launch step where the batch is small (two_launches: the call can take
// it) and records where it is large, grouped or, where there is less room, sorted (sort_records: the call can take those).
static bool plan_step(SgnsPlan& p, void* ws, size_t ws_bytes, size_t extra, int64_t num_pairs, int64_t num_nodes,
                      int32_t k, int32_t dim, int32_t dtype, bool two_launches = true, bool force_compact = false,
                      bool sort_records = true) {
  const SgnsPlan counters = plan_sgns(ws, num_pairs, num_nodes, k, dim, force_compact);
  if (counters.bytes + extra > ws_bytes) return false;
  if (two_launches && small_batch(num_pairs, num_nodes, k, dim, dtype)) {
    p = plan_small(ws, num_pairs, k, dim, dtype);
    if (p.bytes + extra <= ws_bytes) return true;
  }
  const bool sorted = sort_records && sorted_batch(num_pairs, num_nodes, k);
  if (grouped_batch(num_pairs, num_nodes, k) && !(sorted && group_crowded(num_pairs * (int64_t)(k + 1), num_nodes))) {
    p = plan_grouped(ws, num_pairs, num_nodes, k, dim);
    if (p.bytes + extra <= ws_bytes) return true;
  }
  if (sorted)
    for (const bool wide : {true, false}) {
      p = plan_sorted(ws, num_pairs, num_nodes, k, dim, wide);
      if (p.bytes + extra <= ws_bytes) return true;
    }
  p = counters;
  return true;
}
// The largest plan that a batch of num_pairs may take.
static size_t plan_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim, int32_t dtype, bool two_launches) {
  size_t bytes = plan_sgns(nullptr, num_pairs, num_nodes, k, dim).bytes;
  if (two_launches && small_batch(num_pairs, num_nodes, k, dim, dtype))
    bytes = std::max(bytes, plan_small(nullptr, num_pairs, k, dim, dtype).bytes);
  const bool grouped = grouped_batch(num_pairs, num_nodes, k);
  if (grouped) bytes = std::max(bytes, plan_grouped(nullptr, num_pairs, num_nodes, k, dim).bytes);
  if ((!grouped || group_crowded(num_pairs * (int64_t)(k + 1), num_nodes)) && sorted_batch(num_pairs, num_nodes, k)) bytes = std::max(bytes, plan_sorted(nullptr, num_pairs, num_nodes, k, dim, true).bytes);
  return bytes;
}
// The same over all batches of up to num_pairs: the workspace of a program's largest batch serves every
// batch, on the way that it would take with a workspace of its own.  A plan grows with its batch but for a few
// borders behind which a smaller one follows.
static size_t step_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k, int32_t dim, int32_t dtype, bool two_launches = true) {
  size_t bytes = plan_bytes(num_pairs, num_nodes, k, dim, dtype, two_launches);
  int64_t power = 1;                                      // the largest power of two below the nodes
  while (2 * power < num_nodes) power *= 2;
  const int64_t small_ids = std::min(kSmallMaxEntries, (int64_t)std::sqrt((double)(num_nodes << kSmallShareShift)));
  const int64_t last[] = {(1 << 18) - 1, (1 << 20) - 1,   // before fewer, longer chunks and segments
                          (int64_t)((2 * (size_t)std::max(num_nodes, (int64_t)1) - 1) / kCompactFactor) / (k + 2),
                                                          // of those with counters for the batch's keys only
                          power / 2,                      // of those with a table of the input keys
                          small_ids / (k + 2)};           // of those with two launches
  for (const int64_t pairs : last)
    if (pairs > 0 && pairs < num_pairs) bytes = std::max(bytes, plan_bytes(pairs, num_nodes, k, dim, dtype, two_launches));
  for (int bits = kBucketRowBits; bits > 0; --bits)       // of grouped ones with more rows per bucket
    for (const int64_t pairs : {group_border(num_nodes, false, bits) / (k + 1), group_border(num_nodes, true, bits)})
      if (pairs < num_pairs && grouped_batch(pairs, num_nodes, k)) bytes = std::max(bytes, plan_bytes(pairs, num_nodes, k, dim, dtype, two_launches));
  return bytes;
}

// the two update passes (context-table keys, then input-table keys) in the piece layout that
// fits the row: 64 lanes x WPP words x PPL pieces cover the row, UB source rows in flight
template <typename T, int WPP, int PPL, int UB, int kOpt>
static int32_t launch_updates(const SgnsArgs& a, hipStream_t stream) {
  constexpr int kWaves = kSgnsThreads / 64;
  // context-table keys: exactly num_terms positions; input-table keys: at most one per pair
  const unsigned out_blocks = (unsigned)ceil_div(ceil_div(a.num_terms, a.slice_terms), kWaves);
  const unsigned in_blocks = (unsigned)std::min((int64_t)kStageMaxBlocks, ceil_div(ceil_div(a.num_pairs, kStageSlice), kWaves));
  const size_t lds = 0;
  const unsigned finish_blocks = (unsigned)ceil_div(a.long_slots, kGroupsPerBlock) + 1;
  sgns_update_kernel<T, WPP, PPL, UB, kOpt, false><<<out_blocks, kSgnsThreads, lds, stream>>>(a);
  if constexpr (kOpt == kPlain)
    if (a.snap != nullptr) sgns_finish_kernel<T, kOpt><<<finish_blocks, kSgnsThreads, 0, stream>>>(a, 1);   // one table
  sgns_update_kernel<T, WPP, PPL, UB, kOpt, true><<<in_blocks, kSgnsThreads, lds, stream>>>(a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename T, int VPL, int RB>
static int32_t launch_small(const SgnsArgs& a, hipStream_t stream) {
  const size_t idx_lds = (size_t)(kSmallForwardThreads / kGroupLanes) * a.chunk_pairs * (a.k + 2) * sizeof(int32_t);
  sgns_forward_kernel<T, VPL, RB, kInLds, kSmallForwardThreads>
      <<<(unsigned)(a.forward_blocks_per_xcd * 8), kSmallForwardThreads, idx_lds, stream>>>(a);
  GS_LAUNCH_CHECK();
  const int row_bytes = a.dim * (int)sizeof(T);            // one block more adds up the loss
  if (row_bytes <= 256) sgns_small_update_kernel<T, 1, 8><<<kSmallBlocks + 1, kSmallThreads, 0, stream>>>(a);
  else if (row_bytes <= 512) sgns_small_update_kernel<T, 2, 8><<<kSmallBlocks + 1, kSmallThreads, 0, stream>>>(a);
  else sgns_small_update_kernel<T, 4, 4><<<kSmallBlocks + 1, kSmallThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename T, int kOpt>
static int32_t launch_dense_rest(const SgnsArgs& a, bool any_named, hipStream_t stream);

// everything behind the place kernel
template <typename T, int kOpt>
static int32_t launch_rows(const SgnsArgs& a, hipStream_t stream) {
  const int row_bytes = a.dim * (int)sizeof(T);
  int32_t rc;
  if (row_bytes <= 256) rc = launch_updates<T, 1, 1, 16, kOpt>(a, stream);
  else if (row_bytes <= 512) rc = launch_updates<T, 2, 1, 16, kOpt>(a, stream);
  else if (row_bytes <= 1024) rc = launch_updates<T, 4, 1, 8, kOpt>(a, stream);
  else if (row_bytes <= 2048) rc = launch_updates<T, 4, 2, 4, kOpt>(a, stream);
  else rc = launch_updates<T, 4, 4, 2, kOpt>(a, stream);
  if (rc != GS_OK) return rc;
  // long rows (of both tables, unless the context-table ones are done); one more block sums the loss
  const unsigned finish_blocks = (unsigned)ceil_div(a.long_slots, kGroupsPerBlock) + 1;
  sgns_finish_kernel<T, kOpt><<<finish_blocks, kSgnsThreads, 0, stream>>>(a, a.snap != nullptr ? 2 : 0);
  GS_LAUNCH_CHECK();
  if constexpr (kOpt != kPlain) return launch_dense_rest<T, kOpt>(a, true, stream);
  return GS_OK;
}

// counters 0, key tables empty
static int32_t launch_clear(const SgnsArgs& a, hipStream_t stream) {
  const int64_t keys4 = ceil_div(a.cnt_last + 1, 4);
  const int64_t table4 = a.table_places / 4;   // (tables have at least 256 places each)
  sgns_clear_kernel<<<(unsigned)ceil_div(std::max(keys4, table4), 256), 256, 0, stream>>>(
      (uint4*)a.cnt, keys4, (uint4*)a.key_table, table4, a.bad_ids);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

// counters to offsets
static int32_t launch_scan(const SgnsArgs& a, hipStream_t stream) {
  const int64_t keys1 = a.cnt_last + 1;
  const int64_t tiles = ceil_div(keys1, kScanTile);
  if (keys1 <= kScanSmallMax) {
    scan_small_kernel<<<1, 1024, 0, stream>>>(a.cnt, keys1);
    GS_LAUNCH_CHECK();
  } else {
    scan_reduce_kernel<<<(unsigned)tiles, kScanThreads, 0, stream>>>(a.cnt, keys1, a.tile_sums);
    GS_LAUNCH_CHECK();
    const int raw_sums = tiles <= kFewTiles ? 1 : 0;
    if (!raw_sums) {
      scan_tiles_kernel<<<1, 1024, 0, stream>>>(a.tile_sums, tiles);
      GS_LAUNCH_CHECK();
    }
    scan_apply_kernel<<<(unsigned)tiles, kScanThreads, 0, stream>>>(a.cnt, keys1, a.tile_sums, raw_sums);
    GS_LAUNCH_CHECK();
  }
  return GS_OK;
}

// everything behind the sort but the long input-table rows: the context-table keys from the records, their
// long rows before and after, then the input-table keys
template <typename T, int WPP, int PPL, int UB>
static int32_t launch_sorted_updates(const SgnsArgs& a, uint2* further, hipStream_t stream) {
  constexpr int kWaves = kSgnsThreads / 64;
  const unsigned out_blocks = (unsigned)ceil_div(ceil_div(a.num_terms, a.slice_terms), kWaves);
  const unsigned in_blocks = (unsigned)std::min((int64_t)kStageMaxBlocks, ceil_div(ceil_div(a.num_pairs, kStageSlice), kWaves));
  const unsigned long_blocks = (unsigned)ceil_div(a.stage_long_base + 1, kGroupsPerBlock);
  sgns_sorted_long_kernel<T, true><<<long_blocks, kSgnsThreads, 0, stream>>>(a, further);
  sgns_sorted_update_kernel<T, WPP, PPL, UB, kPlain, false><<<out_blocks, kSgnsThreads, 0, stream>>>(a, further);
  sgns_sorted_long_kernel<T, false><<<long_blocks, kSgnsThreads, 0, stream>>>(a, nullptr);
  sgns_update_kernel<T, WPP, PPL, UB, kPlain, true><<<in_blocks, kSgnsThreads, 0, stream>>>(a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

// The kernel waits for rows, and waves are what covers that: where a few registers less make one more wave per SIMD, batches that
// fill the chip take them.  Steps of 60,000 pairs, 256 fp32 columns 190 -> 179 us (131 registers before), 100,000 pairs, 400 bf16
// columns 450 -> 393 us (175), 300,000, 200 fp16 columns 650 -> 630, 1 M, 256 bf16 columns 2559 -> 2440; 7712 pairs, 196 fp32 columns
// (482 waves) 101 -> 103.5, so not there; 384 and 512 fp32 columns with 3 instead of 2 waves 248 -> 263 and 277 -> 289, up to 128
// with 5 instead of 4 208 -> 217, so neither there.  With 16-bit tables that holds for every batch from there on; with fp32 tables,
// where the kernel with fewer registers is 2 to 5 % slower by itself, where the waves are up to twice the chip's and come in fewer turns: 256
// columns, 1 M nodes, 52,000 pairs (1 turn instead of 2) 192 -> 183 us, 100,000 (2 instead of 3) 315 -> 308, but 72,000 (2 and 2)
// 238 -> 251, 200,000 (4 instead of 5) 548 -> 557; 10,000 nodes 152 -> 144, 230 -> 224, 178 -> 188, 352 -> 357.
template <typename T, int VPL, int RB, int kGroup>
static void launch_forward(const SgnsArgs& a, hipStream_t stream) {
  constexpr int kMore = VPL == 4 ? 4 : (VPL == 8 && sizeof(T) == 2 ? 3 : 0);
  const unsigned blocks = (unsigned)(a.forward_blocks_per_xcd * 8);
  const size_t idx_lds = (size_t)kGroupsPerBlock * a.chunk_pairs * (a.k + 2) * sizeof(int32_t);
  constexpr int64_t kSimds = 1024;
  const int64_t waves = a.forward_blocks * (kSgnsThreads / 64);
  bool more = kMore != 0 && waves > (kMore - 1) * kSimds;
  if constexpr (kMore != 0 && sizeof(T) == 4)
    more = waves <= 2 * kMore * kSimds && ceil_div(waves, kMore * kSimds) < ceil_div(waves, (kMore - 1) * kSimds);
  if (more)
    sgns_forward_kernel<T, VPL, RB, kGroup, kSgnsThreads, kMore><<<blocks, kSgnsThreads, idx_lds, stream>>>(a);
  else
    sgns_forward_kernel<T, VPL, RB, kGroup, kSgnsThreads><<<blocks, kSgnsThreads, idx_lds, stream>>>(a);
}

template <typename T, int VPL, int RB>
static int32_t launch_sorted(const SgnsArgs& unsorted, const SgnsPlan& p, hipStream_t stream) {
  SgnsArgs a = unsorted;
  const int bits = bits_for_rows(a.num_nodes);
  const SortPlan sort = radix_sort_plan(a.num_terms, bits, p.sort_bytes);
  const int made = sort.passes & 1;                          // the passes end in buffer 0
  a.term_key = p.term_key[made];
  a.term_src = p.term_src[made];
  int32_t rc = launch_clear(a, stream);
  if (rc != GS_OK) return rc;
  launch_forward<T, VPL, RB, kBySort>(a, stream);
  GS_LAUNCH_CHECK();
  rc = launch_scan(a, stream);
  if (rc != GS_OK) return rc;
  sgns_place_kernel<<<(unsigned)ceil_div(a.num_pairs, 256), 256, 0, stream>>>(a, a.num_terms);
  GS_LAUNCH_CHECK();
  rc = radix_sort(sort, a.term_key, a.term_src, p.term_key[0], p.term_src[0], p.term_key[1], p.term_src[1], a.num_terms,
                  ~0u, bits, p.sort_scratch, stream);
  if (rc != GS_OK) return rc;
  a.term_key = p.term_key[0];
  a.term_src = p.term_src[0];
  uint2* further = static_cast<uint2*>(p.sort_scratch);
  const int row_bytes = a.dim * (int)sizeof(T);
  if (row_bytes <= 256) rc = launch_sorted_updates<T, 1, 1, 16>(a, further, stream);
  else if (row_bytes <= 512) rc = launch_sorted_updates<T, 2, 1, 16>(a, further, stream);
  else if (row_bytes <= 1024) rc = launch_sorted_updates<T, 4, 1, 8>(a, further, stream);
  else if (row_bytes <= 2048) rc = launch_sorted_updates<T, 4, 2, 4>(a, further, stream);
  else rc = launch_sorted_updates<T, 4, 4, 2>(a, further, stream);
  if (rc != GS_OK) return rc;
  // long rows of the input table; one more block sums the loss
  sgns_finish_kernel<T, kPlain><<<(unsigned)ceil_div(a.long_slots, kGroupsPerBlock) + 1, kSgnsThreads, 0, stream>>>(a, 2);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename T, int WPP, int PPL, int UB, int kOpt>
static int32_t launch_grouped_updates(const SgnsArgs& a, const uint2* further, hipStream_t stream) {
  constexpr int kWaves = kSgnsThreads / 64;
  const unsigned out_blocks = (unsigned)ceil_div(ceil_div(a.num_terms, a.slice_terms), kWaves);
  const unsigned in_blocks = (unsigned)std::min((int64_t)kStageMaxBlocks, ceil_div(ceil_div(a.num_pairs, kStageSlice), kWaves));
  const unsigned long_blocks = (unsigned)std::min((int64_t)kLongRowBlocks, ceil_div(a.long_slots, kGroupsPerBlock)) + 1;
  sgns_sorted_update_kernel<T, WPP, PPL, UB, kOpt, false><<<out_blocks, kSgnsThreads, 0, stream>>>(a, further);
  const bool one_table = a.dst_in == a.dst_out;
  if constexpr (kOpt == kPlain)
    if (one_table) sgns_long_rows_kernel<T, kOpt><<<long_blocks, kSgnsThreads, 0, stream>>>(a, 1);
  sgns_sorted_update_kernel<T, WPP, PPL, UB, kOpt, true><<<in_blocks, kSgnsThreads, 0, stream>>>(a, further);
  sgns_long_rows_kernel<T, kOpt><<<long_blocks, kSgnsThreads, 0, stream>>>(a, one_table ? 2 : 0);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename T, int kOpt>
static int32_t launch_grouped_rows(const SgnsArgs& a, const uint2* further, hipStream_t stream) {
  const int row_bytes = a.dim * (int)sizeof(T);
  int32_t rc;
  if (row_bytes <= 256) rc = launch_grouped_updates<T, 1, 1, 16, kOpt>(a, further, stream);
  else if (row_bytes <= 512) rc = launch_grouped_updates<T, 2, 1, 16, kOpt>(a, further, stream);
  else if (row_bytes <= 1024) rc = launch_grouped_updates<T, 4, 1, 8, kOpt>(a, further, stream);
  else if (row_bytes <= 2048) rc = launch_grouped_updates<T, 4, 2, 4, kOpt>(a, further, stream);
  else rc = launch_grouped_updates<T, 4, 4, 2, kOpt>(a, further, stream);
  if (rc != GS_OK) return rc;
  if constexpr (kOpt != kPlain) return launch_dense_rest<T, kOpt>(a, true, stream);
  return GS_OK;
}

template <typename T, int VPL, int RB>
static int32_t launch_grouped(const SgnsArgs& ungrouped, const SgnsPlan& p, int opt, hipStream_t stream) {
  SgnsArgs a = ungrouped;
  a.term_key = p.term_key[0];
  a.term_src = p.term_src[0];
  launch_forward<T, VPL, RB, kGrouped>(a, stream);
  GS_LAUNCH_CHECK();
  GroupArgs g = p.group;
  g.rows = g.keys_out = p.term_key[0];
  g.vals = g.vals_out = p.term_src[0];
  g.n = a.num_terms;
  g.second = a.stage_center;
  g.second_n = a.num_pairs;
  const float coef = -a.lr;
  std::memcpy(&g.second_word, &coef, sizeof(coef));
  g.second_key = (uint32_t)a.num_nodes;
  g.rows_mid = p.term_key[1];
  g.vals_mid = p.term_src[1];
  g.seg_shift = a.seg_shift;
  g.dim = a.dim;
  g.long_acc = a.long_acc;
  if (opt == kPlain) g.named = nullptr;
  const int32_t rc = group_rows(g, a.num_nodes, stream);
  if (rc != GS_OK) return rc;
  a.num_records = g.counters + kGroupRecords;
  a.num_long_rows = g.counters + kGroupLong;
  a.long_rows = g.long_rows;
  a.named = g.named;
  a.named_in = g.second_named;
  if (opt == kMomentum) return launch_grouped_rows<T, kMomentum>(a, g.further, stream);
  if constexpr (std::is_same<T, float>::value)
    if (opt == kAdam) return launch_grouped_rows<T, kAdam>(a, g.further, stream);
  return launch_grouped_rows<T, kPlain>(a, g.further, stream);
}

template <typename T, int VPL, int RB>
static int32_t launch_sgns(const SgnsArgs& a, const SgnsPlan& p, int opt, hipStream_t stream) {
  if (p.small) {
    // (row_bytes <= kSmallMaxRowBytes)
    if constexpr (VPL * 64 * sizeof(T) <= (size_t)kSmallMaxRowBytes) return launch_small<T, VPL, RB>(a, stream);
    return GS_EINVAL;
  }
  if (p.grouped) return launch_grouped<T, VPL, RB>(a, p, opt, stream);
  if (p.by_sort) return launch_sorted<T, VPL, RB>(a, p, stream);
  int32_t rc = launch_clear(a, stream);
  if (rc != GS_OK) return rc;
  launch_forward<T, VPL, RB, kByCounter>(a, stream);
  GS_LAUNCH_CHECK();
  rc = launch_scan(a, stream);
  if (rc != GS_OK) return rc;
  sgns_place_kernel<<<(unsigned)ceil_div(a.num_terms + a.num_pairs, 256), 256, 0, stream>>>(a, 0);
  GS_LAUNCH_CHECK();
  if (opt == kMomentum) return launch_rows<T, kMomentum>(a, stream);
  if constexpr (std::is_same<T, float>::value)
    if (opt == kAdam) return launch_rows<T, kAdam>(a, stream);
  return launch_rows<T, kPlain>(a, stream);
}

__global__ void zero_double_kernel(double* p) { *p = 0.0; }

// ---- dense passes of the momentum step (16 bytes per lane, grid-stride) ----------------
// momentum <- mu * momentum over a whole table ("mult" of GraphScale Sec. 3.2)
__global__ __launch_bounds__(256) void table_scale_kernel(float4* __restrict__ m, int64_t n4, float mu) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x) {
    float4 x = m[i];
    x.x *= mu; x.y *= mu; x.z *= mu; x.w *= mu;
    m[i] = x;
  }
}
template <typename T>
__global__ __launch_bounds__(256) void table_scale16_kernel(uint4* __restrict__ m, int64_t n8, float mu) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n8;
       i += (int64_t)gridDim.x * blockDim.x) {
    uint4 x = m[i];
    x.x = pack16<T>(T::lo(x.x) * mu, T::hi(x.x) * mu);
    x.y = pack16<T>(T::lo(x.y) * mu, T::hi(x.y) * mu);
    x.z = pack16<T>(T::lo(x.z) * mu, T::hi(x.z) * mu);
    x.w = pack16<T>(T::lo(x.w) * mu, T::hi(x.w) * mu);
    m[i] = x;
  }
}
// model <- model - lr * momentum over a whole table ("mult_add")
__global__ __launch_bounds__(256) void table_axpy_kernel(float4* __restrict__ w,
                                                         const float4* __restrict__ m, int64_t n4,
                                                         float lr) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
       i += (int64_t)gridDim.x * blockDim.x) {
    float4 x = w[i];
    const float4 y = m[i];
    x.x -= lr * y.x; x.y -= lr * y.y; x.z -= lr * y.z; x.w -= lr * y.w;
    w[i] = x;
  }
}
template <typename T>
__global__ __launch_bounds__(256) void table_axpy16_kernel(uint4* __restrict__ w,
                                                           const uint4* __restrict__ m, int64_t n8,
                                                           float lr) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n8;
       i += (int64_t)gridDim.x * blockDim.x) {
    uint4 x = w[i];
    const uint4 y = m[i];
    x.x = pack16<T>(T::lo(x.x) - lr * T::lo(y.x), T::hi(x.x) - lr * T::hi(y.x));
    x.y = pack16<T>(T::lo(x.y) - lr * T::lo(y.y), T::hi(x.y) - lr * T::hi(y.y));
    x.z = pack16<T>(T::lo(x.z) - lr * T::lo(y.z), T::hi(x.z) - lr * T::hi(y.z));
    x.w = pack16<T>(T::lo(x.w) - lr * T::lo(y.w), T::hi(x.w) - lr * T::hi(y.w));
    w[i] = x;
  }
}

// Whether the batch named the row of `key`: its counter slot holds terms, or the key is in the table of
// the batch's keys.
__device__ __forceinline__ bool row_named(const SgnsArgs& a, uint32_t key) {
  if (a.named != nullptr) return a.named[key >= (uint32_t)a.num_nodes ? key - (uint32_t)a.num_nodes + a.named_in : key] != 0;
  const KeyRegion r = key_region(a, key);
  if (r.bits == 0) return a.cnt[r.slot_base + r.vertex] != a.cnt[r.slot_base + r.vertex + 1u];
  const uint32_t mask = (1u << r.bits) - 1u;
  uint32_t h = (key * 2654435761u) >> (32 - r.bits);
  for (uint32_t probes = 0; probes <= mask; ++probes) {
    const uint32_t seen = r.table[h];
    if (seen == key) return true;
    if (seen == kNoRow) return false;
    h = (h + 1u) & mask;
  }
  return false;
}

// The optimizer on the rows outside the batch (the update and finish kernels have done the others): one
// pass that reads and writes every table once, where decay, put and apply as passes of their own read
// the moments twice and write them twice.  Bound by memory: with 1 M rows of 128 fp32 columns and
// 262,144 pairs, the rest of both tables takes 0.57 ms (momentum) and 0.88 ms (Adam), 5.0 TB/s, against
// 0.99 and 1.74 ms for the separate passes; the update kernels take 0.04 and 0.06 ms more for the rows of
// the batch.  A row takes `pieces` lanes of 16 bytes; a lane has kDenseRows rows in flight, and a workgroup ends with
// them: 0.65 and 1.00 ms with four rows, a loop over the rest of the table and accesses that go through the caches
// (plain against uncached accesses, no rows left out: 5.5 and 6.1 TB/s).
// Tables that the 256 MB of cache in front of the memory hold together are still there when the next step reads them, so
// they go through the caches.  Where a workgroup's rows end inside its lanes (its first and last lines are then shared), that
// is better up to a quarter more.  Whole steps, us, with the former kernel / past the caches / through them: momentum, 20,000 pairs,
// 64 columns, 200 MB of tables 126 / 131 / 123, 290 MB 174 / 167 / 165, 310 MB 181 / 165 / 170, 400 MB 225 / 196 / 217; 16 columns, 200 MB 133 / 142 / 129;
// 100 columns, 240 MB 158 / 169 / 154, 290 MB 186 / 183 / 180, 340 MB 216 / 201 / 206; Adam, 1000 pairs, 128 columns, 60 MB 90 / 85 / 87, 200 MB 141
// / 141 / 136, 290 MB 184 / 172 / 175, 400 MB 242 / 214 / 235; 100 columns, 240 MB 159 / 180 / 154, 310 MB 203 / 207 / 196, 400 MB 248 / 242 / 240.
constexpr int kDenseRows = 2;
constexpr int64_t kDenseCached = (int64_t)256 << 20;          // bytes
constexpr int kDenseBlocks = 1 << 23;          // workgroups in one dimension of the launch
// kOnce: accesses to memory that no cache will be asked for again
typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));
template <bool kOnce>
__device__ __forceinline__ uint4 dense_load(const uint4* p) {
  if constexpr (!kOnce) return *p;
  const Vec4 v = __builtin_nontemporal_load(reinterpret_cast<const Vec4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <bool kOnce>
__device__ __forceinline__ void dense_store(uint4* p, const uint4& v) {
  if constexpr (kOnce) __builtin_nontemporal_store(Vec4{v.x, v.y, v.z, v.w}, reinterpret_cast<Vec4*>(p));
  else *p = v;
}
template <typename T, int kOpt, bool kOnce>
__global__ __launch_bounds__(256) void dense_rest_kernel(SgnsArgs a, int pieces, bool any_named) {
  const int rows_at_once = 256 / pieces;
  const int in_iter = (int)threadIdx.x / pieces, piece = (int)threadIdx.x - in_iter * pieces;
  if (in_iter >= rows_at_once) return;
  const bool input_table = blockIdx.y != 0;
  uint4* __restrict__ m_t = static_cast<uint4*>(input_table ? a.dst_in : a.dst_out);
  uint4* __restrict__ w_t = static_cast<uint4*>(input_table ? a.w_in : a.w_out);
  uint4* __restrict__ v_t = reinterpret_cast<uint4*>(input_table ? a.sq_in : a.sq_out);
  const int64_t block = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;
  const int64_t first = block * (rows_at_once * kDenseRows) + in_iter;
  bool mine[kDenseRows];
#pragma unroll
  for (int u = 0; u < kDenseRows; ++u) {
    const int64_t row = first + (int64_t)u * rows_at_once;
    mine[u] = row < a.num_nodes &&
              !(any_named && row_named(a, (uint32_t)row + (input_table ? (uint32_t)a.num_nodes : 0u)));
  }
  uint4 m[kDenseRows], w[kDenseRows], v[kOpt == kAdam ? kDenseRows : 1];
#pragma unroll
  for (int u = 0; u < kDenseRows; ++u) {
    if (!mine[u]) continue;
    const int64_t at = (first + (int64_t)u * rows_at_once) * pieces + piece;
    m[u] = dense_load<kOnce>(m_t + at);
    w[u] = dense_load<kOnce>(w_t + at);
    if constexpr (kOpt == kAdam) v[u] = dense_load<kOnce>(v_t + at);
  }
#pragma unroll
  for (int u = 0; u < kDenseRows; ++u) {
    if (!mine[u]) continue;
    const int64_t at = (first + (int64_t)u * rows_at_once) * pieces + piece;
    constexpr int kElems = 4 * Words<T>::kPerWord;
    const uint32_t mw[4] = {m[u].x, m[u].y, m[u].z, m[u].w}, ww[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
    float me[kElems], we[kElems];
#pragma unroll
    for (int i = 0; i < kElems; ++i) { me[i] = piece_elem<T, 4>(mw, i); we[i] = piece_elem<T, 4>(ww, i); }
    if constexpr (kOpt == kMomentum) {
#pragma unroll
      for (int i = 0; i < kElems; ++i) {
        me[i] = as_stored<T>(me[i] * a.opt.decay1);
        we[i] = we[i] - a.opt.lr * me[i];
      }
    } else {
      float ve[4] = {__uint_as_float(v[u].x), __uint_as_float(v[u].y), __uint_as_float(v[u].z), __uint_as_float(v[u].w)};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        me[i] *= a.opt.decay1;
        ve[i] *= a.opt.decay2;
        we[i] -= adam_move(me[i], ve[i], a.opt.lr, a.opt.root_c2, a.opt.eps);
      }
      dense_store<kOnce>(v_t + at, make_uint4(__float_as_uint(ve[0]), __float_as_uint(ve[1]), __float_as_uint(ve[2]), __float_as_uint(ve[3])));
    }
    uint32_t mo[4], wo[4];
    pack_piece<T, 4>(me, mo);
    pack_piece<T, 4>(we, wo);
    dense_store<kOnce>(m_t + at, make_uint4(mo[0], mo[1], mo[2], mo[3]));
    dense_store<kOnce>(w_t + at, make_uint4(wo[0], wo[1], wo[2], wo[3]));
  }
}

template <typename T, int kOpt>
static int32_t launch_dense_rest(const SgnsArgs& a, bool any_named, hipStream_t stream) {
  const int pieces = a.dim * (int)sizeof(T) / 16;
  const int64_t per_block = (int64_t)(256 / pieces) * kDenseRows;
  // (a dimension of a launch is below 2^32 lanes, which 2 rows of 129 pieces per workgroup leave within this card's memory)
  const int64_t blocks = ceil_div(a.num_nodes, per_block);
  const int64_t layers = std::max((int64_t)1, ceil_div(blocks, (int64_t)kDenseBlocks));
  const dim3 grid((unsigned)ceil_div(blocks, layers), 2, (unsigned)layers);
  const int64_t bytes = 2 * a.num_nodes * a.dim * (int64_t)sizeof(T) * (kOpt == kAdam ? 3 : 2);
  if (bytes <= (256 % pieces == 0 ? kDenseCached : kDenseCached / 4 * 5)) dense_rest_kernel<T, kOpt, false><<<grid, 256, 0, stream>>>(a, pieces, any_named);
  else dense_rest_kernel<T, kOpt, true><<<grid, 256, 0, stream>>>(a, pieces, any_named);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

static int32_t check_sgns_args(const void* w_in, const void* w_out, int64_t num_nodes, int32_t dim,
                               int32_t dtype, const int32_t* centers, const int32_t* contexts,
                               const int32_t* negs, int64_t num_pairs, int32_t k,
                               const double* loss_sum_out, const void* ws, bool one_table = false) {
  if (!w_in || !w_out || num_nodes < 1 || num_nodes > (int64_t)INT32_MAX) return GS_EINVAL;
  if (dtype != GS_F32 && dtype != GS_BF16 && dtype != GS_F16) return GS_EINVAL;
  const int granule = (dtype == GS_F32) ? 4 : 8;   // elements per 16-byte piece
  if (dim < granule || dim > 1024 || (dim % granule) != 0) return GS_EINVAL;
  if (num_pairs < 0 || k < 0 || k > 60 || !loss_sum_out) return GS_EINVAL;
  if (num_pairs > 0 && (!centers || !contexts || (k > 0 && !negs))) return GS_EINVAL;
  if (num_pairs * (int64_t)(k + 1) > (int64_t)0x7fffffff) return GS_EOVERFLOW;
  if (!aligned(w_in, 16) || !aligned(w_out, 16)) return GS_EINVAL;
  if (w_in == w_out && !one_table) return GS_EINVAL;   // needs the one-table entry point
  if (!ws || !aligned(ws, 256)) return GS_EINVAL;
  return GS_OK;
}

// What the variants of the step add to the plain one.
struct SgnsExtras {
  int opt = kPlain;                // the optimizer behind the update, its rates
  OptRates rates = {};
  float* sq_in = nullptr;          // Adam: second-moment tables
  float* sq_out = nullptr;
  const gs_alias* noise = nullptr; // negatives drawn inside the step (negs_draw != null)
  uint64_t neg_seed = 0, neg_pair_base = 0;
  int32_t* negs_draw = nullptr;
  void* snap = nullptr;            // one table on both sides: copies of the input rows, pair slots
  int32_t* pair_slot = nullptr;
  const int32_t* walks = nullptr;  // pairs made inside the step
  const int64_t* pair_offsets = nullptr;
  int64_t num_walks = 0, first_pair = 0;
  int32_t walk_len = 0, window = 0;
  int32_t* gen_centers = nullptr;
  int32_t* gen_contexts = nullptr;
};

// Logits from (w_in, w_out); every touched row r of the destination tables becomes
// round(dst[r] - lr * gradient_r).  Plain SGD: destination = the tables themselves.
static int32_t run_sgns(void* w_in, void* w_out, void* dst_in, void* dst_out, int64_t num_nodes,
                        int32_t dim, int32_t dtype, const int32_t* centers, const int32_t* contexts,
                        const int32_t* negs, int64_t num_pairs, int32_t k, float lr,
                        double* loss_sum_out, const SgnsPlan& p, hipStream_t stream,
                        const SgnsExtras& x = SgnsExtras()) {
  SgnsArgs a;
  a.sq_in = x.sq_in;
  a.sq_out = x.sq_out;
  a.opt = x.rates;
  a.draw_negs = x.negs_draw != nullptr ? 1 : 0;
  const bool weighted = x.noise != nullptr && x.noise->prob != nullptr;
  a.noise_prob = weighted ? x.noise->prob : nullptr;
  a.noise_alias = weighted ? x.noise->alias : nullptr;
  a.noise_packed = weighted ? reinterpret_cast<const uint2*>(x.noise->packed) : nullptr;
  a.neg_seed = x.neg_seed;
  a.neg_pair_base = x.neg_pair_base;
  a.negs_draw = x.negs_draw;
  if (a.draw_negs) negs = x.negs_draw;
  a.snap = p.small ? p.snap : x.snap;
  a.pair_slot = p.small ? p.pair_slot : x.pair_slot;
  a.walks = x.walks;
  a.pair_offsets = x.pair_offsets;
  a.num_walks = x.num_walks;
  a.first_pair = x.first_pair;
  a.walk_len = x.walk_len;
  a.window = x.window;
  a.gen_centers = x.gen_centers;
  a.gen_contexts = x.gen_contexts;
  if (a.walks != nullptr) {
    centers = x.gen_centers;
    contexts = x.gen_contexts;
  }
  a.w_in = w_in;
  a.w_out = w_out;
  a.dst_in = dst_in;
  a.dst_out = dst_out;
  a.centers = centers;
  a.contexts = contexts;
  a.negs = negs;
  a.num_pairs = num_pairs;
  a.num_nodes = num_nodes;
  a.num_terms = num_pairs * (int64_t)(k + 1);
  a.long_slots = p.long_slots;
  a.seg_shift = p.seg_shift;
  a.k = k;
  a.per_k1 = (65535u + (uint32_t)(k + 1)) / (uint32_t)(k + 1);
  a.dim = dim;
  a.lr = lr;
  a.g = p.g;
  a.rank = p.rank;
  a.cnt = p.cnt;
  a.cnt_last = p.cnt_last;
  a.key_table = p.key_table;
  a.table_places = p.table_places;
  a.out_bits = p.out_bits;
  a.in_bits = p.in_bits;
  a.in_base = p.in_base;
  a.tile_sums = p.tile_sums;
  a.bad_ids = p.bad_ids;
  a.sorted = p.sorted;
  a.stage_base = p.stage_base;
  a.stage_long_base = p.stage_long_base;
  a.term_key = nullptr;
  a.term_src = nullptr;
  a.num_records = nullptr;
  a.long_rows = nullptr;
  a.num_long_rows = nullptr;
  a.named = nullptr;
  a.named_in = 0;
  a.long_acc = p.long_acc;
  a.stage_center = p.stage_center;
  a.stage_rank = p.stage_rank;
  a.stage_delta = p.stage_delta;
  a.chunk_pairs = p.small ? kSmallChunkPairs : chunk_pairs_for(num_pairs);
  a.slice_terms = p.grouped ? grouped_slice_for(a.num_terms) : (p.by_sort ? sorted_slice_for(a.num_terms) : slice_terms_for(num_pairs));
  a.loss_partials = p.loss_partials;
  a.forward_blocks = p.small ? small_forward_blocks(num_pairs) : forward_blocks_for(num_pairs);
  a.forward_blocks_per_xcd = ceil_div(a.forward_blocks, 8);
  a.loss_out = loss_sum_out;
  // float4 registers per lane for one row: 16 lanes x 4 floats = 64 elements each
  const int vpl = (dim + 63) / 64;
  if (dtype == GS_F32) {
    if (vpl <= 1) return launch_sgns<float, 1, 6>(a, p, x.opt, stream);
    if (vpl <= 2) return launch_sgns<float, 2, 6>(a, p, x.opt, stream);
    if (vpl <= 4) return launch_sgns<float, 4, 3>(a, p, x.opt, stream);
    if (vpl <= 8) return launch_sgns<float, 8, 2>(a, p, x.opt, stream);
    return launch_sgns<float, 16, 1>(a, p, x.opt, stream);
  }
  // 16-bit rows: a 16-byte piece is 8 elements = two float4, so the register count is even.  With one negative, whose pairs have two terms, blocks of
  // two rows, since a block's reads are all made: 120,000 pairs on 1 M nodes, 400 and 512 bf16 columns 219 and 236 us with blocks of four (212
  // and 228 with a branch in front of every read), now 193 and 207; 200 fp16 and 256 bf16 columns with six 137 and 139 (136, 138), now 130 and 134;
  // 128 columns 110 (112) and 106: not worth the kernels.  With two negatives the blocks of four and six are no slower than the branches were.
  if (dtype == GS_BF16) {
    if (vpl <= 2) return launch_sgns<bf16_t, 2, 6>(a, p, x.opt, stream);
    if (vpl <= 4) return k <= 1 ? launch_sgns<bf16_t, 4, 2>(a, p, x.opt, stream) : launch_sgns<bf16_t, 4, 6>(a, p, x.opt, stream);
    if (vpl <= 8) return k <= 1 ? launch_sgns<bf16_t, 8, 2>(a, p, x.opt, stream) : launch_sgns<bf16_t, 8, 4>(a, p, x.opt, stream);
    return launch_sgns<bf16_t, 16, 2>(a, p, x.opt, stream);
  }
  if (vpl <= 2) return launch_sgns<f16_t, 2, 6>(a, p, x.opt, stream);
  if (vpl <= 4) return k <= 1 ? launch_sgns<f16_t, 4, 2>(a, p, x.opt, stream) : launch_sgns<f16_t, 4, 6>(a, p, x.opt, stream);
  if (vpl <= 8) return k <= 1 ? launch_sgns<f16_t, 8, 2>(a, p, x.opt, stream) : launch_sgns<f16_t, 8, 4>(a, p, x.opt, stream);
  return launch_sgns<f16_t, 16, 2>(a, p, x.opt, stream);
}

}  // namespace gs

using namespace gs;

extern "C" size_t gs_sgns_step_workspace_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k,
                                               int32_t dim, int32_t dtype) {
  if (num_pairs < 0 || num_nodes < 0 || k < 0 || dim < 1) return 0;
  return step_bytes(num_pairs, num_nodes, k, dim, dtype);
}

extern "C" int32_t gs_sgns_step(void* w_in, void* w_out, int64_t num_nodes, int32_t dim,
                                int32_t dtype, const int32_t* centers, const int32_t* contexts,
                                const int32_t* negs, int64_t num_pairs, int32_t k, float lr,
                                double* loss_sum_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, dtype, centers, contexts, negs,
                                      num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, 0, num_pairs, num_nodes, k, dim, dtype)) return GS_EWORKSPACE;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  return run_sgns(w_in, w_out, w_in, w_out, num_nodes, dim, dtype, centers, contexts, negs, num_pairs,
                  k, lr, loss_sum_out, p, stream);
}

// ---- the step for callers that cannot allocate ------------------------------------------
// Scratch memory of gs_sgns_step_static: one array per GPU, part of the loaded code object,
// held until the process ends.  Host code never uses the array's name as an address: the
// device address is asked for once per device (hipGetSymbolAddress, with that device
// current) and kept.
constexpr int64_t kStaticMaxPairs = 4096;
constexpr int64_t kStaticMaxTerms = 65536;
constexpr int32_t kStaticMaxDim = 256;
constexpr size_t kStaticScratchBytes = (size_t)12 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kStaticMaxDevices = 64;
static void* g_scratch_ptr[kStaticMaxDevices];   // device address of `scratch`, per device
static std::mutex g_scratch_mutex;

static int32_t static_scratch(void** out) {
  int dev = -1;
  GS_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kStaticMaxDevices) return GS_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    GS_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (ptr == nullptr) return GS_EHIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return GS_OK;
}

extern "C" int32_t gs_sgns_step_static(void* w_in, void* w_out, int64_t num_nodes, int32_t dim,
                                       int32_t dtype, const int32_t* centers, const int32_t* contexts,
                                       const int32_t* negs, int64_t num_pairs, int32_t k, float lr,
                                       double* loss_sum_out, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (num_pairs > kStaticMaxPairs || dim > kStaticMaxDim) return GS_EWORKSPACE;
  if (num_pairs > 0 && k >= 0 && num_pairs * (int64_t)(k + 1) > kStaticMaxTerms) return GS_EWORKSPACE;
  void* ws = nullptr;
  const int32_t got = static_scratch(&ws);
  if (got != GS_OK) return got;
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, dtype, centers, contexts, negs,
                                      num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  SgnsPlan p;
  if (!plan_step(p, ws, kStaticScratchBytes, 0, num_pairs, num_nodes, k, dim, dtype, true, true)) return GS_EWORKSPACE;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  return run_sgns(w_in, w_out, w_in, w_out, num_nodes, dim, dtype, centers, contexts, negs, num_pairs,
                  k, lr, loss_sum_out, p, stream);
}

// workspace of the fused call: the step's own, then the drawn negatives
static size_t fused_negs_bytes(int64_t num_pairs, int32_t k) {
  return align_up((size_t)(num_pairs > 0 ? num_pairs : 1) * (size_t)(k > 0 ? k : 1) * sizeof(int32_t));
}

extern "C" size_t gs_sgns_step_fused_workspace_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k,
                                                     int32_t dim, int32_t dtype) {
  if (num_pairs < 0 || num_nodes < 0 || k < 0 || dim < 1) return 0;
  return step_bytes(num_pairs, num_nodes, k, dim, dtype) + fused_negs_bytes(num_pairs, k);
}

extern "C" int32_t gs_sgns_step_fused(void* w_in, void* w_out, int64_t num_nodes, int32_t dim,
                                      int32_t dtype, const int32_t* centers, const int32_t* contexts,
                                      int64_t num_pairs, const gs_alias* noise,
                                      uint64_t pair_index_base, uint64_t neg_seed, int32_t k, float lr,
                                      double* loss_sum_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  // the negatives live in the workspace: hand the checker a non-null stand-in
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, dtype, centers, contexts,
                                      static_cast<const int32_t*>(ws), num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  if (noise != nullptr && noise->prob != nullptr && !noise->alias) return GS_EINVAL;
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, fused_negs_bytes(num_pairs, k), num_pairs, num_nodes, k, dim, dtype)) return GS_EWORKSPACE;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  int32_t* negs_ws = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + p.bytes);
  SgnsExtras x;
  x.noise = noise;
  x.neg_seed = neg_seed;
  x.neg_pair_base = pair_index_base;
  x.negs_draw = negs_ws;
  return run_sgns(w_in, w_out, w_in, w_out, num_nodes, dim, dtype, centers, contexts, nullptr,
                  num_pairs, k, lr, loss_sum_out, p, stream, x);
}

// workspace of the call that makes its pairs: the step's own, the drawn negatives, the derived ids
static size_t walk_ids_bytes(int64_t num_pairs) {
  return align_up((size_t)(num_pairs > 0 ? num_pairs : 1) * sizeof(int32_t));
}

extern "C" size_t gs_sgns_step_from_walks_workspace_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k,
                                                          int32_t dim, int32_t dtype) {
  if (num_pairs < 0 || num_nodes < 0 || k < 0 || dim < 1) return 0;
  return step_bytes(num_pairs, num_nodes, k, dim, dtype) + fused_negs_bytes(num_pairs, k) +
         2 * walk_ids_bytes(num_pairs);
}

extern "C" int32_t gs_sgns_step_from_walks(void* w_in, void* w_out, int64_t num_nodes, int32_t dim,
                                           int32_t dtype, const int32_t* walks, int64_t num_walks,
                                           int32_t walk_len, int32_t window, const int64_t* pair_offsets,
                                           int64_t first_pair, int64_t num_pairs, const gs_alias* noise,
                                           uint64_t pair_index_base, uint64_t neg_seed, int32_t k,
                                           float lr, double* loss_sum_out, void* ws, size_t ws_bytes,
                                           void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!walks || !pair_offsets || num_walks < 1 || walk_len < 1 || walk_len > 4096 || window < 1 ||
      first_pair < 0)
    return GS_EINVAL;
  // the ids live in the workspace: hand the checker non-null stand-ins
  const int32_t* stand_in = static_cast<const int32_t*>(ws);
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, dtype, stand_in, stand_in, stand_in,
                                      num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  if (noise != nullptr && noise->prob != nullptr && !noise->alias) return GS_EINVAL;
  const size_t negs_bytes = fused_negs_bytes(num_pairs, k), ids_bytes = walk_ids_bytes(num_pairs);
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, negs_bytes + 2 * ids_bytes, num_pairs, num_nodes, k, dim, dtype)) return GS_EWORKSPACE;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  char* extra = static_cast<char*>(ws) + p.bytes;
  SgnsExtras x;
  x.noise = noise;
  x.neg_seed = neg_seed;
  x.neg_pair_base = pair_index_base;
  x.negs_draw = reinterpret_cast<int32_t*>(extra);
  x.gen_centers = reinterpret_cast<int32_t*>(extra + negs_bytes);
  x.gen_contexts = reinterpret_cast<int32_t*>(extra + negs_bytes + ids_bytes);
  x.walks = walks;
  x.pair_offsets = pair_offsets;
  x.num_walks = num_walks;
  x.first_pair = first_pair;
  x.walk_len = walk_len;
  x.window = window;
  return run_sgns(w_in, w_out, w_in, w_out, num_nodes, dim, dtype, nullptr, nullptr, nullptr, num_pairs,
                  k, lr, loss_sum_out, p, stream, x);
}

// workspace of the one-table step: the step's own, the copies of the input rows, the pair slots
static size_t line1_snap_bytes(int64_t num_pairs, int32_t dim, int32_t dtype) {
  return align_up((size_t)(num_pairs > 0 ? num_pairs : 1) * (size_t)dim * (dtype == GS_F32 ? 4 : 2));
}
static size_t line1_slot_bytes(int64_t num_pairs) {
  return align_up((size_t)(num_pairs > 0 ? num_pairs : 1) * sizeof(int32_t));
}

extern "C" size_t gs_line1_step_workspace_bytes(int64_t num_pairs, int64_t num_nodes, int32_t k,
                                                int32_t dim, int32_t dtype) {
  if (num_pairs < 0 || num_nodes < 0 || k < 0 || dim < 1) return 0;
  return step_bytes(num_pairs, num_nodes, k, dim, dtype, false) + line1_snap_bytes(num_pairs, dim, dtype) +
         line1_slot_bytes(num_pairs);
}

extern "C" int32_t gs_line1_step(void* w, int64_t num_nodes, int32_t dim, int32_t dtype,
                                 const int32_t* sources, const int32_t* targets, const int32_t* negs,
                                 int64_t num_pairs, int32_t k, float lr, double* loss_sum_out,
                                 void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  const int32_t bad = check_sgns_args(w, w, num_nodes, dim, dtype, sources, targets, negs, num_pairs,
                                      k, loss_sum_out, ws, true);
  if (bad != GS_OK) return bad;
  const size_t snap_bytes = line1_snap_bytes(num_pairs, dim, dtype), own_bytes = snap_bytes + line1_slot_bytes(num_pairs);
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, own_bytes, num_pairs, num_nodes, k, dim, dtype, false)) return GS_EWORKSPACE;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  SgnsExtras x;
  x.snap = static_cast<char*>(ws) + p.bytes;
  x.pair_slot = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + p.bytes + snap_bytes);
  return run_sgns(w, w, w, w, num_nodes, dim, dtype, sources, targets, negs, num_pairs, k, lr,
                  loss_sum_out, p, stream, x);
}

// Small batches on small tables: the two-launch step between dense passes of their own; else the rows of
// the batch get the whole optimizer in the update and one pass does the rest.  The single pass moves two
// tables' worth of momentum less, 2 * table_bytes * 2 / 5 TB/s, and the step in front of it is up to 57
// us slower (82 against 25 us for 2048 pairs on 1 M nodes): even at about 70 MB per table.
constexpr int64_t kSeparatePassBytes = (int64_t)64 << 20;

extern "C" int32_t gs_sgns_momentum_step(void* w_in, void* w_out, void* m_in, void* m_out,
                                         int64_t num_nodes, int32_t dim, int32_t dtype,
                                         const int32_t* centers, const int32_t* contexts,
                                         const int32_t* negs, int64_t num_pairs, int32_t k, float lr,
                                         float mu, double* loss_sum_out, void* ws, size_t ws_bytes,
                                         void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, dtype, centers, contexts, negs,
                                      num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  if (!m_in || !m_out || !aligned(m_in, 16) || !aligned(m_out, 16)) return GS_EINVAL;
  if (m_in == w_in || m_in == w_out || m_out == w_in || m_out == w_out || m_in == m_out)
    return GS_EINVAL;
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, 0, num_pairs, num_nodes, k, dim, dtype)) return GS_EWORKSPACE;
  const int64_t table_bytes = num_nodes * (int64_t)dim * (dtype == GS_F32 ? 4 : 2);
  if (num_pairs > 0 && !(p.small && table_bytes <= kSeparatePassBytes)) {
    if (!plan_step(p, ws, ws_bytes, 0, num_pairs, num_nodes, k, dim, dtype, false, false, false)) return GS_EWORKSPACE;
    SgnsExtras x;
    x.opt = kMomentum;
    x.rates.decay1 = mu;
    x.rates.lr = lr;
    return run_sgns(w_in, w_out, m_in, m_out, num_nodes, dim, dtype, centers, contexts, negs, num_pairs, k, -1.0f,
                    loss_sum_out, p, stream, x);
  }
  const int per16 = (dtype == GS_F32) ? 4 : 8;
  const int64_t pieces = num_nodes * (int64_t)dim / per16;
  const unsigned blocks = (unsigned)std::min((int64_t)(256 * 64), ceil_div(pieces, 256));
  // mult: momentum <- mu * momentum, every row
  if (dtype == GS_F32) {
    table_scale_kernel<<<blocks, 256, 0, stream>>>((float4*)m_in, pieces, mu);
    table_scale_kernel<<<blocks, 256, 0, stream>>>((float4*)m_out, pieces, mu);
  } else if (dtype == GS_BF16) {
    table_scale16_kernel<bf16_t><<<blocks, 256, 0, stream>>>((uint4*)m_in, pieces, mu);
    table_scale16_kernel<bf16_t><<<blocks, 256, 0, stream>>>((uint4*)m_out, pieces, mu);
  } else {
    table_scale16_kernel<f16_t><<<blocks, 256, 0, stream>>>((uint4*)m_in, pieces, mu);
    table_scale16_kernel<f16_t><<<blocks, 256, 0, stream>>>((uint4*)m_out, pieces, mu);
  }
  GS_LAUNCH_CHECK();
  // put: momentum[rows of the batch] += gradient (the update machinery with step -1)
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
  } else {
    const int32_t rc = run_sgns(w_in, w_out, m_in, m_out, num_nodes, dim, dtype, centers, contexts,
                                negs, num_pairs, k, -1.0f, loss_sum_out, p, stream);
    if (rc != GS_OK) return rc;
  }
  // mult_add: model <- model - lr * momentum, every row
  if (dtype == GS_F32) {
    table_axpy_kernel<<<blocks, 256, 0, stream>>>((float4*)w_in, (const float4*)m_in, pieces, lr);
    table_axpy_kernel<<<blocks, 256, 0, stream>>>((float4*)w_out, (const float4*)m_out, pieces, lr);
  } else if (dtype == GS_BF16) {
    table_axpy16_kernel<bf16_t><<<blocks, 256, 0, stream>>>((uint4*)w_in, (const uint4*)m_in, pieces, lr);
    table_axpy16_kernel<bf16_t><<<blocks, 256, 0, stream>>>((uint4*)w_out, (const uint4*)m_out, pieces, lr);
  } else {
    table_axpy16_kernel<f16_t><<<blocks, 256, 0, stream>>>((uint4*)w_in, (const uint4*)m_in, pieces, lr);
    table_axpy16_kernel<f16_t><<<blocks, 256, 0, stream>>>((uint4*)w_out, (const uint4*)m_out, pieces, lr);
  }
  GS_LAUNCH_CHECK();
  return GS_OK;
}

extern "C" int32_t gs_sgns_adam_step(float* w_in, float* w_out, float* m_in, float* m_out, float* v_in,
                                     float* v_out, int64_t num_nodes, int32_t dim,
                                     const int32_t* centers, const int32_t* contexts,
                                     const int32_t* negs, int64_t num_pairs, int32_t k, float lr,
                                     float beta1, float beta2, float eps, int64_t t,
                                     double* loss_sum_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  const int32_t bad = check_sgns_args(w_in, w_out, num_nodes, dim, GS_F32, centers, contexts, negs,
                                      num_pairs, k, loss_sum_out, ws);
  if (bad != GS_OK) return bad;
  float* tables[6] = {w_in, w_out, m_in, m_out, v_in, v_out};
  for (int i = 0; i < 6; ++i) {
    if (!tables[i] || !aligned(tables[i], 16)) return GS_EINVAL;
    for (int j = 0; j < i; ++j)
      if (tables[i] == tables[j]) return GS_EINVAL;
  }
  if (t < 1 || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps >= 0.f))
    return GS_EINVAL;
  SgnsPlan p;
  if (!plan_step(p, ws, ws_bytes, 0, num_pairs, num_nodes, k, dim, GS_F32, false, false, false)) return GS_EWORKSPACE;
  SgnsExtras x;
  x.opt = kAdam;
  x.sq_in = v_in;
  x.sq_out = v_out;
  x.rates.decay1 = beta1;
  x.rates.decay2 = beta2;
  x.rates.c1 = 1.0f - beta1;
  x.rates.c2 = 1.0f - beta2;
  // w -= (lr / (1 - beta1^t)) * m / (sqrt(v) / sqrt(1 - beta2^t) + eps), every row
  x.rates.lr = (float)((double)lr / (1.0 - pow((double)beta1, (double)t)));
  x.rates.root_c2 = (float)sqrt(1.0 - pow((double)beta2, (double)t));
  x.rates.eps = eps;
  if (num_pairs == 0) {
    zero_double_kernel<<<1, 1, 0, stream>>>(loss_sum_out);
    GS_LAUNCH_CHECK();
    SgnsArgs a = {};
    a.w_in = w_in;
    a.w_out = w_out;
    a.dst_in = m_in;
    a.dst_out = m_out;
    a.sq_in = v_in;
    a.sq_out = v_out;
    a.opt = x.rates;
    a.num_nodes = num_nodes;
    a.dim = dim;
    return launch_dense_rest<float, kAdam>(a, false, stream);
  }
  return run_sgns(w_in, w_out, m_in, m_out, num_nodes, dim, GS_F32, centers, contexts, negs, num_pairs, k, -1.0f,
                  loss_sum_out, p, stream, x);
}
