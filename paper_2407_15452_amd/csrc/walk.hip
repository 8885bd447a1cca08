// gs_random_walk / gs_node2vec_walk (GraphScale Sec. 2.2: DeepWalk-style walks
// from every node and node2vec's biased second-order walk).
//
// One lane per walk.  Every transition is a chain of dependent random reads
// (row bounds -> neighbour -> for node2vec, the previous node's row), each of
// which costs a whole cache line from HBM, so throughput comes from many walks
// in flight and from touching few lines per step.  Output rows are staged in LDS
// in windows of kWin positions and written out as 64-byte row segments instead
// of one scattered 4-byte store per position.
#include "common.h"

namespace gs {

constexpr int kWalkThreads = 256;
constexpr int kWin = 16;          // positions staged per flush
constexpr int kWinPad = kWin + 1; // odd stride: conflict-free column writes
constexpr uint32_t kMaxAttempts = 1024;

struct WalkArgs {
  const void* offsets;
  const int32_t* nbrs;
  const float* prob;
  const int32_t* alias;
  const uint2* packed;      // optional interleaved (prob bits, alias)
  const int32_t* starts;
  int32_t* walks;
  int64_t num_nodes;
  int64_t num_entries;
  int64_t num_walks;
  uint64_t id_base;
  uint64_t seed;
  int32_t walk_len;
  float inv_p, inv_q, max_bias;
};

// Alias step of a weighted draw: keep slot j, or move to the slot's alias.
__device__ __forceinline__ int64_t alias_pick(const WalkArgs& a, int64_t at, int64_t j, uint32_t word) {
  if (a.packed != nullptr) {
    const uint2 e = a.packed[at];
    return (unit_float(word) < __uint_as_float(e.x)) ? j : (int64_t)(int32_t)e.y;
  }
  return (unit_float(word) < a.prob[at]) ? j : (int64_t)a.alias[at];
}

// slot in a row of n entries
__device__ __forceinline__ int64_t row_slot(const Block4& b, int64_t n) { return (int64_t)slot_of(b, (uint64_t)n); }
__device__ __forceinline__ int32_t row_slot(const Block4& b, int32_t n) { return (int32_t)slot_of32(b, (uint32_t)n); }

// both bounds of a row in one read
template <typename OffT>
struct __attribute__((packed, aligned(4))) OffsetPair { OffT lo, hi; };

// First-order walks: one lane per walk, one dependent pair of random reads per
// step (row bounds, then the neighbour).  The 64 walks of a wave advance in
// lock step, so their positions are staged in LDS in windows of kWin and the
// wave writes them out together, 64 bytes per row segment.
template <typename OffT, bool kWeighted>
__global__ __launch_bounds__(kWalkThreads) void walk_kernel(WalkArgs a) {
  __shared__ int32_t tile[kWalkThreads / 64][64][kWinPad];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t wave_first = ((int64_t)blockIdx.x * (kWalkThreads / 64) + wave) * 64;
  const int64_t i = wave_first + lane;
  const bool live = i < a.num_walks;
  const uint64_t id = a.id_base + (uint64_t)i;
  const int32_t* __restrict__ nbrs = a.nbrs;
  const OffT* __restrict__ offsets = static_cast<const OffT*>(a.offsets);

  int32_t cur = -1;
  if (live) {
    cur = a.starts[i];
    if (cur < 0 || (int64_t)cur >= a.num_nodes) cur = -1;
  }

  for (int32_t t0 = 0; t0 < a.walk_len; t0 += kWin) {
    const int cols = min(kWin, a.walk_len - t0);
    for (int tt = 0; tt < cols; ++tt) {
      const int32_t t = t0 + tt;
      tile[wave][lane][tt] = cur;
      if (t + 1 >= a.walk_len) break;
      int32_t next = -1;
      if (cur >= 0) {
        const OffsetPair<OffT> row = *reinterpret_cast<const OffsetPair<OffT>*>(offsets + cur);
        // (does not depend on the row: computed while its bounds are under way; with that and the
        // bounds in one read, 300 walks of 40 nodes 22.4 -> 21.0 us, weighted 32.5 -> 29.8; a million
        // walks are bound by random cache lines and stay at 574 and 1050 us)
        const Block4 b = philox_at(a.seed, id, (uint32_t)t, 0u);
        const int64_t lo = (int64_t)row.lo, hi = (int64_t)row.hi;
        if (hi > lo) {
          int64_t j = row_slot(b, (OffT)(hi - lo));
          if (kWeighted) {
            j = alias_pick(a, lo + j, j, b.x2);
          }
          next = nbrs[lo + j];
          // a neighbour id that is not a node (a CSR not built by gs_csr_build) ends the walk
          if ((uint32_t)next >= (uint32_t)a.num_nodes) next = -1;
        }
      }
      cur = next;
    }
    wave_fence();                             // the tile is the wave's own
    // flush: 4 rows per pass, 16 lanes (64 bytes) per row
    const int c = lane & 15;
#pragma unroll 4
    for (int pass = 0; pass < 16; ++pass) {
      const int r = pass * 4 + (lane >> 4);
      const int64_t w = wave_first + r;
      if (w < a.num_walks && c < cols)
        a.walks[w * (int64_t)a.walk_len + t0 + c] = tile[wave][r][c];
    }
    wave_fence();
  }
}

// Second-order walks as a per-lane state machine with ONE memory access
// instruction per loop iteration.  A step of a walk is a chain of dependent random reads of
// very different length (row bounds; one candidate per attempt, 3.5 attempts on
// average at p=0.5, q=2; for a quarter of the attempts a search in the previous
// node's row).  Written as nested loops, a wave waits in every inner loop for
// its slowest lane and keeps about a third of its lanes busy.  Here every lane
// carries its own state (which read it needs next), each iteration issues that
// one read for all 64 lanes together, and the lane then moves to its next state;
// lanes never wait for each other except at the one load per iteration.
// The membership search in the previous node's row is an interpolation search (the ids of
// a row are spread evenly over [0, num_nodes), so x is expected where a straight line
// between the entries that bound the remaining range puts it; every third probe bisects
// instead, which bounds the search on rows that are not spread evenly).  A probe reads four
// neighbouring entries (one 16-byte access, the same cache line as a 4-byte one), and a
// probe whose entries lie on both sides of x ends the search at once.
// Each lane stages its own last kWin positions in LDS and writes them out as one
// 64-byte row segment when the window is full (or the walk is over).
struct __attribute__((packed, aligned(4))) Quad { int32_t v[4]; };   // four entries, 4-byte aligned
// kAhead: one read instruction per trip and random numbers drawn ahead, where that pays (reads_ahead()).
template <typename OffT, bool kWeighted, bool kAhead>
__global__ __launch_bounds__(kWalkThreads) void node2vec_kernel(WalkArgs a) {
  __shared__ int32_t tile[kWalkThreads / 64][64][kWinPad];
  using Pos = OffT;                         // positions in nbrs: below num_entries, which the offsets hold
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = ((int64_t)blockIdx.x * (kWalkThreads / 64) + wave) * 64 + lane;
  if (i >= a.num_walks) return;
  const uint64_t id = a.id_base + (uint64_t)i;
  const int32_t* __restrict__ nbrs = a.nbrs;
  const OffT* __restrict__ offsets = static_cast<const OffT*>(a.offsets);
  int32_t* __restrict__ out = a.walks + i * (int64_t)a.walk_len;
  int32_t* mine = tile[wave][lane];
  const int32_t last = a.walk_len - 1;      // index of the last position
  const float bias_lo = fminf(1.0f, a.inv_q), bias_hi = fmaxf(1.0f, a.inv_q);

  enum : int { kRow, kNewDraw, kAlias, kDraw, kSearch, kDone };
  enum : int { kNone, kCommit, kReject };
  const uint2* __restrict__ packed = a.packed;
  const Pos entries = (Pos)a.num_entries;
  const bool wide = a.num_entries >= 4;     // (a probe never reads past the array)
  int32_t cur = a.starts[i];
  if (cur < 0 || (int64_t)cur >= a.num_nodes) cur = -1;
  int32_t prev = -1;
  Pos prev_lo = 0, prev_hi = 0, lo = 0, hi = 0;
  int32_t t = 0;                            // position of cur
  uint32_t att = 0;
  int state = kRow;
  int decision = kNone;                     // what the last read decided: taken at the top of the loop
  int32_t next = -1;                        // the node a commit moves to
  mine[0] = cur;
  if (last == 0) { out[0] = cur; return; }

  // the attempt in flight
  Pos j = 0;                                // slot in the row of cur
  uint32_t word2 = 0;                       // alias uniform (weighted)
  float s = 0.f;                            // acceptance uniform * max_bias
  int32_t x = 0;                            // candidate
  // the membership search in flight: entries before L are < x, entries from H on are > x;
  // v_lo < x is the entry before L (or -1), v_hi > x the entry at H (or num_nodes)
  Pos L = 0, H = 0;
  int32_t v_lo = 0, v_hi = 0;
  int probes = 0;                           // probes made in this search
  Pos pos = 0;                              // what this iteration reads: nbrs[pos] (or the alias entry at pos)

  // kAhead: random numbers of the attempt after the one whose read is under way: the first of a step while
  // its row bounds arrive, the next one while a candidate arrives (three of four are rejected at
  // p = 0.5, q = 2); a membership search keeps those of its attempt's draw.  With 32-bit positions for
  // 32-bit offsets, 1.49 -> 1.31 ms for the 47,000 walks below.
  Block4 ahead = {0u, 0u, 0u, 0u};
  auto draw_ahead = [&]() {
    if (state == kRow || state == kDraw)
      ahead = philox_at(a.seed, id, (uint32_t)t, state == kRow ? 0u : att + 1u);
  };

  // position t + 1 of the walk is `node`: into the lane's window, and out when it is full
  auto put = [&](int32_t node) {
    ++t;
    const int col = t & (kWin - 1);
    mine[col] = node;
    if (col == kWin - 1 || t == last) {
      const int32_t first = t - col;
      for (int c = 0; c <= col; ++c) out[first + c] = mine[c];
    }
  };

  // Every stage below appears once, so a wave whose lanes are in different states runs each
  // of them once per trip: the decision of the last read (a step taken, or an attempt
  // rejected), the random numbers of a new attempt, the address of the next read, the read,
  // and what the value read means for the lane's state.
  while (true) {
    // ---- the decision of the last read ----------------------------------------------------
    if (decision == kCommit) {
      prev = cur; prev_lo = lo; prev_hi = hi;
      cur = next;
      att = 0;
      put(cur);
      state = (t == last) ? kDone : kRow;
    } else if (decision == kReject) {
      ++att;
      state = kNewDraw;
    }
    decision = kNone;
    if (state == kRow && cur < 0) {          // dead walk: -1 to the end
      while (t < last) put(-1);
      state = kDone;
    }
    if (state == kDone) break;

    // ---- arithmetic ahead of the read -----------------------------------------------------
    if (state == kNewDraw) {
      const Block4 b = kAhead ? ahead : philox_at(a.seed, id, (uint32_t)t, att);
      j = row_slot(b, (Pos)(hi - lo));
      word2 = b.x2;
      s = unit_float(b.x3) * a.max_bias;
      pos = lo + j;
      state = (kWeighted ? kAlias : kDraw);
    } else if (state == kSearch) {           // (the range [L, H) is never empty here)
      Pos p;
      if (probes % 3 == 2) {
        p = L + ((H - L) >> 1);
      } else {
        // (differences of ids and of -1 .. num_nodes, so below 2^32; a row that is not sorted may give anything)
        const float part = fminf(fmaxf((float)((uint32_t)x - (uint32_t)v_lo) / (float)((uint32_t)v_hi - (uint32_t)v_lo), 0.f), 1.f);
        p = L + (Pos)(part * (float)(H - L));
      }
      p = min(max(p, L), H - 1);
      // the four entries around p: an aligned group, or the array's last four
      pos = wide ? min((Pos)(p & ~(Pos)3), (Pos)(entries - 4)) : p;
    }

    // ---- the one read of this iteration ---------------------------------------------------
    // Whatever a lane needs next (two row bounds, an alias entry, a neighbour, four entries of prev's
    // row), it is part of 16 bytes of one array, so with kAhead all lanes read through one instruction
    // and a trip waits once; reads in branches of their own wait one after the other (47,000 walks of 80
    // nodes on a 4 M-node graph, bound by the chain of reads: 1.78 -> 1.49 ms).
    Pos r0 = 0, r1 = 0;
    int32_t v = 0;
    Quad quad = {{0, 0, 0, 0}};
    uint32_t e_prob = 0, e_alias = 0;
    if constexpr (kAhead) {
      const char* from;
      int skip = 0;                           // 32-bit words in front of what is wanted
      if (state == kRow) {
        if (sizeof(OffT) == 8) {
          from = reinterpret_cast<const char*>(offsets + cur);
        } else {                              // (the last rows' bounds are the tail of the last 16 bytes)
          const int32_t at = min(cur, (int32_t)(a.num_nodes - 3));
          skip = cur - at;
          from = reinterpret_cast<const char*>(offsets + at);
        }
      } else if (kWeighted && state == kAlias) {
        const Pos at = min(pos, (Pos)(entries - 2));
        skip = 2 * (int)(pos - at);
        from = reinterpret_cast<const char*>(packed + at);
      } else {                                // a probe's four entries; a neighbour among four that are aligned likewise
        const Pos at = state == kSearch ? pos : min((Pos)(pos & ~(Pos)3), (Pos)(entries - 4));
        skip = (int)(pos - at);
        from = reinterpret_cast<const char*>(nbrs + at);
      }
      quad = *reinterpret_cast<const Quad*>(from);
      draw_ahead();                           // (while the read is under way)
      const int32_t w0 = skip == 0 ? quad.v[0] : (skip == 1 ? quad.v[1] : (skip == 2 ? quad.v[2] : quad.v[3]));
      const int32_t w1 = skip == 0 ? quad.v[1] : (skip == 1 ? quad.v[2] : quad.v[3]);
      v = w0;
      e_prob = (uint32_t)w0;
      e_alias = (uint32_t)w1;
      if (sizeof(OffT) == 8) {
        r0 = (Pos)(((uint64_t)(uint32_t)quad.v[1] << 32) | (uint32_t)quad.v[0]);
        r1 = (Pos)(((uint64_t)(uint32_t)quad.v[3] << 32) | (uint32_t)quad.v[2]);
      } else {
        r0 = w0;
        r1 = w1;
      }
    } else if (state == kSearch) {
      if (wide) quad = *reinterpret_cast<const Quad*>(nbrs + pos);
      else quad.v[0] = nbrs[pos];
    } else if (state == kRow) {
      r0 = offsets[cur];
      r1 = offsets[(int64_t)cur + 1];
    } else if (kWeighted && state == kAlias) {
      if (packed != nullptr) { const uint2 e = packed[pos]; e_prob = e.x; e_alias = e.y; }
      else { e_prob = __float_as_uint(a.prob[pos]); e_alias = (uint32_t)a.alias[pos]; }
    } else {
      v = nbrs[pos];
    }

    // ---- consume it: new state, or a decision ----------------------------------------------
    bool known = false, member = false;      // membership of x in the row of prev has been settled
    switch (state) {
      case kRow:
        lo = r0; hi = r1;
        if (hi > lo) state = kNewDraw;
        else { decision = kCommit; next = -1; }                    // dead end
        break;
      case kAlias:
        if (!(unit_float(word2) < __uint_as_float(e_prob))) j = (Pos)(int32_t)e_alias;
        pos = lo + j;
        state = kDraw;
        break;
      case kDraw:
        x = v;
        next = x;
        // a neighbour id that is not a node (a CSR not built by gs_csr_build) ends the walk
        if ((uint32_t)x >= (uint32_t)a.num_nodes) { decision = kCommit; next = -1; break; }
        if (t == 0 || att == kMaxAttempts - 1) { decision = kCommit; break; }   // unbiased first step; last attempt is taken
        // accept iff s < bias(x).  For x != prev the bias is 1 or 1/q, so the
        // membership search is only needed when s falls between the two.
        if (x == prev) { decision = (s < a.inv_p) ? kCommit : kReject; break; }
        if (s < bias_lo) { decision = kCommit; break; }
        if (!(s < bias_hi)) { decision = kReject; break; }
        L = prev_lo; H = prev_hi;
        if (L >= H) { known = true; break; }                       // (prev has no row: cannot happen after a step)
        v_lo = -1;
        v_hi = (int32_t)a.num_nodes;
        probes = 0;
        state = kSearch;
        break;
      case kSearch: {
        // entries pos + i0 .. pos + i1 of the probe lie in the remaining range [L, H)
        const int width = wide ? 4 : 1;
        const int i0 = (int)(max(pos, L) - pos), i1 = (int)(min((Pos)(pos + width), H) - 1 - pos);
        bool found = false;
        int32_t first_v = 0, last_v = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          found = found || (q >= i0 && q <= i1 && quad.v[q] == x);
          if (q == i0) first_v = quad.v[q];
          if (q == i1) last_v = quad.v[q];
        }
        ++probes;
        if (found) { known = true; member = true; break; }
        if (x < first_v) { H = pos + i0; v_hi = first_v; }
        else if (x > last_v) { L = pos + i1 + 1; v_lo = last_v; }
        else known = true;                  // x lies between two neighbouring entries
        if (L >= H) known = true;
        break;
      }
      default:
        break;
    }
    if (known) decision = (s < (member ? 1.0f : a.inv_q)) ? kCommit : kReject;
  }
}

// One read instruction for all states and an attempt drawn ahead cost instructions on every trip and pay where a
// trip waits for memory: waves that are full but few (two per SIMD are 2^17 walks), attempts that are rejected, rows
// beyond the caches; sooner with alias tables (a read more per attempt), later with 64-bit offsets (more
// arithmetic).  Times of reads in branches of their own over times of one read ahead, R-MAT graphs, walks of 20 to 80
// nodes, p = 0.5, q = 2 unless stated:
//   unweighted  47,000 walks: 128 M entries 1.26, 3.2 M 1.13, 1.6 M 1.08, 0.4 M 0.97; 1000 walks: 128 M 1.17, 6 M 0.97;
//               200,000 walks 0.91; 10 walks 0.91
//   64 bits     47,000 walks: 128 M 1.07, 8 M 1.04, 0.4 M 0.94; 10 walks 0.91
//   alias       47,000 walks: 128 M 1.47, 8 M 1.34, 0.4 M 1.14; 40 walks 1.05; 200,000 walks 0.90
//   both        47,000 walks: 128 M 1.17, 8 M 1.09, 0.8 M 1.07; 600 walks on 280 entries 0.96; 200 walks 0.98 to 1.07
// p = q = 1 (every candidate is taken) 0.78 to 0.97.  q = 1, p = 2: 47,000 walks on 128 M entries 1.18, 64 bits 0.97, alias
// table 1.50; 120,000 walks 0.95, alias table 1.15, on 280 entries 0.95.  q = 0.25, p = 4 on rows of 8 entries: 47,000
// walks 0.95, 3000 walks 1.17, both 0.95.
static bool reads_ahead(bool weighted, bool bits64, float p, float q, const WalkArgs& a) {
  // (every read is part of 16 bytes of one array; an alias table that is not interleaved takes two)
  if (a.num_entries < 4 || a.num_nodes < 3 || (weighted && a.packed == nullptr)) return false;
  if ((p == 1.0f && q == 1.0f) || a.num_walks > (int64_t)1 << 17) return false;
  if (q == 1.0f && a.num_walks > (int64_t)3 << 15 && (bits64 || !weighted)) return false;
  if (q < 1.0f && a.num_entries < 10 * a.num_nodes && (bits64 || a.num_walks > 4096)) return false;
  if (weighted && !bits64) return a.num_walks >= 32 && a.num_entries >= 4096;
  if (a.num_walks < 512) return false;
  if (weighted) return a.num_entries >= (int64_t)3 << 18;
  if (bits64) return q != 1.0f && a.num_entries >= (int64_t)1 << 23;
  return a.num_entries >= (a.num_walks >= (1 << 14) ? (int64_t)3 << 19 : (int64_t)1 << 22);
}

template <typename OffT>
static void launch_walk(bool weighted, bool second, float p, float q, const WalkArgs& a, hipStream_t stream) {
  const unsigned blocks = (unsigned)ceil_div(a.num_walks, kWalkThreads);
  if (second) {
    const bool ahead = reads_ahead(weighted, sizeof(OffT) == 8, p, q, a);
    auto kernel = weighted ? (ahead ? node2vec_kernel<OffT, true, true> : node2vec_kernel<OffT, true, false>)
                           : (ahead ? node2vec_kernel<OffT, false, true> : node2vec_kernel<OffT, false, false>);
    kernel<<<blocks, kWalkThreads, 0, stream>>>(a);
  } else {
    if (weighted) walk_kernel<OffT, true><<<blocks, kWalkThreads, 0, stream>>>(a);
    else walk_kernel<OffT, false><<<blocks, kWalkThreads, 0, stream>>>(a);
  }
}

static int32_t walk_common(const gs_csr* g, const gs_alias* al, const int32_t* starts,
                           int64_t num_walks, uint64_t id_base, int32_t walk_len, bool second,
                           float p, float q, uint64_t seed, int32_t* walks_out, hipStream_t stream) {
  if (!g || num_walks < 0 || walk_len < 1) return GS_EINVAL;
  if (g->num_nodes < 0 || g->num_nodes > (int64_t)INT32_MAX || g->num_entries < 0) return GS_EINVAL;
  if (g->offset_bits != 32 && g->offset_bits != 64) return GS_EINVAL;
  if (!g->offsets || (g->num_entries > 0 && !g->nbrs)) return GS_EINVAL;
  if (second && (!(p > 0.0f) || !(q > 0.0f))) return GS_EINVAL;
  if (num_walks > 0 && (!starts || !walks_out)) return GS_EINVAL;
  if (num_walks > ((int64_t)1 << 38)) return GS_EOVERFLOW;
  const bool weighted = al != nullptr && al->prob != nullptr;
  if (weighted && !al->alias) return GS_EINVAL;
  if (num_walks == 0) return GS_OK;
  WalkArgs a;
  a.offsets = g->offsets;
  a.nbrs = g->nbrs;
  a.prob = weighted ? al->prob : nullptr;
  a.alias = weighted ? al->alias : nullptr;
  a.packed = weighted ? reinterpret_cast<const uint2*>(al->packed) : nullptr;
  a.starts = starts;
  a.walks = walks_out;
  a.num_nodes = g->num_nodes;
  a.num_entries = g->num_entries;
  a.num_walks = num_walks;
  a.id_base = id_base;
  a.seed = seed;
  a.walk_len = walk_len;
  a.inv_p = 1.0f / p;
  a.inv_q = 1.0f / q;
  a.max_bias = fmaxf(a.inv_p, fmaxf(1.0f, a.inv_q));
  if (g->offset_bits == 64) launch_walk<int64_t>(weighted, second, p, q, a, stream);
  else launch_walk<int32_t>(weighted, second, p, q, a, stream);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

}  // namespace gs

extern "C" int32_t gs_random_walk(const gs_csr* g, const gs_alias* a, const int32_t* starts,
                                  int64_t num_walks, uint64_t walk_id_base, int32_t walk_len,
                                  uint64_t seed, int32_t* walks_out, void* stream) {
  return gs::walk_common(g, a, starts, num_walks, walk_id_base, walk_len, false, 1.0f, 1.0f, seed,
                         walks_out, (hipStream_t)stream);
}

extern "C" int32_t gs_node2vec_walk(const gs_csr* g, const gs_alias* a, const int32_t* starts,
                                    int64_t num_walks, uint64_t walk_id_base, int32_t walk_len,
                                    float p, float q, uint64_t seed, int32_t* walks_out,
                                    void* stream) {
  return gs::walk_common(g, a, starts, num_walks, walk_id_base, walk_len, true, p, q, seed,
                         walks_out, (hipStream_t)stream);
}
