// gs_random_walk / gs_node2vec_walk (GraphScale Sec. 2.2: DeepWalk-style walks
// from every node and node2vec's biased second-order walk).
//
// Every transition is a chain of dependent random reads
// (row bounds -> neighbour -> for node2vec, the previous node's row), each of
// which costs a whole cache line from HBM, so throughput comes from many walks
// in flight and from touching few lines per step; node2vec launches of few walks put several
// lanes to one.  Output rows are staged in LDS
// in windows of kWin positions and written out as 64-byte row segments instead
// of one scattered 4-byte store per position.
#include <type_traits>

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

typedef int32_t Quad __attribute__((ext_vector_type(4), aligned(4)));   // four entries, 4-byte aligned

// Second-order walks, a step of which is a chain of dependent random reads of very different length: the row's
// bounds, a candidate per attempt (3.7 attempts on average at p = 0.5, q = 2), for a quarter of the attempts a membership search
// in the previous node's row, and an alias entry before every candidate of a weighted graph.  Two kernels: a state machine with
// a lane per walk, for unweighted launches that fill the chip with walks of many attempts, and a team of lanes per walk; which
// and how many lanes: team_size() below.
//
// The membership search is an interpolation search (the ids of a row are spread evenly over [0, num_nodes), so x
// is expected where a straight line between the entries that bound the remaining range puts it; every
// third probe bisects instead, which bounds the search on rows that are not spread evenly).  A probe reads
// four neighbouring entries (one 16-byte access, the same cache line as a 4-byte one), and a probe whose
// entries lie on both sides of x ends the search at once.  The state of a search: entries before L are < x, entries from
// H on are > x; v_lo < x is the entry before L (or -1), v_hi > x the entry at H (or num_nodes).

// the first of the four entries to read next; [L, H) is not empty, and the array has at least four
template <typename Pos>
__device__ __forceinline__ Pos probe_at(int32_t x, Pos L, Pos H, int32_t v_lo, int32_t v_hi, bool bisect, Pos entries) {
  Pos p;
  if (bisect) {
    p = L + ((H - L) >> 1);
  } else {
    // (differences of ids and of -1 .. num_nodes, so below 2^32; a row that is not sorted may give anything.  Only a
    // guess, so the approximate reciprocal will do)
    const float part = (float)((uint32_t)x - (uint32_t)v_lo) * __builtin_amdgcn_rcpf((float)((uint32_t)v_hi - (uint32_t)v_lo));
    p = L + (Pos)(fminf(fmaxf(part, 0.f), 1.f) * (float)(H - L));
  }
  p = min(max(p, L), H - 1);
  return min((Pos)(p & ~(Pos)3), (Pos)(entries - 4));           // an aligned group, or the array's last four
}
// What the entries at pos say.  true: the search is over, and found says how
template <typename Pos>
__device__ __forceinline__ bool probe_says(int32_t x, Pos pos, Quad quad, Pos& L, Pos& H, int32_t& v_lo, int32_t& v_hi,
                                           bool& found) {
  // entries pos + i0 .. pos + i1 of the probe lie in the remaining range [L, H)
  const int i0 = (int)(max(pos, L) - pos), i1 = (int)(min((Pos)(pos + 4), H) - 1 - pos);
  int32_t first_v = 0, last_v = 0;
  bool hit = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    hit = hit | ((q >= i0) & (q <= i1) & (quad[q] == x));
    first_v = q == i0 ? quad[q] : first_v;
    last_v = q == i1 ? quad[q] : last_v;
  }
  found = hit;
  const bool left = x < first_v, right = x > last_v;            // (neither: x lies between two neighbouring entries)
  if (left) { H = pos + i0; v_hi = first_v; }
  else if (right) { L = pos + i1 + 1; v_lo = last_v; }
  return hit || !(left || right) || L >= H;
}

// A lane per walk (no alias tables), as a state machine with ONE read instruction per trip through the loop.  Written as
// nested loops, a wave waits in every inner loop for its slowest lane and keeps about a third of its lanes busy.  Here
// every lane carries its own state (which read it needs next), each trip issues that one read for all 64 lanes
// together, and the lane then moves to its next state; lanes never wait for each other except at the one read.
// Whatever a lane needs (two row bounds, a neighbour, four entries of prev's row), it is part of 16 bytes of one array, so
// all lanes read through one instruction and a trip waits once; the random numbers of the attempt that may come next are
// drawn while the read is under way.
// Each lane stages its own last kWin positions in LDS and writes them out as one
// 64-byte row segment when the window is full (or the walk is over).
// Needs at least four entries and three nodes.
template <typename OffT, typename Pos>
__global__ __launch_bounds__(kWalkThreads) void node2vec_kernel(WalkArgs a) {
  __shared__ int32_t tile[kWalkThreads][kWinPad];
  const int64_t i = (int64_t)blockIdx.x * kWalkThreads + threadIdx.x;
  if (i >= a.num_walks) return;
  const uint64_t id = a.id_base + (uint64_t)i;
  const int32_t* __restrict__ nbrs = a.nbrs;
  const OffT* __restrict__ offsets = static_cast<const OffT*>(a.offsets);
  int32_t* __restrict__ out = a.walks + i * (int64_t)a.walk_len;
  int32_t* mine = tile[threadIdx.x];
  const int32_t last = a.walk_len - 1;      // index of the last position
  const float bias_lo = fminf(1.0f, a.inv_q), bias_hi = fmaxf(1.0f, a.inv_q);
  const Pos entries = (Pos)a.num_entries;

  enum : int { kRow, kDraw, kSearch };
  int32_t cur = a.starts[i];
  if (cur < 0 || (int64_t)cur >= a.num_nodes) cur = -1;
  int32_t prev = -1;
  Pos prev_lo = 0, prev_hi = 0, lo = 0, hi = 0;
  int32_t t = 0;                            // position of cur
  uint32_t att = 0;
  int state = kRow;
  bool fresh = false;                       // a new attempt begins
  mine[0] = cur;
  if (last == 0) { out[0] = cur; return; }

  // the attempt in flight
  Block4 ahead = {0u, 0u, 0u, 0u};          // random numbers of the next one
  float s = 0.f;                            // acceptance uniform * max_bias
  int32_t x = 0;                            // candidate
  Pos L = 0, H = 0;                         // its membership search
  int32_t v_lo = 0, v_hi = 0;
  int turn = 0;                             // every third probe bisects
  Pos pos = 0;                              // what this trip reads: nbrs[pos]

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

  while (true) {
    if (state == kRow) {
      if (cur < 0)                          // dead walk: -1 to the end
        while (t < last) put(-1);
      if (t == last) break;
    }
    if (fresh) {
      s = unit_float(ahead.x3) * a.max_bias;
      pos = lo + row_slot(ahead, (Pos)(hi - lo));
      state = kDraw;
      fresh = false;
    }

    // ---- the one read of this trip --------------------------------------------------------
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
    } else {                                // a probe's four entries; a neighbour among four that are aligned likewise
      Pos at;
      if (state == kSearch) at = pos = probe_at(x, L, H, v_lo, v_hi, turn == 2, entries);
      else at = min((Pos)(pos & ~(Pos)3), (Pos)(entries - 4));
      skip = (int)(pos - at);
      from = reinterpret_cast<const char*>(nbrs + at);
    }
    const Quad quad = *reinterpret_cast<const Quad*>(from);
    // while it is under way: the first attempt of the next step, or the one after the one at hand
    if (state == kRow || state == kDraw)
      ahead = philox_at(a.seed, id, (uint32_t)t, state == kRow ? 0u : att + 1u);
    const int32_t w0 = skip == 0 ? quad[0] : (skip == 1 ? quad[1] : (skip == 2 ? quad[2] : quad[3]));
    const int32_t w1 = skip == 0 ? quad[1] : (skip == 1 ? quad[2] : quad[3]);

    // ---- what it means ----------------------------------------------------------------------
    bool taken = false;                     // the walk moves to x
    if (state == kRow) {
      if (sizeof(OffT) == 8) {
        lo = (Pos)(((uint64_t)(uint32_t)quad[1] << 32) | (uint32_t)quad[0]);
        hi = (Pos)(((uint64_t)(uint32_t)quad[3] << 32) | (uint32_t)quad[2]);
      } else {
        lo = w0;
        hi = w1;
      }
      att = 0;
      fresh = hi > lo;
      taken = !fresh;                       // dead end
      x = -1;
    } else {
      bool known = false, member = false;   // membership of x in the row of prev has been settled
      bool decided = true;
      if (state == kDraw) {
        x = w0;
        if ((uint32_t)x >= (uint32_t)a.num_nodes) {
          x = -1;                           // not a node (a CSR not built by gs_csr_build): ends the walk
          taken = true;
        } else if (t == 0 || att == kMaxAttempts - 1) {
          taken = true;                     // unbiased first step; the last attempt is taken
        } else if (x == prev) {
          taken = s < a.inv_p;
        } else if (s < bias_lo) {           // for x != prev the bias is 1 or 1/q: the search is only
          taken = true;                     // needed when s falls between the two
        } else if (s < bias_hi) {
          L = prev_lo; H = prev_hi;
          v_lo = -1; v_hi = (int32_t)a.num_nodes;
          known = L >= H;             // (prev has no row: cannot happen after a step)
          decided = known;
          state = kSearch;
          turn = 0;
        }
      } else {
        known = probe_says(x, pos, quad, L, H, v_lo, v_hi, member);
        decided = known;
        turn = turn == 2 ? 0 : turn + 1;
      }
      if (known) taken = s < (member ? 1.0f : a.inv_q);
      if (decided && !taken) {
        ++att;
        fresh = true;
      }
    }
    if (taken) {
      prev = cur; prev_lo = lo; prev_hi = hi;
      cur = x;
      put(cur);
      state = kRow;
    }
  }
}

// A team of kTeam lanes per walk, for launches whose walks do not fill the chip and wait for their chains of reads.  The
// random numbers of an attempt depend on nothing but its number, so lane l of a team makes attempt att + l: the
// candidates of kTeam attempts are under way at once, and the walk takes the first of them, in order of their numbers, that
// is accepted.  An attempt whose acceptance uniform is below every bias is accepted whatever its candidate is, so the
// lanes behind the first such one read nothing.  Candidates behind one that turns out accepted are read in vain: few where
// most accepted attempts are of that kind (p = 0.5, q = 2: all but those of prev and its neighbours), most of a team's where
// few are (p = 4, q = 0.25: one attempt in 16), so the widths go by the attempts a step takes (team_size() below).
// Lanes whose candidate needs the membership search search side by side, as long as no attempt before theirs is accepted.
// The walks of a wave advance in lock step (most steps take one round of attempts), which leaves few instructions
// per step: row bounds, draw, one read of candidates, votes.
template <int kTeam>
__device__ __forceinline__ uint32_t first_in_team(bool vote, int base) {     // ~0u: none
  const uint64_t votes = __ballot(vote);
  if constexpr (kTeam == 64) return votes != 0ull ? (uint32_t)__builtin_ctzll(votes) : ~0u;
  const uint32_t own = (uint32_t)(votes >> base) & (uint32_t)((1ull << (kTeam & 63)) - 1ull);
  return (uint32_t)(__ffs((int)own) - 1);
}
// x of the team's lane `who` (anything if ~0u)
template <int kTeam>
__device__ __forceinline__ int32_t from_lane(int32_t x, uint32_t who, uint32_t sub, int base) {
  if constexpr (kTeam > 16) return __shfl(x, base + (int)(who & 63u), 64);
  uint32_t v = sub == who ? (uint32_t)x : 0u;
  auto step = [&](auto ctrl) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, true);
  };
  if constexpr (kTeam >= 2) step(std::integral_constant<int, 0xB1>());     // quad_perm [1,0,3,2]
  if constexpr (kTeam >= 4) step(std::integral_constant<int, 0x4E>());     // quad_perm [2,3,0,1]
  if constexpr (kTeam >= 8) step(std::integral_constant<int, 0x141>());    // row_half_mirror
  if constexpr (kTeam >= 16) step(std::integral_constant<int, 0x140>());   // row_mirror
  return (int32_t)v;
}

template <typename OffT, typename Pos, bool kWeighted, int kTeam>
__global__ __launch_bounds__(kWalkThreads) void node2vec_team_kernel(WalkArgs a) {
  constexpr int kTeams = kWalkThreads / kTeam;
  static_assert(kMaxAttempts % kTeam == 0, "the last attempt belongs to a team's last lane");
  __shared__ int32_t tile[kTeams][kWinPad];
  const int lane = threadIdx.x & 63, base = lane & ~(kTeam - 1);
  const uint32_t sub = lane & (kTeam - 1);
  const int64_t i = (int64_t)blockIdx.x * kTeams + (int)threadIdx.x / kTeam;
  const bool live = i < a.num_walks;
  const uint64_t id = a.id_base + (uint64_t)i;
  const int32_t* __restrict__ nbrs = a.nbrs;
  const OffT* __restrict__ offsets = static_cast<const OffT*>(a.offsets);
  int32_t* __restrict__ out = a.walks + i * (int64_t)a.walk_len;
  int32_t* mine = tile[(int)threadIdx.x / kTeam];      // (every lane of the team writes all of it, the same values)
  const int32_t last = a.walk_len - 1;      // index of the last position
  const float bias_lo = fminf(1.0f, a.inv_q), bias_hi = fmaxf(1.0f, a.inv_q), bias_min = fminf(a.inv_p, bias_lo);
  const Pos entries = (Pos)a.num_entries;
  const bool wide = a.num_entries >= 4;     // (a probe reads four entries)

  int32_t cur = -1, prev = -1;
  if (live) {
    cur = a.starts[i];
    if (cur < 0 || (int64_t)cur >= a.num_nodes) cur = -1;
  }
  Pos prev_lo = 0, prev_hi = 0;
  for (int32_t t = 0;; ++t) {
    const int col = t & (kWin - 1);
    mine[col] = cur;
    if (col == kWin - 1 || t == last) {
      const int32_t first = t - col;
      if (live)
        for (int c = (int)sub; c <= col; c += kTeam) out[first + c] = mine[c];
    }
    if (t == last) break;
    OffsetPair<OffT> row = {0, 0};
    if (cur >= 0) row = *reinterpret_cast<const OffsetPair<OffT>*>(offsets + cur);
    Block4 b = philox_at(a.seed, id, (uint32_t)t, sub);         // (while the bounds are under way)
    // (registers of upper halves that nobody asks for are given out again at once, and whoever gets one waits for the read)
    if constexpr (sizeof(OffT) > sizeof(Pos)) asm volatile("" : : "v"(row.lo), "v"(row.hi), "v"(b.x0), "v"(b.x3));
    const Pos lo = (Pos)row.lo, hi = (Pos)row.hi;
    bool pending = hi > lo;                 // (the same in all lanes of a team)
    int32_t next = -1;
    for (uint32_t att = sub; __ballot(pending) != 0ull;) {
      Pos j = row_slot(b, (Pos)(hi - lo));
      const float s = unit_float(b.x3) * a.max_bias;
      // unbiased first step; the last attempt is taken
      const bool sure = pending && (t == 0 || s < bias_min || att == kMaxAttempts - 1);
      const bool reads = pending && sub <= first_in_team<kTeam>(sure, base);
      int32_t x = -1;
      if (reads) {
        if (kWeighted) j = (Pos)alias_pick(a, (int64_t)(lo + j), (int64_t)j, b.x2);
        x = nbrs[lo + j];
      }
      bool accepted = false, open = false;
      if ((uint32_t)x >= (uint32_t)a.num_nodes) { x = -1; accepted = reads; }   // not a node (a CSR not built by gs_csr_build): ends the walk
      else if (sure) accepted = true;
      else if (x == prev) accepted = s < a.inv_p;
      else if (s < bias_lo) accepted = true;                    // for x != prev the bias is 1 or 1/q: the search is
      else open = s < bias_hi;                                  // only needed when s falls between the two
      uint32_t winner = first_in_team<kTeam>(accepted, base);
      open = open && sub < winner;
      if (__ballot(open) != 0ull) {
        Pos L = prev_lo, H = prev_hi;
        int32_t v_lo = -1, v_hi = (int32_t)a.num_nodes;
        if (open && (L >= H || !wide)) {    // (prev has a row after a step)
          bool member = false;
          for (Pos e = L; e < H; ++e) member = member || nbrs[e] == x;
          open = false;
          accepted = s < (member ? 1.0f : a.inv_q);
        }
        for (int turn = 0;; turn = turn == 2 ? 0 : turn + 1) {                      // every third probe bisects
          if (open) {
            const Pos pos = probe_at(x, L, H, v_lo, v_hi, turn == 2, entries);
            const Quad quad = *reinterpret_cast<const Quad*>(nbrs + pos);
            bool member;
            if (probe_says(x, pos, quad, L, H, v_lo, v_hi, member)) {
              open = false;
              accepted = s < (member ? 1.0f : a.inv_q);
            }
          }
          winner = first_in_team<kTeam>(accepted, base);
          open = open && sub < winner;
          if (__ballot(open) == 0ull) break;
        }
      }
      const int32_t moved = from_lane<kTeam>(x, winner, sub, base);
      if (pending && winner != ~0u) { next = moved; pending = false; }
      if (__ballot(pending) == 0ull) break;
      att += kTeam;
      b = philox_at(a.seed, id, (uint32_t)t, att);
    }
    prev = cur; prev_lo = lo; prev_hi = hi;
    cur = next;
  }
}

// Lanes per walk; 0: the state machine (unweighted only).  Wide teams have the candidates of more attempts under way and
// cost instructions and lines for attempts that do not matter, so they pay while few walks share the chip, and the
// more attempts a step takes.  Most candidates are no neighbours of prev, so that is about max_bias * q of them: 4 at p =
// 0.5, q = 2, 2 at p = 1, q = 2, 1 at p = 1, q = 0.5 and p = 4, q = 0.25 (more where candidates are prev or its neighbours).
// Microseconds of 40 nodes per walk (20 from 700,000 walks on), R-MAT graph of 4 M nodes and 126 M entries (alias tables: 1 M nodes,
// 18 M entries); "before" is the better of two kernels that are gone, a lane per walk with a read per state or one read per trip.
//   p 0.5, q 2   1000 walks: teams of 64 66, 16 100, 8 140, a lane 475; 6000: 64 119, 32 118, 16 135; 10,000: 64 167, 32 136, 16 142, 8
//                192; 20,000: 32 218, 16 170, 8 207; 47,000: 16 323, 8 273, 4 409, a lane 563; 150,000: 16 821, 8 669, 4 779, a lane 711;
//                200,000: 8 862, a lane 813, before 1013; 400,000: 4 1575, a lane 1508, before 1496; 1 M: 1706, 1555, 1679; 4 M: 6481,
//                5250, 5374; 64-bit offsets, 1 M nodes, 4 M: a lane 4700, before 4629
//      alias     200,000: 8 826, 4 851, 2 993, before 1449; 400,000: 4 1544, 2 1733, 2018; 4 M: 6551, 6797, 7478
//   p 1, q 2     4096 walks: 64 97, 32 112, 16 127, before 475; 12,000: 64 181, 32 145, 16 149, 8 154, 485; 30,000: 16 210, 8 178, 4 222;
//                100,000: 8 398, 4 313, 2 462, 538; 260,000: 4 651, 2 657, a lane 687, 799; 400,000: 990, 1022, 1129, 1145; 4 M:
//                4091, 3850, 3902, 4031
//      alias     100,000: 4 299, 2 434, 660; 260,000: 687, 828, 1020; 1 M: 1086, 1091, 1528; 4 M: 4183, 4045, 4919
//   p 1, q 0.5   4096 walks: 64 95, 32 101, 16 117, before 273; 12,000: 64 170, 32 131, 16 131, 8 143, 275; 20,000: 32 200, 16 152, 8
//                148, 4 157, 270; 47,000: 8 203, 4 192, 2 213, 284; 100,000: 4 251, 2 243, 1 335, 314; 160,000: 403, 280, 363, 428;
//                400,000: 2 643, 1 528, a lane 687, 682; 1 M: 711, 605, 738, 763; 4 M: 2691, 2242, 2599, 2549
//      alias     100,000: 4 238, 2 234, 1 319, before 375; 200,000: 446, 392, 374, 577; 260,000: 595, 589, 411, 598; 4 M: 2 3391, 1
//                2746, 3015
//   p 4, q 0.25  4096 walks: 64 112, 32 121, before 482; 12,000: 32 167, 16 163, 726; 47,000: 8 261, 4 301, 759; 100,000: 4 361, 2 436, 754;
//                160,000: 593, 490, 822; 400,000: 2 984, 1 932, a lane 1139, 1125; 4 M: 3656, 2748, 3139, 3227
// Where reads are quick (an XCD's cache holds the rows of 2^20 entries) what repeats costs more, and where biases are uneven more
// repeats than the attempts say; 10,000 nodes, 180,000 entries, before / then:
//   p 1, q 0.5   400,000 walks: 2 409, 1 444, before 470; 4 M: 2 1534, 1 1383, a lane 1539, before 1612; p 1, q 0.25: 2072, 2057, 1975, 2057
//   p 4, q 0.25  160,000: 4 345, 2 424, before 688; 400,000: 4 692, 2 720, 1 960, a lane 917, before 908; 4 M: 2 2510, 1 2785, a lane 2443, 2493
//      alias     160,000: 4 388, 2 492, 1 820, before 1261; 400,000: 803, 844, 1140, 1624; 4 M: 2 3101, 1 3511, 4013
//   (300,000 nodes, 5.6 M entries, p 4, q 0.25, 160,000 walks: 4 428, 2 461, before 839; 4 M: 2 2393, 1 2473, a lane 2526, 2659)
// Where every candidate other than prev is accepted (the least bias of those is the greatest of all) rounds hardly
// repeat: p = 2, q = 1, 10,000 walks: 4 45, 1 59; 30,000: 4 50, 1 68, a lane 100; 100,000: 4 121, 1 102, a lane 129; p = q = 1,
// 1 M: 1 765, a lane 845.
static int team_size(bool weighted, float q, const WalkArgs& a) {
  const int64_t walks = a.num_walks;
  if (a.max_bias <= fminf(1.0f, a.inv_q)) return walks <= (int64_t)3 << 14 ? 4 : 1;
  const float attempts = a.max_bias * q;
  if (walks <= (int64_t)1 << 12) return 64;
  if (walks <= (int64_t)3 << 12) return 32;
  if (walks <= (int64_t)3 << 13) return 16;
  if (walks <= (attempts >= 3.0f ? (int64_t)5 << 15 : (int64_t)3 << 14)) return 8;
  const int lane = a.num_entries >= 4 && a.num_nodes >= 3 ? 0 : 1;         // (what one read of the state machine needs)
  if (attempts >= 3.0f) return weighted ? 4 : lane;
  if (attempts >= 1.5f) return walks <= (int64_t)1 << 18 ? 4 : (weighted ? 2 : lane);
  // about one attempt: 4 lanes, 2, then 1
  const int64_t entries = a.num_entries;
  const bool uneven = a.max_bias >= 8.0f * fminf(a.inv_p, fminf(1.0f, a.inv_q)), quick = entries <= (int64_t)1 << 20;
  int64_t four = (int64_t)7 << 14, two = quick ? (int64_t)1 << 20 : (weighted ? (int64_t)7 << 15 : (int64_t)1 << 19);
  if (uneven) {
    if (entries <= (int64_t)1 << 23) four = quick ? (int64_t)1 << 19 : (int64_t)1 << 18;
    two = (int64_t)1 << 20;
  }
  if (walks <= four) return 4;
  if (walks <= two || (weighted && uneven && entries <= (int64_t)1 << 21)) return 2;
  return !weighted && (quick || (uneven && entries <= (int64_t)1 << 21)) ? lane : 1;
}

template <typename OffT, typename Pos, bool kWeighted, int kTeam>
static void launch_team(const WalkArgs& a, hipStream_t stream) {
  node2vec_team_kernel<OffT, Pos, kWeighted, kTeam>
      <<<(unsigned)ceil_div(a.num_walks, kWalkThreads / kTeam), kWalkThreads, 0, stream>>>(a);
}

template <typename OffT, typename Pos, bool kWeighted>
static void launch_node2vec(int team, const WalkArgs& a, hipStream_t stream) {
  switch (team) {
    case 1: return launch_team<OffT, Pos, kWeighted, 1>(a, stream);
    case 2: return launch_team<OffT, Pos, kWeighted, 2>(a, stream);
    case 4: return launch_team<OffT, Pos, kWeighted, 4>(a, stream);
    case 8: return launch_team<OffT, Pos, kWeighted, 8>(a, stream);
    case 16: return launch_team<OffT, Pos, kWeighted, 16>(a, stream);
    case 32: return launch_team<OffT, Pos, kWeighted, 32>(a, stream);
    case 64: return launch_team<OffT, Pos, kWeighted, 64>(a, stream);
    default:
      if constexpr (!kWeighted)
        node2vec_kernel<OffT, Pos><<<(unsigned)ceil_div(a.num_walks, kWalkThreads), kWalkThreads, 0, stream>>>(a);
  }
}

// Pos holds the node2vec walker's positions in nbrs, 64 bits only where there are so many entries, whatever the offsets: 64-bit
// offsets, 1 M nodes, 18 M entries, 400,000 walks of 40 nodes at p = 0.5, q = 2 1349 us with 64-bit positions, 1283 with 32; 4 M walks of
// 20 4699 / 4540, at p = 0.25, q = 4 12741 / 12444, with alias tables 21989 / 19367; p = q = 1, 1 M walks of 20 327 / 329.
template <typename OffT, typename Pos>
static void launch_walk(bool weighted, bool second, int team, const WalkArgs& a, hipStream_t stream) {
  const unsigned blocks = (unsigned)ceil_div(a.num_walks, kWalkThreads);
  if (second) {
    if (weighted) launch_node2vec<OffT, Pos, true>(team, a, stream);
    else launch_node2vec<OffT, Pos, false>(team, a, stream);
  } else {
    if (weighted) walk_kernel<OffT, true><<<blocks, kWalkThreads, 0, stream>>>(a);
    else walk_kernel<OffT, false><<<blocks, kWalkThreads, 0, stream>>>(a);
  }
}

// Walks in one launch, whose lanes (at most four to a walk where there are so many) have to stay below 2^32.
constexpr int64_t kLaunchWalks = (int64_t)1 << 28;

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
  a.num_nodes = g->num_nodes;
  a.num_entries = g->num_entries;
  a.num_walks = num_walks;
  a.seed = seed;
  a.walk_len = walk_len;
  a.inv_p = 1.0f / p;
  a.inv_q = 1.0f / q;
  a.max_bias = fmaxf(a.inv_p, fmaxf(1.0f, a.inv_q));
  const int team = second ? team_size(weighted, q, a) : 1;
  for (int64_t first = 0; first < num_walks; first += kLaunchWalks) {
    a.starts = starts + first;
    a.walks = walks_out + first * walk_len;
    a.id_base = id_base + (uint64_t)first;
    a.num_walks = std::min(kLaunchWalks, num_walks - first);
    if (g->offset_bits == 32) launch_walk<int32_t, int32_t>(weighted, second, team, a, stream);
    else if (g->num_entries <= (int64_t)INT32_MAX) launch_walk<int64_t, int32_t>(weighted, second, team, a, stream);
    else launch_walk<int64_t, int64_t>(weighted, second, team, a, stream);
    GS_LAUNCH_CHECK();
  }
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
