// gs_alias_build: alias tables, one per segment, in the canonical first-in
// first-out construction order stated in gs.h (Walker 1977 / Vose 1991).
// The order of the fp64 operations is part of the definition of the table; what
// can run side by side without changing it:
//
//  * The sequential loop pairs the oldest small with the oldest large and appends the
//    large to the back of one of the two lists.  If both lists hold at least m
//    entries, the next m iterations use exactly the first m entries of each list
//    as they stand now (appends go to the back), touch 2m distinct entries, and
//    are independent of each other: they can run side by side, and appending
//    their larges in iteration order (a rank over the "became small" flags)
//    leaves both lists exactly as the sequential loop would.
//  * S, the index-order fp64 sum of the weights: while the running sum stays in one binade,
//    [2^e, 2^(e+1)), it is a whole number N of units u = 2^(e-52), and adding a weight w >= 0 adds
//    round(w / u) to it, where only an exact tie depends on N, and only on whether N is even.  A run of
//    weights is therefore the pair of whole numbers it adds to an even and to an odd N, and such
//    pairs combine in any grouping that keeps their order.  Stretches in which the sum leaves its
//    binade (at most one per doubling of the sum) are added one by one.
//
// Segments of up to kLaneSegment entries are built by one lane each, up to kWaveSegment by one wave
// in LDS, longer ones (the rows of hub nodes) by a workgroup of 1024 lanes; a very long one that is
// alone in its call (the noise table) gets its sum, its lists and its first rounds from the whole chip.
// All are bound by latency, so the limits lie where the next larger team finishes the longest segment
// sooner.  Measured on a 1 M-node graph of 22 M weighted entries: row tables 1.9 ms (lanes 0.29, waves
// 0.20 + 0.45, workgroups 0.92), against 9.5 ms with one lane per row up to 8191 entries; the noise table
// of 1 M entries 2.5 ms (sum 0.45, lists and 16 rounds 0.28, the rest 1.77 in one workgroup), against 18.0
// ms in one workgroup whose lane 0 summed the weights and ran the narrow stretches from global memory.
#include "common.h"

namespace gs {

constexpr int64_t kLaneSegment = 32;
constexpr int kWaveSegment = 2048;

// ---- one lane per segment ------------------------------------------------------------------
template <typename OffT>
__global__ __launch_bounds__(64) void alias_build_kernel(const OffT* __restrict__ seg_offsets,
                                                         int64_t num_segments,
                                                         const float* __restrict__ weights,
                                                         float* __restrict__ prob_out,
                                                         int32_t* __restrict__ alias_out,
                                                         double* __restrict__ mass_ws,
                                                         int32_t* __restrict__ small_ws,
                                                         int32_t* __restrict__ large_ws) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= num_segments) return;
  const int64_t begin = (int64_t)seg_offsets[s];
  const int64_t n = (int64_t)seg_offsets[s + 1] - begin;
  if (n <= 0 || n > kLaneSegment) return;
  const float* w = weights + begin;
  float* prob = prob_out + begin;
  int32_t* alias = alias_out + begin;
  double* mass = mass_ws + begin;
  int32_t* small_q = small_ws + begin;   // every entry enters at most once: no wrap
  int32_t* large_q = large_ws + begin;   // ring of capacity n

  double S = 0.0;
  for (int64_t i = 0; i < n; ++i) S += (double)w[i];
  int64_t small_head = 0, small_tail = 0;
  int64_t large_head = 0, large_count = 0;
  const double dn = (double)n;
  for (int64_t i = 0; i < n; ++i) {
    const double m = (double)w[i] * dn;
    mass[i] = m;
    if (m < S) small_q[small_tail++] = (int32_t)i;
    else large_q[large_count++] = (int32_t)i;
  }
  while (small_head < small_tail && large_count > 0) {
    const int32_t a = small_q[small_head++];
    const int32_t b = large_q[large_head];
    large_head = (large_head + 1 == n) ? 0 : large_head + 1;
    --large_count;
    const double ma = mass[a];
    prob[a] = (float)(ma / S);
    alias[a] = b;
    const double mb = (mass[b] + ma) - S;
    mass[b] = mb;
    if (mb < S) {
      small_q[small_tail++] = b;
    } else {
      int64_t at = large_head + large_count;
      if (at >= n) at -= n;
      large_q[at] = b;
      ++large_count;
    }
  }
  for (; small_head < small_tail; ++small_head) {
    const int32_t i = small_q[small_head];
    prob[i] = 1.0f;
    alias[i] = i;
  }
  for (; large_count > 0; --large_count) {
    const int32_t i = large_q[large_head];
    large_head = (large_head + 1 == n) ? 0 : large_head + 1;
    prob[i] = 1.0f;
    alias[i] = i;
  }
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// ---- one wave per segment --------------------------------------------------------------------
// Segments of MIN_N .. MAX_N entries: masses and both lists in LDS, up to 64 iterations at a time.  A
// wave looks at `per_wave` consecutive segments and takes those of its size.
template <typename OffT, int MIN_N, int MAX_N>
__global__ __launch_bounds__(64) void alias_build_wave_kernel(const OffT* __restrict__ seg_offsets,
                                                              int64_t num_segments, int per_wave,
                                                              const float* __restrict__ weights,
                                                              float* __restrict__ prob_out,
                                                              int32_t* __restrict__ alias_out) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  static_assert((MAX_N & (MAX_N - 1)) == 0, "the list of larges wraps by a mask");
  __shared__ double mass[MAX_N];
  __shared__ uint16_t small_q[MAX_N];          // every entry enters at most once: no wrap
  __shared__ uint16_t large_q[MAX_N];
  const int lane = threadIdx.x;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t first = (int64_t)blockIdx.x * per_wave;
  int64_t my_begin = 0, my_n = 0;
  if (lane < per_wave && first + lane < num_segments) {
    my_begin = (int64_t)seg_offsets[first + lane];
    my_n = (int64_t)seg_offsets[first + lane + 1] - my_begin;
  }
  uint64_t todo = __ballot(my_n >= MIN_N && my_n <= MAX_N);
  while (todo != 0ull) {
    const int who = __ffsll((unsigned long long)todo) - 1;
    todo &= todo - 1ull;
    const int n = __builtin_amdgcn_readlane((int)my_n, who);
    const int64_t begin = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(my_begin >> 32), who) << 32) |
                                    (uint32_t)__builtin_amdgcn_readlane((int)my_begin, who));
    const float* w = weights + begin;
    float* prob = prob_out + begin;
    int32_t* alias = alias_out + begin;
    const double dn = (double)n;
    double S = 0.0;
    for (int base = 0; base < n; base += 64) {
      const double v = base + lane < n ? (double)w[base + lane] : 0.0;
#pragma unroll 16
      for (int k = 0; k < 64; ++k) S += lane_value(v, k);       // (+ 0.0 behind the end changes nothing)
      if (base + lane < n) mass[base + lane] = v * dn;
    }
    int sh = 0, st = 0, lh = 0, lt = 0;        // heads and tails of the lists, the same in every lane
    wave_fence();
    for (int base = 0; base < n; base += 64) {
      const bool valid = base + lane < n;
      const bool is_small = valid && mass[base + lane] < S;
      const uint64_t smalls = __ballot(is_small), larges = __ballot(valid && !is_small);
      if (is_small) small_q[st + __popcll(smalls & below)] = (uint16_t)(base + lane);
      else if (valid) large_q[lt + __popcll(larges & below)] = (uint16_t)(base + lane);
      st += __popcll(smalls);
      lt += __popcll(larges);
    }
    wave_fence();
    while (sh < st && lh < lt) {
      const int m = min(64, min(st - sh, lt - lh));
      int b = 0;
      bool demoted = false;
      if (lane < m) {
        const int a = small_q[sh + lane];
        b = large_q[(lh + lane) & (MAX_N - 1)];
        const double ma = mass[a];
        prob[a] = (float)(ma / S);
        alias[a] = b;
        const double mb = (mass[b] + ma) - S;
        mass[b] = mb;
        demoted = mb < S;
      }
      const uint64_t down = __ballot(lane < m && demoted), stay = __ballot(lane < m && !demoted);
      sh += m;
      lh += m;
      wave_fence();
      if (lane < m) {
        if (demoted) small_q[st + __popcll(down & below)] = (uint16_t)b;
        else large_q[(lt + __popcll(stay & below)) & (MAX_N - 1)] = (uint16_t)b;
      }
      st += __popcll(down);
      lt += __popcll(stay);
      wave_fence();
    }
    for (int i = sh + lane; i < st; i += 64) {
      const int x = small_q[i];
      prob[x] = 1.0f;
      alias[x] = x;
    }
    for (int i = lh + lane; i < lt; i += 64) {
      const int x = large_q[i & (MAX_N - 1)];
      prob[x] = 1.0f;
      alias[x] = x;
    }
    wave_fence();
  }
}

// ---- one workgroup per long segment --------------------------------------------------------
// The lists live in global memory (all of a workgroup's accesses go through one compute unit's
// cache, so a barrier is all that orders them).  Rounds of at least kNarrow iterations are run by
// the workgroup, kLongTrip iterations at a time; narrower ones by one wave that keeps the heads of
// both lists in LDS.
constexpr int kLongThreads = 1024, kLongWaves = kLongThreads / 64;
constexpr int kLongItems = 4;                                  // iterations per lane and trip
constexpr int kLongTrip = kLongThreads * kLongItems;
constexpr int kSumItems = 16;                                  // consecutive weights per lane of the sum
constexpr int kSumChunk = 64 * kSumItems;                      // per wave
constexpr int64_t kNarrow = 512;
constexpr int kRing = 1024;                                    // list entries kept in LDS

struct Runs { long long even, odd; };          // what a run of weights adds to an even / odd whole number of units
__device__ __forceinline__ Runs then(const Runs& a, const Runs& b) {
  Runs r;
  r.even = a.even + ((a.even & 1) ? b.odd : b.even);
  r.odd = a.odd + ((a.odd & 1) ? b.even : b.odd);
  return r;
}

struct __attribute__((packed, aligned(4))) Weight4 { float v[4]; };

// The run of the kSumChunk weights from `at` on (lane l: kSumItems of them), for sums in the binade of
// exponent e; lane 0 gets it.  false: some weight is negative, not finite or beyond the binade.
__device__ __forceinline__ bool run_of_chunk(const float* __restrict__ w, int64_t at, int64_t n, int e, Runs& run) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const double per_unit = __longlong_as_double((long long)(uint64_t)(52 - e + 1023) << 52);
  at += lane * kSumItems;
  float v[kSumItems];
  if (at + kSumItems <= n) {
#pragma unroll
    for (int q = 0; q < kSumItems / 4; ++q) {
      const Weight4 x = *reinterpret_cast<const Weight4*>(w + at + 4 * q);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[4 * q + k] = x.v[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < kSumItems; ++k) v[k] = at + k < n ? w[at + k] : 0.f;
  }
  Runs r = {0, 0};
  bool bad = false;
#pragma unroll
  for (int k = 0; k < kSumItems; ++k) {
    const double t = (double)v[k] * per_unit;                  // exact: a power of two
    if (!(t >= 0.0 && t < 0x1p52)) { bad = true; continue; }
    const double fl = floor(t), rest = t - fl;
    const long long whole = (long long)fl;
    const long long tie = rest == 0.5, up = rest > 0.5;
    // N + whole + rest, rounded to the nearest whole number, ties to even
    r.even += whole + (up | (tie & (r.even + whole)));
    r.odd += whole + (up | (tie & (r.odd + 1 + whole)));
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {                            // lane l: the run of lanes l .. l + d - 1
    Runs next;
    next.even = __shfl_down(r.even, d, 64);
    next.odd = __shfl_down(r.odd, d, 64);
    r = then(r, next);
  }
  run = r;
  return __ballot(bad) == 0ull;
}

// kSumChunk weights from `pos` on added to S one by one, by a wave
__device__ __forceinline__ double add_one_by_one(double S, const float* __restrict__ w, int64_t pos, int64_t n) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  float v[kSumItems];
#pragma unroll
  for (int k = 0; k < kSumItems; ++k) v[k] = pos + k * 64 + lane < n ? w[pos + k * 64 + lane] : 0.f;
#pragma unroll 1
  for (int k = 0; k < kSumItems; ++k) {        // (+ 0.0 behind the end changes nothing)
    const double x = (double)v[0];
#pragma unroll 16
    for (int l = 0; l < 64; ++l) S += lane_value(x, l);
#pragma unroll
    for (int q = 1; q < kSumItems; ++q) v[q - 1] = v[q];
  }
  return S;
}

__device__ __forceinline__ bool sums_by_runs(double S) { return S >= 0x1p-200 && S < 0x1p+200; }
__device__ __forceinline__ int exponent_of(double S) {
  return (int)(((uint64_t)__double_as_longlong(S) >> 52) & 2047u) - 1023;
}
// S after a run; false (S unchanged): the sum would leave its binade
__device__ __forceinline__ bool add_run(double& S, const Runs& run) {
  const int e = exponent_of(S);
  const double per_unit = __longlong_as_double((long long)(uint64_t)(52 - e + 1023) << 52);
  const double unit = __longlong_as_double((long long)(uint64_t)(e - 52 + 1023) << 52);
  const long long N = (long long)(S * per_unit);                // in [2^52, 2^53)
  const long long more = N + ((N & 1) ? run.odd : run.even);
  if (more >= (1ll << 53)) return false;
  S = (double)more * unit;
  return true;
}

// index-order fp64 sum of w[0..n); every lane gets it
__device__ double ordered_sum(const float* __restrict__ w, int64_t n, Runs* run_s, uint32_t* bad_s, double* sum_s) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double S = 0.0;
  int64_t pos = 0;
  while (pos < n) {
    int taken = 0;                             // waves whose chunk has been added
    if (sums_by_runs(S)) {
      Runs r;
      const bool good = run_of_chunk(w, pos + wave * kSumChunk, n, exponent_of(S), r);
      if (lane == 0) { run_s[wave] = r; bad_s[wave] = !good; }
      __syncthreads();
      while (taken < kLongWaves && bad_s[taken] == 0u && add_run(S, run_s[taken])) ++taken;
      pos += (int64_t)taken * kSumChunk;
    }
    if (taken < kLongWaves && pos < n) {       // the sum leaves its binade in this chunk (or starts)
      if (wave == 0) {                         // (all waves at once would share the issue slots)
        S = add_one_by_one(S, w, pos, n);
        if (lane == 0) *sum_s = S;
      }
      __syncthreads();
      S = *sum_s;
      pos += kSumChunk;
    }
    __syncthreads();
  }
  return S;
}

// places of the wave's votes in the workgroup's order, for two kinds of votes at once: c0 and c1
// are the wave's totals; returns the totals of the waves before, and all of them
__device__ __forceinline__ void block_before(int c0, int c1, int (*tot)[kLongWaves], int& before0, int& before1,
                                             int& all0, int& all1) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if ((threadIdx.x & 63) == 0) { tot[0][wave] = c0; tot[1][wave] = c1; }
  __syncthreads();
  int v0[kLongWaves], v1[kLongWaves];
#pragma unroll
  for (int v = 0; v < kLongWaves; ++v) { v0[v] = tot[0][v]; v1[v] = tot[1][v]; }
  before0 = before1 = all0 = all1 = 0;
#pragma unroll
  for (int v = 0; v < kLongWaves; ++v) {
    before0 += v < wave ? v0[v] : 0;
    before1 += v < wave ? v1[v] : 0;
    all0 += v0[v];
    all1 += v1[v];
  }
}

template <typename OffT>
__global__ void alias_find_long_kernel(const OffT* __restrict__ seg_offsets, int64_t num_segments,
                                       int64_t* __restrict__ long_ids, int64_t capacity,
                                       unsigned long long* __restrict__ long_count) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= num_segments) return;
  if ((int64_t)seg_offsets[s + 1] - (int64_t)seg_offsets[s] > kWaveSegment) {
    // capacity = total_entries / (kWaveSegment + 1) bounds the count when the offsets add up to
    // total_entries; an inconsistent pair of arguments must still not write out of bounds
    const unsigned long long at = atomicAdd(long_count, 1ull);
    if (at < (unsigned long long)capacity) long_ids[at] = s;
  }
}

__global__ void zero_u64_kernel(unsigned long long* p) { *p = 0ull; }

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)x));
}

// The head of a list as one wave keeps it: entries [head, loaded) of the list in a ring in LDS.
struct Window {
  int32_t* id;
  double* mass;
  int64_t head, loaded, tail;                  // the list itself is [head, tail)
};
__device__ __forceinline__ void refill(Window& q, const int32_t* list, const double* mass, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");       // what this wave appended has to be there
  const int64_t end = min(q.tail, q.head + kRing);
  int32_t x[kRing / 64];                       // (entries behind the end: the last one again, so that no read waits in a branch)
  double m[kRing / 64];
#pragma unroll
  for (int c = 0; c < kRing / 64; ++c) x[c] = list[min(q.loaded + c * 64 + lane, end - 1)];
#pragma unroll
  for (int c = 0; c < kRing / 64; ++c) m[c] = mass[x[c]];
#pragma unroll
  for (int c = 0; c < kRing / 64; ++c) {
    const int64_t i = q.loaded + c * 64 + lane;
    if (i < end) {
      q.id[i & (kRing - 1)] = x[c];
      q.mass[i & (kRing - 1)] = m[c];
    }
  }
  q.loaded = end;
  wave_fence();
}
// appends the lanes with `mine` set, in lane order, to the list and, if the ring reaches that far, to the ring
__device__ __forceinline__ void append(Window& q, int32_t* list, bool mine, int32_t x, double m, int lane) {
  const uint64_t votes = __ballot(mine);
  const int count = __popcll(votes);
  const bool in_ring = q.loaded == q.tail && q.tail + count <= q.head + kRing;
  if (mine) {
    const int64_t at = q.tail + __popcll(votes & ((1ull << lane) - 1ull));
    list[at] = x;
    if (in_ring) { q.id[at & (kRing - 1)] = x; q.mass[at & (kRing - 1)] = m; }
  }
  q.tail += count;
  if (in_ring) q.loaded = q.tail;
}

// ---- a single very long segment: its first rounds by the whole chip -------------------------
// One workgroup moves about one cache line per cycle, which bounds the rounds of hundreds of
// thousands of iterations a noise table starts with.  A segment that is alone in its call and long
// enough therefore gets its sum, its lists and its first rounds from launches of many workgroups (a round is
// two kernels: iterate, then append behind both lists), and the rest from the workgroup kernel.
// A round that has become narrower than kWideRound is left to that one.  Measured in ms, degree^0.75 of a skewed
// graph and lognormal weights: the whole chip against one workgroup, 2^15 entries 0.39 / 0.34 and 0.32 / 0.28, 2^16
// 0.56 / 0.55 and 0.41 / 0.42 (2^17 equal weights 0.32 / 0.33, half of them zero 0.37 / 0.52; 2^18 0.40 / 0.52 and
// 0.44 / 0.93).  16 rounds against 48: 1 M entries 1.99 / 2.07 and 1.31 / 1.41, 2 M 3.36 / 3.18 and 1.83 / 1.84, 4 M
// 4.83 / 3.93 and 3.03 / 2.68, 8 M 8.61 / 5.95 and 5.36 / 3.99 (so the line between them could lie at 2 M).
// kWideRound of 2048, 8192 and 32768: 1 M entries 1.99, 1.99, 2.37, 8 M 5.92, 5.96, 7.15.
struct ListState { int64_t sh, st, lh, lt; };
constexpr int64_t kWideSegment = (int64_t)1 << 17;
constexpr int64_t kWideRound = 8192;
static int wide_rounds(int64_t n) { return n < ((int64_t)1 << 22) ? 16 : 48; }
constexpr int kMostWideRounds = 48;

// The sum in three steps: plain sums of the chunks, their prefix sums (which name the binade that the
// running sum is in when it reaches a chunk, but for those next to a border), and the run of every
// chunk for that binade; then one workgroup adds run after run, and one by one where the binade was not
// the one or is left.
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_chunks_kernel(const OffT* __restrict__ seg_offsets,
                                                                         const float* __restrict__ weights,
                                                                         double* __restrict__ chunk_sums) {
  const int lane = threadIdx.x & 63;
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const int64_t waves = (int64_t)gridDim.x * kLongWaves;
  for (int64_t c = (int64_t)blockIdx.x * kLongWaves + (threadIdx.x >> 6); c * kSumChunk < n; c += waves) {
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kSumItems; ++k) {
      const int64_t i = c * kSumChunk + k * 64 + lane;
      sum += i < n ? (double)weights[begin + i] : 0.0;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) chunk_sums[c] = sum;
  }
}

template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_prefix_kernel(const OffT* __restrict__ seg_offsets,
                                                                         double* __restrict__ chunk_sums) {
  __shared__ double part[2][kLongWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = (int64_t)seg_offsets[1] - (int64_t)seg_offsets[0], chunks = (n + kSumChunk - 1) / kSumChunk;
  double carry = 0.0;
  int turn = 0;
  for (int64_t base = 0; base < chunks; base += kLongThreads, turn ^= 1) {
    const int64_t c = base + threadIdx.x;
    const double own = c < chunks ? chunk_sums[c] : 0.0;
    double incl = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const double up = __shfl_up(incl, d, 64);
      if (lane >= d) incl += up;
    }
    if (lane == 63) part[turn][wave] = incl;
    __syncthreads();
    double before = carry + incl - own;
#pragma unroll
    for (int w = 0; w < kLongWaves; ++w) {
      if (w < wave) before += part[turn][w];
      carry += part[turn][w];
    }
    if (c < chunks) chunk_sums[c] = before;
  }
}

struct ChunkRun { Runs run; int e; int good; };
template <typename OffT>
__global__ __launch_bounds__(256) void alias_wide_runs_kernel(const OffT* __restrict__ seg_offsets,
                                                              const float* __restrict__ weights,
                                                              const double* __restrict__ chunk_sums,
                                                              ChunkRun* __restrict__ runs) {
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const int64_t waves = (int64_t)gridDim.x * 4;
  for (int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); c * kSumChunk < n; c += waves) {
    const double S = chunk_sums[c];
    ChunkRun x = {{0, 0}, 0, 0};
    if (sums_by_runs(S)) {
      x.e = exponent_of(S);
      x.good = run_of_chunk(weights + begin, c * kSumChunk, n, x.e, x.run) ? 1 : 0;
    }
    if ((threadIdx.x & 63) == 0) runs[c] = x;
  }
}

template <typename OffT>
__global__ __launch_bounds__(256) void alias_wide_sum_kernel(const OffT* __restrict__ seg_offsets,
                                                             const float* __restrict__ weights,
                                                             const ChunkRun* __restrict__ runs,
                                                             double* __restrict__ sum_out) {
  constexpr int kAtOnce = 512;
  __shared__ ChunkRun run_s[kAtOnce];
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const int64_t chunks = (n + kSumChunk - 1) / kSumChunk;
  double S = 0.0;
  for (int64_t base = 0; base < chunks; base += kAtOnce) {
    __syncthreads();
    for (int64_t c = base + threadIdx.x; c < min(chunks, base + kAtOnce); c += 256) run_s[c - base] = runs[c];
    __syncthreads();
    const int here = (int)min((int64_t)kAtOnce, chunks - base);
    for (int c = 0; c < here; ++c) {
      const ChunkRun& x = run_s[c];
      if (x.good != 0 && sums_by_runs(S) && exponent_of(S) == x.e && add_run(S, x.run)) continue;
      S = add_one_by_one(S, weights + begin, (base + c) * kSumChunk, n);
    }
  }
  if (threadIdx.x == 0) *sum_out = S;
}

// sum of counts[0 .. tile), by the whole workgroup
__device__ __forceinline__ int64_t counts_before(const int32_t* __restrict__ counts, int64_t tile, int64_t* part) {
  int64_t sum = 0;
  for (int64_t i = threadIdx.x; i < tile; i += kLongThreads) sum += counts[i];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = 0;
#pragma unroll
  for (int w = 0; w < kLongWaves; ++w) sum += part[w];
  return sum;
}

// masses, and which entries start as smalls: a bit per entry and a count per tile
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_masses_kernel(const OffT* __restrict__ seg_offsets,
                                                                         const float* __restrict__ weights,
                                                                         const double* __restrict__ sum, double* mass_ws,
                                                                         uint64_t* __restrict__ flags,
                                                                         int32_t* __restrict__ counts) {
#pragma clang fp contract(off)
  __shared__ int32_t tot[kLongWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const double S = *sum, dn = (double)n;
  for (int64_t tile = blockIdx.x; tile * kLongTrip < n; tile += gridDim.x) {
    const int64_t first = tile * kLongTrip + wave * (64 * kLongItems);
    int32_t count = 0;
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      const int64_t i = first + c * 64 + lane;
      const double m = i < n ? (double)weights[begin + i] * dn : 0.0;
      if (i < n) mass_ws[begin + i] = m;
      const uint64_t smalls = __ballot(i < n && m < S);
      if (lane == 0 && first + c * 64 < n) flags[(first >> 6) + c] = smalls;
      count += __popcll(smalls);
    }
    if (lane == 0) tot[wave] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t all = 0;
#pragma unroll
      for (int w = 0; w < kLongWaves; ++w) all += tot[w];
      counts[tile] = all;
    }
    __syncthreads();
  }
}

// Appends entries 0 .. m - 1 (entry i is i itself, or large_q[lh + i]) behind the smalls or the larges, in
// order, by their flags; the workgroup with the last tile writes the lists' next state.
// initial: the lists are empty and the entries are the segment's.
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_append_kernel(const OffT* __restrict__ seg_offsets,
                                                                         int32_t* small_ws, int32_t* large_ws,
                                                                         const uint64_t* __restrict__ flags,
                                                                         const int32_t* __restrict__ counts,
                                                                         ListState* __restrict__ states, int initial) {
  __shared__ int64_t part[kLongWaves];
  __shared__ int32_t tot[kLongWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  int32_t* small_q = small_ws + begin;
  int32_t* large_q = large_ws + 2 * begin;
  ListState at = {0, 0, 0, 0};
  if (!initial) at = states[0];
  const int64_t m = initial ? n : min(at.st - at.sh, at.lt - at.lh);
  if (!initial && m < kWideRound) {
    if (blockIdx.x == 0 && threadIdx.x == 0) states[1] = at;
    return;
  }
  const int64_t tiles = (m + kLongTrip - 1) / kLongTrip;
  if (tiles == 0 && blockIdx.x == 0 && threadIdx.x == 0) states[0] = at;     // (an empty segment)
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t before = counts_before(counts, tile, part);
    const int64_t first = tile * kLongTrip + wave * (64 * kLongItems);
    uint64_t down[kLongItems];
    int32_t count = 0;
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      down[c] = first + c * 64 < m ? flags[(first >> 6) + c] : 0ull;
      count += __popcll(down[c]);
    }
    if (lane == 0) tot[wave] = count;
    __syncthreads();
    int64_t rank = before;
    int32_t all = 0;
#pragma unroll
    for (int w = 0; w < kLongWaves; ++w) {
      if (w < wave) rank += tot[w];
      all += tot[w];
    }
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      const int64_t i = first + c * 64 + lane;
      const int64_t d = rank + __popcll(down[c] & below);           // flagged entries before i
      if (i < m) {
        const int32_t b = initial ? (int32_t)i : large_q[at.lh + i];
        if ((down[c] >> lane) & 1ull) small_q[at.st + d] = b;
        else large_q[at.lt + (i - d)] = b;
      }
      rank += __popcll(down[c]);
    }
    if (tile == tiles - 1 && threadIdx.x == 0) {
      const int64_t flagged = before + all;
      ListState next = {at.sh + m, at.st + flagged, at.lh + m, at.lt + (m - flagged)};
      if (initial) next = {0, flagged, 0, n - flagged};
      states[initial ? 0 : 1] = next;
    }
    __syncthreads();
  }
}

// one round: m iterations, which larges became smalls
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_round_kernel(
    const OffT* __restrict__ seg_offsets, const double* __restrict__ sum, float* __restrict__ prob_out,
    int32_t* __restrict__ alias_out, double* mass_ws, const int32_t* __restrict__ small_ws,
    const int32_t* __restrict__ large_ws, uint64_t* __restrict__ flags, int32_t* __restrict__ counts,
    const ListState* __restrict__ states) {
#pragma clang fp contract(off)
  __shared__ int32_t tot[kLongWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t begin = (int64_t)seg_offsets[0];
  const ListState at = states[0];
  const int64_t m = min(at.st - at.sh, at.lt - at.lh);
  if (m < kWideRound) return;
  const double S = *sum;
  const int32_t* small_q = small_ws + begin + at.sh;
  const int32_t* large_q = large_ws + 2 * begin + at.lh;
  float* prob = prob_out + begin;
  int32_t* alias = alias_out + begin;
  double* mass = mass_ws + begin;
  for (int64_t tile = blockIdx.x; tile * kLongTrip < m; tile += gridDim.x) {
    const int64_t first = tile * kLongTrip + wave * (64 * kLongItems);
    int32_t count = 0;
    int32_t a[kLongItems], b[kLongItems];
    double ma[kLongItems], mb[kLongItems];
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {                      // (behind the end: the last one again, read but not used)
      const int64_t i = min(first + c * 64 + lane, m - 1);
      a[c] = small_q[i];
      b[c] = large_q[i];
    }
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      ma[c] = mass[a[c]];
      mb[c] = mass[b[c]];
    }
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      const bool valid = first + c * 64 + lane < m;
      mb[c] = (mb[c] + ma[c]) - S;
      if (valid) {
        prob[a[c]] = (float)(ma[c] / S);
        alias[a[c]] = b[c];
        mass[b[c]] = mb[c];
      }
      const uint64_t down = __ballot(valid && mb[c] < S);
      if (lane == 0 && first + c * 64 < m) flags[(first >> 6) + c] = down;
      count += __popcll(down);
    }
    if (lane == 0) tot[wave] = count;
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t all = 0;
#pragma unroll
      for (int w = 0; w < kLongWaves; ++w) all += tot[w];
      counts[tile] = all;
    }
    __syncthreads();
  }
}

// long_ids == null: the single segment 0; resume != null: whose sum and lists exist already.
// Scratch per entry of the segment, at the segment's own offsets: mass, the
// small list (n entries), the large list (2n: appended without wrapping).
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_build_long_kernel(
    const OffT* __restrict__ seg_offsets, const int64_t* __restrict__ long_ids,
    const unsigned long long* __restrict__ long_count, const float* __restrict__ weights,
    float* __restrict__ prob_out, int32_t* __restrict__ alias_out, double* mass_ws,
    int32_t* small_ws, int32_t* large_ws, const ListState* __restrict__ resume, const double* __restrict__ sum) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  __shared__ Runs run_s[kLongWaves];
  __shared__ uint32_t bad_s[kLongWaves];
  __shared__ double sum_s;
  __shared__ int tot[2][2][kLongWaves];        // (two sets, used in turn: one barrier per use)
  __shared__ int64_t q_s[4];                   // small head/tail, large head/tail after a narrow stretch
  __shared__ int32_t ring_id[2][kRing];
  __shared__ double ring_mass[2][kRing];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
  if (long_ids != nullptr && (unsigned long long)blockIdx.x >= *long_count) return;
  const int64_t seg = long_ids != nullptr ? long_ids[blockIdx.x] : 0;
  const int64_t begin = (int64_t)seg_offsets[seg];
  const int64_t n = (int64_t)seg_offsets[seg + 1] - begin;
  if (n <= 0) return;
  const float* w = weights + begin;
  float* prob = prob_out + begin;
  int32_t* alias = alias_out + begin;
  double* mass = mass_ws + begin;
  int32_t* small_q = small_ws + begin;
  int32_t* large_q = large_ws + 2 * begin;

  const double S = resume != nullptr ? *sum : ordered_sum(w, n, run_s, bad_s, &sum_s);
  const double dn = (double)n;
  int turn = 0;

  // initial lists, in index order (a wave takes 64 * kLongItems consecutive entries of a trip)
  int64_t sh = 0, st = 0, lh = 0, lt = 0;     // heads and tails, identical in every lane
  if (resume != nullptr) {
    sh = resume->sh; st = resume->st; lh = resume->lh; lt = resume->lt;
  }
  for (int64_t base = resume != nullptr ? n : 0; base < n; base += kLongTrip, turn ^= 1) {
    const int64_t first = base + wave * (64 * kLongItems) + lane;
    float v[kLongItems];
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) v[c] = first + c * 64 < n ? w[first + c * 64] : 0.f;
    uint64_t smalls[kLongItems], larges[kLongItems];
    int cs = 0, cl = 0;
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      const bool valid = first + c * 64 < n;
      const double m = (double)v[c] * dn;
      if (valid) mass[first + c * 64] = m;
      smalls[c] = __ballot(valid && m < S);
      larges[c] = __ballot(valid && !(m < S));
      cs += __popcll(smalls[c]);
      cl += __popcll(larges[c]);
    }
    int bs, bl, as, al;
    block_before(cs, cl, tot[turn], bs, bl, as, al);
#pragma unroll
    for (int c = 0; c < kLongItems; ++c) {
      const int32_t i = (int32_t)(first + c * 64);
      if ((smalls[c] >> lane) & 1ull) small_q[st + bs + __popcll(smalls[c] & below)] = i;
      else if ((larges[c] >> lane) & 1ull) large_q[lt + bl + __popcll(larges[c] & below)] = i;
      bs += __popcll(smalls[c]);
      bl += __popcll(larges[c]);
    }
    st += as;
    lt += al;
  }

  while (true) {
    __syncthreads();
    const int64_t m = min(st - sh, lt - lh);
    if (m <= 0) break;
    if (m < kNarrow) {
      const int64_t popped = sh;               // the smalls from here on are taken in this stretch
      if (wave == 0) {
        Window s = {ring_id[0], ring_mass[0], uniform64(sh), uniform64(sh), uniform64(st)};
        Window l = {ring_id[1], ring_mass[1], uniform64(lh), uniform64(lh), uniform64(lt)};
        while (true) {
          const int64_t both = min(s.tail - s.head, l.tail - l.head);
          if (both <= 0 || both >= 2 * kNarrow) break;
          if (s.head == s.loaded) refill(s, small_q, mass, lane);
          if (l.head == l.loaded) refill(l, large_q, mass, lane);
          const int k = (int)min((int64_t)64, min(s.loaded - s.head, l.loaded - l.head));
          int32_t b = 0;
          double mb = 0.0;
          if (lane < k) {
            const int at_s = ((int)s.head + lane) & (kRing - 1), at_l = ((int)l.head + lane) & (kRing - 1);
            const int32_t a = s.id[at_s];
            b = l.id[at_l];
            mb = (l.mass[at_l] + s.mass[at_s]) - S;
            alias[a] = b;
            mass[b] = mb;
          }
          s.head += k;
          l.head += k;
          wave_fence();
          const bool demoted = mb < S;
          append(s, small_q, lane < k && demoted, b, mb, lane);
          append(l, large_q, lane < k && !demoted, b, mb, lane);
          wave_fence();
        }
        if (lane == 0) { q_s[0] = s.head; q_s[1] = s.tail; q_s[2] = l.head; q_s[3] = l.tail; }
      }
      __syncthreads();
      sh = q_s[0]; st = q_s[1]; lh = q_s[2]; lt = q_s[3];
      // (a small's mass does not change once it is one: the divisions are left to all lanes)
      for (int64_t i = popped + tid; i < sh; i += kLongThreads) {
        const int32_t a = small_q[i];
        prob[a] = (float)(mass[a] / S);
      }
      continue;
    }
    int64_t add_s = 0, add_l = 0;
    for (int64_t base = 0; base < m; base += kLongTrip, turn ^= 1) {
      const int64_t first = base + wave * (64 * kLongItems) + lane;
      int32_t a[kLongItems], b[kLongItems];
      double ma[kLongItems], mb[kLongItems];
#pragma unroll
      for (int c = 0; c < kLongItems; ++c) {                   // (behind the end: the last one again, read but not used)
        const int64_t i = min(first + c * 64, m - 1);
        a[c] = small_q[sh + i];
        b[c] = large_q[lh + i];
      }
#pragma unroll
      for (int c = 0; c < kLongItems; ++c) {
        ma[c] = mass[a[c]];
        mb[c] = mass[b[c]];
      }
      uint64_t down[kLongItems], stay[kLongItems];
      int cd = 0, cs = 0;
#pragma unroll
      for (int c = 0; c < kLongItems; ++c) {
        const bool valid = first + c * 64 < m;
        mb[c] = (mb[c] + ma[c]) - S;
        if (valid) {
          prob[a[c]] = (float)(ma[c] / S);
          alias[a[c]] = b[c];
          mass[b[c]] = mb[c];
        }
        down[c] = __ballot(valid && mb[c] < S);
        stay[c] = __ballot(valid && !(mb[c] < S));
        cd += __popcll(down[c]);
        cs += __popcll(stay[c]);
      }
      int bd, bs, ad, as;
      block_before(cd, cs, tot[turn], bd, bs, ad, as);
#pragma unroll
      for (int c = 0; c < kLongItems; ++c) {
        if ((down[c] >> lane) & 1ull) small_q[st + add_s + bd + __popcll(down[c] & below)] = b[c];
        else if ((stay[c] >> lane) & 1ull) large_q[lt + add_l + bs + __popcll(stay[c] & below)] = b[c];
        bd += __popcll(down[c]);
        bs += __popcll(stay[c]);
      }
      add_s += ad;
      add_l += as;
    }
    sh += m; lh += m;
    st += add_s; lt += add_l;
  }
  for (int64_t i = sh + tid; i < st; i += kLongThreads) {
    const int32_t x = small_q[i];
    prob[x] = 1.0f; alias[x] = x;
  }
  for (int64_t i = lh + tid; i < lt; i += kLongThreads) {
    const int32_t x = large_q[i];
    prob[x] = 1.0f; alias[x] = x;
  }
}

__global__ void alias_pack_kernel(const float* __restrict__ prob, const int32_t* __restrict__ alias,
                                  int64_t n, uint64_t* __restrict__ packed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) packed[i] = ((uint64_t)(uint32_t)alias[i] << 32) | (uint64_t)__float_as_uint(prob[i]);
}

struct AliasPlan {
  double* mass;
  int32_t *small_q, *large_q;
  int64_t* long_ids;
  unsigned long long* long_count;
  int64_t max_long;
  size_t bytes;
  // a single very long segment only, behind the rest: null in a workspace without room for them
  double* sum;
  double* chunk_sums;
  ChunkRun* runs;
  ListState* states;
  uint64_t* flags;
  int32_t* counts;
  size_t wide_bytes;
};

static AliasPlan plan_alias(void* ws, int64_t total_entries) {
  Carver cv(ws);
  AliasPlan p;
  const size_t t = (size_t)(total_entries > 0 ? total_entries : 1);
  p.mass = cv.take<double>(t);
  p.small_q = cv.take<int32_t>(t);
  p.large_q = cv.take<int32_t>(2 * t);   // the workgroup variant appends without wrapping
  p.max_long = (int64_t)(t / (size_t)(kWaveSegment + 1)) + 1;
  p.long_ids = cv.take<int64_t>((size_t)p.max_long);
  p.long_count = cv.take<unsigned long long>(1);
  p.bytes = cv.used;
  p.sum = cv.take<double>(1);
  p.chunk_sums = cv.take<double>(t / kSumChunk + 1);
  p.runs = cv.take<ChunkRun>(t / kSumChunk + 1);
  p.states = cv.take<ListState>(kMostWideRounds + 1);
  p.flags = cv.take<uint64_t>(t / 64 + 1);
  p.counts = cv.take<int32_t>(t / kLongTrip + 1);
  p.wide_bytes = cv.used;
  return p;
}

static bool wide_segment(int64_t num_segments, int64_t total_entries) {
  return num_segments == 1 && total_entries >= kWideSegment;
}

template <typename OffT>
static int32_t launch_alias_wide(const OffT* seg_offsets, int64_t n, const float* weights, float* prob_out,
                                 int32_t* alias_out, const AliasPlan& p, hipStream_t stream) {
  const unsigned tiles = (unsigned)min((int64_t)2048, ceil_div(n, kLongTrip));
  const int64_t chunks = ceil_div(n, kSumChunk);
  alias_wide_chunks_kernel<OffT><<<(unsigned)min((int64_t)1024, ceil_div(chunks, kLongWaves)), kLongThreads, 0, stream>>>(
      seg_offsets, weights, p.chunk_sums);
  alias_wide_prefix_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, p.chunk_sums);
  alias_wide_runs_kernel<OffT><<<(unsigned)min((int64_t)8192, ceil_div(chunks, 4)), 256, 0, stream>>>(
      seg_offsets, weights, p.chunk_sums, p.runs);
  alias_wide_sum_kernel<OffT><<<1, 256, 0, stream>>>(seg_offsets, weights, p.runs, p.sum);
  alias_wide_masses_kernel<OffT><<<tiles, kLongThreads, 0, stream>>>(seg_offsets, weights, p.sum, p.mass, p.flags, p.counts);
  alias_wide_append_kernel<OffT><<<tiles, kLongThreads, 0, stream>>>(seg_offsets, p.small_q, p.large_q, p.flags, p.counts,
                                                                     p.states, 1);
  GS_LAUNCH_CHECK();
  const int rounds = wide_rounds(n);
  const unsigned half = (unsigned)min((int64_t)2048, ceil_div(n / 2 + 1, kLongTrip));      // m is at most half of n
  for (int r = 0; r < rounds; ++r) {
    alias_wide_round_kernel<OffT><<<half, kLongThreads, 0, stream>>>(seg_offsets, p.sum, prob_out, alias_out, p.mass,
                                                                     p.small_q, p.large_q, p.flags, p.counts, p.states + r);
    alias_wide_append_kernel<OffT><<<half, kLongThreads, 0, stream>>>(seg_offsets, p.small_q, p.large_q, p.flags,
                                                                      p.counts, p.states + r, 0);
    GS_LAUNCH_CHECK();
  }
  alias_build_long_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, nullptr, nullptr, weights, prob_out, alias_out,
                                                                p.mass, p.small_q, p.large_q, p.states + rounds, p.sum);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename OffT>
static int32_t launch_alias_build(const OffT* seg_offsets, int64_t num_segments, int64_t total_entries,
                                  const float* weights, float* prob_out, int32_t* alias_out,
                                  const AliasPlan& p, hipStream_t stream) {
  if (p.sum != nullptr) return launch_alias_wide(seg_offsets, total_entries, weights, prob_out, alias_out, p, stream);
  if (num_segments == 1 && total_entries > kWaveSegment) {
    alias_build_long_kernel<OffT><<<1, kLongThreads, 0, stream>>>(
        seg_offsets, nullptr, nullptr, weights, prob_out, alias_out, p.mass, p.small_q, p.large_q, nullptr, nullptr);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  const int threads = 64;
  alias_build_kernel<OffT><<<(unsigned)ceil_div(num_segments, threads), threads, 0, stream>>>(
      seg_offsets, num_segments, weights, prob_out, alias_out, p.mass, p.small_q, p.large_q);
  GS_LAUNCH_CHECK();
  // few segments: a wave each; many: up to 64 per wave, so that the short ones cost one look
  const int per_wave = (int)max((int64_t)1, min((int64_t)64, num_segments / 16384));
  const unsigned waves = (unsigned)ceil_div(num_segments, per_wave);
  if (total_entries > kLaneSegment) {
    alias_build_wave_kernel<OffT, (int)kLaneSegment + 1, 256><<<waves, 64, 0, stream>>>(
        seg_offsets, num_segments, per_wave, weights, prob_out, alias_out);
    GS_LAUNCH_CHECK();
  }
  if (total_entries > 256) {
    alias_build_wave_kernel<OffT, 257, kWaveSegment><<<waves, 64, 0, stream>>>(
        seg_offsets, num_segments, per_wave, weights, prob_out, alias_out);
    GS_LAUNCH_CHECK();
  }
  // at most this many segments can be longer
  const int64_t max_long = min(num_segments, total_entries / (kWaveSegment + 1));
  if (max_long > 0) {
    zero_u64_kernel<<<1, 1, 0, stream>>>(p.long_count);
    GS_LAUNCH_CHECK();
    alias_find_long_kernel<OffT><<<(unsigned)ceil_div(num_segments, 256), 256, 0, stream>>>(
        seg_offsets, num_segments, p.long_ids, max_long, p.long_count);
    GS_LAUNCH_CHECK();
    alias_build_long_kernel<OffT><<<(unsigned)max_long, kLongThreads, 0, stream>>>(
        seg_offsets, p.long_ids, p.long_count, weights, prob_out, alias_out, p.mass, p.small_q,
        p.large_q, nullptr, nullptr);
    GS_LAUNCH_CHECK();
  }
  return GS_OK;
}

}  // namespace gs

using namespace gs;

extern "C" size_t gs_alias_build_workspace_bytes(int64_t num_segments, int64_t total_entries) {
  if (total_entries < 0) return 0;
  const AliasPlan p = plan_alias(nullptr, total_entries);
  return wide_segment(num_segments, total_entries) ? p.wide_bytes : p.bytes;
}

extern "C" int32_t gs_alias_build(const void* seg_offsets, int32_t offset_bits, int64_t num_segments,
                                  int64_t total_entries, const float* weights, float* prob_out,
                                  int32_t* alias_out, void* ws, size_t ws_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (offset_bits != 32 && offset_bits != 64) return GS_EINVAL;
  if (num_segments < 0 || total_entries < 0 || !seg_offsets) return GS_EINVAL;
  if (total_entries > 0 && (!weights || !prob_out || !alias_out)) return GS_EINVAL;
  if (!ws || !aligned(ws, 256)) return GS_EINVAL;
  AliasPlan p = plan_alias(ws, total_entries);
  if (ws_bytes < p.bytes) return GS_EWORKSPACE;
  if (!wide_segment(num_segments, total_entries) || ws_bytes < p.wide_bytes) p.sum = nullptr;
  // alias[] holds 32-bit positions inside a segment; one segment over everything is the
  // one case the host can see
  if (num_segments == 1 && total_entries > (int64_t)INT32_MAX) return GS_EOVERFLOW;
  if (num_segments == 0 || total_entries == 0) return GS_OK;
  if (offset_bits == 64)
    return launch_alias_build((const int64_t*)seg_offsets, num_segments, total_entries, weights,
                              prob_out, alias_out, p, stream);
  return launch_alias_build((const int32_t*)seg_offsets, num_segments, total_entries, weights, prob_out,
                            alias_out, p, stream);
}

extern "C" int32_t gs_alias_pack(const float* prob, const int32_t* alias, int64_t total_entries,
                                 uint64_t* packed_out, void* stream_) {
  if (total_entries < 0) return GS_EINVAL;
  if (total_entries == 0) return GS_OK;
  if (!prob || !alias || !packed_out || !aligned(packed_out, 8)) return GS_EINVAL;
  alias_pack_kernel<<<(unsigned)ceil_div(total_entries, 256), 256, 0, (hipStream_t)stream_>>>(
      prob, alias, total_entries, packed_out);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
