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
//    binade (at most one per doubling of the sum) are added one by one.  Most weights do without: where
//    every partial sum in any grouping is exact (any_order below), any order gives S.
//  * While the larges are fewer than the smalls, whole runs of rounds are one chain of additions per large
//    (rounds_of_few_larges below).
//
// Segments of up to kLaneSegment entries are built by one lane each, up to kWaveSegment by one wave
// in LDS, longer ones (the rows of hub nodes) by a workgroup of 1024 lanes; a very long one that is
// alone in its call (the noise table) gets its sum, its lists and its first rounds from the whole chip.
// All are bound by latency, so the limits lie where the next larger team finishes the longest segment
// sooner.  Measured on a 1 M-node graph of 22 M weighted entries: row tables 0.76 ms (lanes 0.12, the
// rest, whose longest row takes 0.41, 0.62), 1.9 ms (lanes 0.29, waves 0.20 + 0.45, workgroups 0.92) with a launch per size, lists
// in global memory for the lanes, sums in index order and a look at all lists in every round; the noise table of 1 M entries 0.72 ms (sum 0.02, lists and 16 rounds of the chip 0.18, few
// larges 0.47), 2.5 ms before; that of 4 M nodes 1.6 ms, 7.1 before.
#include <type_traits>

#include "common.h"

namespace gs {

constexpr int64_t kLaneSegment = 32;
constexpr int kWaveSegment = 2048;

// ---- one lane per segment ------------------------------------------------------------------
// Masses and both lists in LDS, entry i of lane l at [i][l].  (In global scratch every step of the loop below
// is a chain of reads of cache lines of its own.)  long_ids: where the segments of more than kWaveSegment entries are
// written to (a launch of its own for that: 10,000 rows of 10 entries 20.6 us, 19.1 like this).
template <typename OffT>
__global__ __launch_bounds__(64) void alias_build_kernel(const OffT* __restrict__ seg_offsets,
                                                         int64_t num_segments,
                                                         const float* __restrict__ weights,
                                                         float* __restrict__ prob_out,
                                                         int32_t* __restrict__ alias_out,
                                                         int64_t* __restrict__ long_ids, int64_t max_long,
                                                         unsigned long long* __restrict__ long_count) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  constexpr int kMost = (int)kLaneSegment;
  static_assert((kMost & (kMost - 1)) == 0, "the list of larges wraps by a mask");
  __shared__ double mass[kMost][64];
  __shared__ uint8_t small_q[kMost][64];       // every entry enters at most once: no wrap
  __shared__ uint8_t large_q[kMost][64];
  const int lane = threadIdx.x;
  const int64_t s = (int64_t)blockIdx.x * 64 + lane;
  if (s >= num_segments) return;
  const int64_t begin = (int64_t)seg_offsets[s];
  const int64_t size = (int64_t)seg_offsets[s + 1] - begin;
  if (size > kWaveSegment && long_ids != nullptr) {
    // max_long bounds the count when the offsets add up to total_entries; an inconsistent pair of arguments must still
    // not write out of bounds
    const unsigned long long at = atomicAdd(long_count, 1ull);
    if (at < (unsigned long long)max_long) long_ids[at] = s;
  }
  if (size <= 0 || size > kLaneSegment) return;
  const int n = (int)size;
  const float* w = weights + begin;
  float* prob = prob_out + begin;
  int32_t* alias = alias_out + begin;

  double S = 0.0;
  const double dn = (double)n;
  for (int i0 = 0; i0 < n; i0 += 4) {          // (four reads under way at a time)
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = w[min(i0 + k, n - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k >= n) break;
      S += (double)v[k];
      mass[i0 + k][lane] = (double)v[k] * dn;
    }
  }
  int small_head = 0, small_tail = 0, large_head = 0, large_tail = 0;
  for (int i = 0; i < n; ++i) {
    if (mass[i][lane] < S) small_q[small_tail++][lane] = (uint8_t)i;
    else large_q[large_tail++][lane] = (uint8_t)i;
  }
  while (small_head < small_tail && large_head < large_tail) {
    const int a = small_q[small_head++][lane];
    const int b = large_q[large_head++ & (kMost - 1)][lane];
    const double ma = mass[a][lane];
    prob[a] = (float)(ma / S);
    alias[a] = b;
    const double mb = (mass[b][lane] + ma) - S;
    mass[b][lane] = mb;
    if (mb < S) small_q[small_tail++][lane] = (uint8_t)b;
    else large_q[large_tail++ & (kMost - 1)][lane] = (uint8_t)b;
  }
  for (; small_head < small_tail; ++small_head) {
    const int i = small_q[small_head][lane];
    prob[i] = 1.0f;
    alias[i] = i;
  }
  for (; large_head < large_tail; ++large_head) {
    const int i = large_q[large_head & (kMost - 1)][lane];
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

// Sums that no order changes.  Every weight is a whole multiple of u = 2^(least exponent - 23); while the sum of the
// weights stays below 2^53 u, every partial sum in every grouping is a whole number of units below 2^53,
// which fp64 holds exactly, so any order gives the index-order sum.  (The check is sound on the computed
// sum: rounding is monotonic, so a partial sum that reached 2^53 u would leave the result there.)  Weights of 1 and more with
// a sum below 2^30 pass, as do lognormal weights of a few million entries.
// The exponent field of a weight; of zeros (multiples of anything) the largest; 0 only for weights below zero
__device__ __forceinline__ int weight_exponent(float v) {
  const uint32_t bits = __float_as_uint(v);
  if ((bits & 0x7fffffffu) == 0u) return 255;
  if (bits >> 31) return 0;
  return max(1, (int)(bits >> 23));
}
__device__ __forceinline__ bool any_order(double sum, int least_exponent) {      // (false for infinities and NaN)
  return least_exponent > 0 &&
         sum < __longlong_as_double((long long)(uint64_t)(least_exponent - 127 - 23 + 53 + 1023) << 52);
}

// ---- one wave per segment --------------------------------------------------------------------
// A segment of n <= MAX_N entries: masses and both lists in LDS, up to 64 iterations at a time.
template <int MAX_N>
struct WaveLists {
  double mass[MAX_N];
  uint16_t small_q[MAX_N];                     // every entry enters at most once: no wrap
  uint16_t large_q[MAX_N];
};
template <int MAX_N>
__device__ __forceinline__ void wave_segment(WaveLists<MAX_N>& lists, int lane, int n, const float* __restrict__ w,
                                             float* __restrict__ prob, int32_t* __restrict__ alias) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  static_assert((MAX_N & (MAX_N - 1)) == 0, "the list of larges wraps by a mask");
  double* mass = lists.mass;
  uint16_t *small_q = lists.small_q, *large_q = lists.large_q;
  const uint64_t below = (1ull << lane) - 1ull;
  const double dn = (double)n;
  double S = 0.0;
  int least = 255;
  for (int base = lane; base < n; base += 64) {
    const float v = w[base];
    mass[base] = (double)v * dn;
    S += (double)v;
    least = min(least, weight_exponent(v));
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    S += __shfl_xor(S, d, 64);
    least = min(least, __shfl_xor(least, d, 64));
  }
  if (!any_order(S, least)) {
    S = 0.0;
    for (int base = 0; base < n; base += 64) {
      const double v = base + lane < n ? (double)w[base + lane] : 0.0;
#pragma unroll 16
      for (int k = 0; k < 64; ++k) S += lane_value(v, k);       // (+ 0.0 behind the end changes nothing)
    }
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
      alias[a] = b;
      const double mb = (mass[b] + mass[a]) - S;
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
  // (a small's mass does not change once it is one: the divisions are left to all lanes)
  for (int i = lane; i < sh; i += 64) {
    const int a = small_q[i];
    prob[a] = (float)(mass[a] / S);
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

// Segments of MIN_N .. MAX_N entries; a wave looks at `per_wave` consecutive segments and takes those of its size.
// unless: nothing is done where this holds a number other than 0.
template <typename OffT, int MIN_N, int MAX_N>
__global__ __launch_bounds__(64) void alias_build_wave_kernel(const OffT* __restrict__ seg_offsets,
                                                              int64_t num_segments, int per_wave,
                                                              const unsigned long long* __restrict__ unless,
                                                              const float* __restrict__ weights,
                                                              float* __restrict__ prob_out,
                                                              int32_t* __restrict__ alias_out) {
  if (unless != nullptr && *unless != 0ull) return;
  __shared__ WaveLists<MAX_N> lists;
  const int lane = threadIdx.x;
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
    wave_segment<MAX_N>(lists, lane, n, weights + begin, prob_out + begin, alias_out + begin);
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
  int least = 255;
  for (int64_t base = threadIdx.x; base < n; base += 4 * kLongThreads) {
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = base + k * kLongThreads < n ? w[base + k * kLongThreads] : 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      S += (double)v[k];
      least = min(least, weight_exponent(v[k]));
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    S += __shfl_xor(S, d, 64);
    least = min(least, __shfl_xor(least, d, 64));
  }
  if (lane == 0) { run_s[wave].even = __double_as_longlong(S); run_s[wave].odd = least; }
  __syncthreads();
  S = 0.0;
#pragma unroll
  for (int v = 0; v < kLongWaves; ++v) {
    S += __longlong_as_double(run_s[v].even);
    least = min(least, (int)run_s[v].odd);
  }
  __syncthreads();
  if (any_order(S, least)) return S;
  S = 0.0;
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

// A barrier for what the waves exchange through LDS alone: it does not wait for stores to global memory.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// places of the wave's votes in the workgroup's order, for two kinds of votes at once: c0 and c1
// are the wave's totals; returns the totals of the waves before, and all of them
__device__ __forceinline__ void block_before(int c0, int c1, int (*tot)[kLongWaves], int& before0, int& before1,
                                             int& all0, int& all1) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if ((threadIdx.x & 63) == 0) { tot[0][wave] = c0; tot[1][wave] = c1; }
  lds_barrier();
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
// two kernels: iterate, then append behind both lists), and the rest from one workgroup.
// Rounds narrower than kWideRound are left to that one: what it keeps in registers.  Measured in ms, degree^0.75 of a skewed graph and
// lognormal weights: the whole chip against one workgroup, 2^15 entries 0.25 / 0.17 and 0.22 / 0.16, 2^16 0.29 / 0.26 and
// 0.26 / 0.25, 2^17 0.35 / 0.43 and 0.30 / 0.41, 2^18 0.41 / 0.85 and 0.36 / 0.82.  Of the launches, those behind the last wide
// round cost 3 to 4 us a round, and a wide round that is left to one workgroup 30 and more: 16, 32 and 96 rounds 1 M entries
// 0.67, 0.72, 0.93 and 0.51, 0.56, 0.78; 2 M 2.32, 0.94, 1.16 and 1.06, 0.68, 0.89; 4 M 4.67, 3.61, 1.62 and 2.87, 1.87, 2.09; 8 M
// 9.23, 7.44, 5.32 (256 rounds 4.00) and 5.32, 3.91, 3.60 (4.42).
struct ListState { int64_t sh, st, lh, lt; };
constexpr int64_t kWideSegment = (int64_t)1 << 17;
// Workgroups of the chip-wide kernels: small ones, so that the scattered accesses of a round spread over all compute
// units, while every workgroup can still add up the counts of the tiles before its own.  Milliseconds, 256 against 1024
// threads, lognormal weights and degree^0.75: 0.3 M entries 0.35 / 0.39 and 1.18 / 1.20, 2 M 0.66 / 0.84 and 2.15 / 2.30, 8 M 3.31 / 3.81
// and 3.85 / 4.38, 32 M 9.74 / 10.9 and 25.9 / 27.5, 64 M 18.7 / 19.7 and 51.7 / 52.4, 128 M 37.5 / 37.2 and 106.3 / 106.1.
constexpr int kWideThreads = 256, kWideTile = kWideThreads * kLongItems;
constexpr int64_t kWideSmallTiles = (int64_t)1 << 26;          // entries
constexpr int64_t kWideRound = 8192;
static int wide_rounds(int64_t n) {
  return n < (int64_t)3 << 19 ? 16 : (n < (int64_t)3 << 20 ? 32 : (n < (int64_t)3 << 21 ? 96 : 128));
}
constexpr int kMostWideRounds = 128;

struct ChunkRun { Runs run; int e; int good; };
// The sum: plain sums of the chunks and their prefix sums, which end in the total.  Where the order of the additions
// does not matter (any_order) that is the sum, and the next two kernels return at once.  Else in three steps: plain sums of the chunks, their prefix sums (which name the binade that the
// running sum is in when it reaches a chunk, but for those next to a border), and the run of every
// chunk for that binade; then one workgroup adds run after run, and one by one where the binade was not
// the one or is left.
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_chunks_kernel(const OffT* __restrict__ seg_offsets,
                                                                         const float* __restrict__ weights,
                                                                         double* __restrict__ chunk_sums,
                                                                         ChunkRun* __restrict__ runs) {
  const int lane = threadIdx.x & 63;
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const int64_t waves = (int64_t)gridDim.x * kLongWaves;
  for (int64_t c = (int64_t)blockIdx.x * kLongWaves + (threadIdx.x >> 6); c * kSumChunk < n; c += waves) {
    double sum = 0.0;
    int least = 255;
#pragma unroll
    for (int k = 0; k < kSumItems; ++k) {
      const int64_t i = c * kSumChunk + k * 64 + lane;
      const float v = i < n ? weights[begin + i] : 0.f;
      sum += (double)v;
      least = min(least, weight_exponent(v));
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      sum += __shfl_xor(sum, d, 64);
      least = min(least, __shfl_xor(least, d, 64));
    }
    if (lane == 0) { chunk_sums[c] = sum; runs[c].e = least; }
  }
}

template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_prefix_kernel(const OffT* __restrict__ seg_offsets,
                                                                         double* __restrict__ chunk_sums,
                                                                         const ChunkRun* __restrict__ runs,
                                                                         double* __restrict__ sum_out,
                                                                         int32_t* __restrict__ summed) {
  __shared__ double part[2][kLongWaves];
  __shared__ int least_s[kLongWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = (int64_t)seg_offsets[1] - (int64_t)seg_offsets[0], chunks = (n + kSumChunk - 1) / kSumChunk;
  double carry = 0.0;
  int turn = 0, least = 255;
  for (int64_t base = 0; base < chunks; base += kLongThreads, turn ^= 1) {
    const int64_t c = base + threadIdx.x;
    const double own = c < chunks ? chunk_sums[c] : 0.0;
    if (c < chunks) least = min(least, runs[c].e);
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
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) least = min(least, __shfl_xor(least, d, 64));
  if (lane == 0) least_s[wave] = least;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < kLongWaves; ++w) least = min(least, least_s[w]);
    const bool done = any_order(carry, least);
    if (done) *sum_out = carry;
    *summed = done ? 1 : 0;
  }
}

template <typename OffT>
__global__ __launch_bounds__(256) void alias_wide_runs_kernel(const OffT* __restrict__ seg_offsets,
                                                              const float* __restrict__ weights,
                                                              const double* __restrict__ chunk_sums,
                                                              ChunkRun* __restrict__ runs,
                                                              const int32_t* __restrict__ summed) {
  if (*summed != 0) return;
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
                                                             double* __restrict__ sum_out,
                                                             const int32_t* __restrict__ summed) {
  if (*summed != 0) return;
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
template <int kThreads>
__device__ __forceinline__ int64_t counts_before(const int32_t* __restrict__ counts, int64_t tile, int64_t* part) {
  int64_t sum = 0;
  for (int64_t i = threadIdx.x; i < tile; i += kThreads) sum += counts[i];
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) sum += part[w];
  return sum;
}

// masses, and which entries start as smalls: a bit per entry and a count per tile
template <typename OffT, int kThreads>
__global__ __launch_bounds__(kThreads) void alias_wide_masses_kernel(const OffT* __restrict__ seg_offsets,
                                                                         const float* __restrict__ weights,
                                                                         const double* __restrict__ sum, double* mass_ws,
                                                                         uint64_t* __restrict__ flags,
                                                                         int32_t* __restrict__ counts) {
#pragma clang fp contract(off)
  __shared__ int32_t tot[kThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t begin = (int64_t)seg_offsets[0], n = (int64_t)seg_offsets[1] - begin;
  const double S = *sum, dn = (double)n;
  for (int64_t tile = blockIdx.x; tile * kThreads * kLongItems < n; tile += gridDim.x) {
    const int64_t first = tile * kThreads * kLongItems + wave * (64 * kLongItems);
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
      for (int w = 0; w < kThreads / 64; ++w) all += tot[w];
      counts[tile] = all;
    }
    __syncthreads();
  }
}

// Appends entries 0 .. m - 1 (entry i is i itself, or large_q[lh + i]) behind the smalls or the larges, in
// order, by their flags; the workgroup with the last tile writes the lists' next state.
// initial: the lists are empty and the entries are the segment's.
template <typename OffT, int kThreads>
__global__ __launch_bounds__(kThreads) void alias_wide_append_kernel(const OffT* __restrict__ seg_offsets,
                                                                         int32_t* small_ws, int32_t* large_ws,
                                                                         const uint64_t* __restrict__ flags,
                                                                         const int32_t* __restrict__ counts,
                                                                         ListState* __restrict__ states, int initial) {
  __shared__ int64_t part[kThreads / 64];
  __shared__ int32_t tot[kThreads / 64];
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
  const int64_t tiles = (m + kThreads * kLongItems - 1) / (kThreads * kLongItems);
  if (tiles == 0 && blockIdx.x == 0 && threadIdx.x == 0) states[0] = at;     // (an empty segment)
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t before = counts_before<kThreads>(counts, tile, part);
    const int64_t first = tile * kThreads * kLongItems + wave * (64 * kLongItems);
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
    for (int w = 0; w < kThreads / 64; ++w) {
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
template <typename OffT, int kThreads>
__global__ __launch_bounds__(kThreads) void alias_wide_round_kernel(
    const OffT* __restrict__ seg_offsets, const double* __restrict__ sum, float* __restrict__ prob_out,
    int32_t* __restrict__ alias_out, double* mass_ws, const int32_t* __restrict__ small_ws,
    const int32_t* __restrict__ large_ws, uint64_t* __restrict__ flags, int32_t* __restrict__ counts,
    const ListState* __restrict__ states) {
#pragma clang fp contract(off)
  __shared__ int32_t tot[kThreads / 64];
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
  for (int64_t tile = blockIdx.x; tile * kThreads * kLongItems < m; tile += gridDim.x) {
    const int64_t first = tile * kThreads * kLongItems + wave * (64 * kLongItems);
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
      for (int w = 0; w < kThreads / 64; ++w) all += tot[w];
      counts[tile] = all;
    }
    __syncthreads();
  }
}

// ---- rounds of few larges -------------------------------------------------------------------
// While there are no more larges than smalls, a round gives every large the next small: large i of l takes the smalls i, i + l,
// i + 2l, ... of the list, until one of the larges has become a small.  So the workgroup keeps the larges in
// registers and the head of the smalls in LDS, and every large runs down its own smalls, a chain of two
// additions per round, with nothing to agree on but the first round in which any of them drops below S.
// After that round the larges that are left close up, in order.  Up to 64 larges are one wave's, which needs no barriers.
// A noise table of 1 M entries (degree^0.75 of a skewed graph) has 1486 rounds of fewer than 8192 larges, all but
// 120 of them without a large that drops out: 1.77 ms with a look at both lists in every round, 0.47 ms like this, bound
// by the instructions of one compute unit (23 rounds of more than 2048 larges 0.10 ms, 232 of more than 64 0.23, the rest 0.11).
//
// A compute unit moves about one cache line per cycle, so for a segment alone in its call (kAlone) the scattered
// accesses of these rounds, a mass in and a probability and an alias out per small, are left to the whole chip: before,
// the masses of the smalls are brought into the order of the list (mass_seq), after, what each small was paired with
// (alias_seq) becomes the table.
constexpr int kBigItems = 2, kBigItemsAlone = 8;               // larges per lane
constexpr int kBig = kLongThreads * kBigItems, kBigAlone = kLongThreads * kBigItemsAlone;
constexpr int kBigRounds = 8;                                  // rounds between two looks at the others
constexpr int kBigRoundsOneWave = 16;
// smalls in LDS: 74 KB for a workgroup that does one row of several (in the launch that has the shorter rows' lists too, 152 KB,
// one workgroup per compute unit: 256 rows of 3000 entries 76 us, 300 123; 200 and 268 with a look at both lists in every round
// and two workgroups per compute unit), or most of a compute unit's for a segment alone
constexpr int kWindow = 3072, kWindowAlone = 12288;
static_assert(kWindow >= kBig && kWindow % kLongThreads == 0 && kWindowAlone % kLongThreads == 0, "a round fits the window");
static_assert(kWindowAlone * sizeof(double) >= kBigAlone * (sizeof(double) + sizeof(int32_t)), "or the larges of the wider rounds");
static_assert(kBigAlone >= kWideRound, "what the chip leaves");
struct RowWindow {
  int32_t id[kWindow];                         // the smalls
  int32_t alias[kWindow];                      // the large that takes each of them
};
struct NoRowWindow {};
template <bool kAlone>
struct BigRounds {
  double mass[kAlone ? kWindowAlone : kWindow];          // of the smalls
  double big_mass[kBig];                       // the larges, where they close up
  int32_t big_id[kBig];
  std::conditional_t<kAlone, NoRowWindow, RowWindow> row;
  int first_event[4];                          // (four, used in turn: a slot is reset two turns ahead of its use)
  int state[4];                                // one wave's rounds: smalls taken, larges left, smalls appended
};

// The larges of all lanes after a round: those below S to the smalls, the others closed up in big_id / big_mass.  Lane's
// larges: mine, mine + 64, ...  Returns larges left and (in demoted) smalls appended.
template <bool kAlone, int ITEMS>
__device__ __forceinline__ int close_up(int32_t* big_id, double* big_mass, const double S, int l, int mine,
                                        const int32_t (&id)[ITEMS], const double (&m)[ITEMS], int64_t st, int32_t* small_q,
                                        double* mass, double* mass_seq, int (*tot)[kLongWaves], int& demoted) {
  const int lane = threadIdx.x & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  const bool busy = __builtin_amdgcn_readfirstlane(mine - lane) < l;
  uint64_t down[ITEMS], stay[ITEMS];
  int cd = 0, cs = 0;
  if (busy) {
#pragma unroll
    for (int c = 0; c < ITEMS; ++c) {
      const bool valid = mine + c * 64 < l;
      down[c] = __ballot(valid && m[c] < S);
      stay[c] = __ballot(valid && !(m[c] < S));
      cd += __popcll(down[c]);
      cs += __popcll(stay[c]);
    }
  }
  int bd, bs, left;
  block_before(cd, cs, tot, bd, bs, demoted, left);
  if (!busy) return left;
#pragma unroll
  for (int c = 0; c < ITEMS; ++c) {
    if ((down[c] >> lane) & 1ull) {
      const int64_t to = st + bd + __popcll(down[c] & below);
      small_q[to] = id[c];
      mass[id[c]] = m[c];
      if (kAlone) mass_seq[to] = m[c];
    } else if ((stay[c] >> lane) & 1ull) {
      const int to = bs + __popcll(stay[c] & below);
      big_id[to] = id[c];
      big_mass[to] = m[c];
    }
    bd += __popcll(down[c]);
    bs += __popcll(stay[c]);
  }
  return left;
}

template <bool kAlone>
__device__ void rounds_of_few_larges(BigRounds<kAlone>& b, const double S, float* prob, int32_t* alias, double* mass,
                                     double* mass_seq, int32_t* alias_seq, int32_t* small_q, int32_t* large_q, int64_t& sh,
                                     int64_t& st, int64_t& lh, int64_t& lt, int (*tot)[2][kLongWaves]) {
#pragma clang fp contract(off)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t below = (1ull << lane) - 1ull;
  int l = (int)(lt - lh);
  int turn = 0, votes_turn = 0;
  bool closed_up = false;                                      // the larges are in wide_id / wide_mass, not in the list
  double* wide_mass = b.mass;                                  // (the window's place)
  int32_t* wide_id = kAlone ? reinterpret_cast<int32_t*>(b.mass + kBigAlone) : nullptr;
  if constexpr (kAlone) {
    // more larges than two per lane: round by round, the smalls straight from memory
    if (l > kBig && st - sh >= l) {
      const int mine = wave * (64 * kBigItemsAlone) + lane;
      if (tid < 4) b.first_event[tid] = 0;
      __syncthreads();
      int32_t id[kBigItemsAlone];
      double m[kBigItemsAlone];
#pragma unroll
      for (int c = 0; c < kBigItemsAlone; ++c) id[c] = large_q[lh + min(mine + c * 64, l - 1)];
#pragma unroll
      for (int c = 0; c < kBigItemsAlone; ++c) m[c] = mass[id[c]];
      int64_t written = st;                                    // the smalls up to here are there for all lanes
      while (l > kBig && st - sh >= l) {
        double v[kBigItemsAlone];
        bool event = false;
        if (sh + l > written) {
          __syncthreads();
          written = st;
        }
        if (wave * (64 * kBigItemsAlone) < l) {                // (waves without larges leave the issue slots to the others)
#pragma unroll
          for (int c = 0; c < kBigItemsAlone; ++c) v[c] = mass_seq[sh + min(mine + c * 64, l - 1)];
#pragma unroll
          for (int c = 0; c < kBigItemsAlone; ++c) {
            m[c] = (m[c] + v[c]) - S;
            if (mine + c * 64 < l) {
              alias_seq[sh + mine + c * 64] = id[c];
              event = event || m[c] < S;
            }
          }
        }
        sh += l;
        if (__ballot(event) != 0ull && lane == 0) b.first_event[turn & 3] = 1;
        if (tid == 0) b.first_event[(turn + 2) & 3] = 0;
        lds_barrier();
        const bool any = b.first_event[turn & 3] != 0;
        ++turn;
        if (!any) continue;
        int demoted;
        l = close_up<kAlone, kBigItemsAlone>(wide_id, wide_mass, S, l, mine, id, m, st, small_q, mass, mass_seq, tot[votes_turn], demoted);
        votes_turn ^= 1;
        st += demoted;
        closed_up = true;
        lds_barrier();
        if (wave * (64 * kBigItemsAlone) < l) {
#pragma unroll
          for (int c = 0; c < kBigItemsAlone; ++c) {
            const int at = min(mine + c * 64, l - 1);
            id[c] = wide_id[at];
            m[c] = wide_mass[at];
          }
        }
        lds_barrier();
      }
      if (l > kBig) {                                          // (too few smalls)
#pragma unroll
        for (int c = 0; c < kBigItemsAlone; ++c)
          if (mine + c * 64 < l) {
            large_q[lt + mine + c * 64] = id[c];
            mass[id[c]] = m[c];
          }
        lh = lt;
        lt += l;
        return;
      }
    }
  }
  const int mine = wave * (64 * kBigItems) + lane;             // this lane's larges: mine, mine + 64
  int32_t id[kBigItems];
  double m[kBigItems];
#pragma unroll
  for (int c = 0; c < kBigItems; ++c) {
    const bool valid = mine + c * 64 < l;
    id[c] = !valid ? 0 : (closed_up ? wide_id[mine + c * 64] : large_q[lh + mine + c * 64]);
    m[c] = !valid ? 0.0 : (closed_up ? wide_mass[mine + c * 64] : mass[id[c]]);
  }
  constexpr int kSmalls = kAlone ? kWindowAlone : kWindow;
  if (kAlone) __syncthreads();                                 // (the flags' last use above)
  if (tid < 4) b.first_event[tid] = kBigRounds;
  while (l > 0 && st - sh >= l) {
    const int count = (int)min((int64_t)kSmalls, st - sh);
    __syncthreads();                                           // (what was appended is there)
    if constexpr (kAlone) {
#pragma unroll
      for (int c = 0; c < kSmalls / kLongThreads; ++c)         // (behind the end: the last one again, not used)
        b.mass[c * kLongThreads + tid] = mass_seq[sh + min(c * kLongThreads + tid, count - 1)];
    } else {
      int32_t a[kWindow / kLongThreads];
#pragma unroll
      for (int c = 0; c < kWindow / kLongThreads; ++c) a[c] = small_q[sh + min(c * kLongThreads + tid, count - 1)];
#pragma unroll
      for (int c = 0; c < kWindow / kLongThreads; ++c) {
        b.row.id[c * kLongThreads + tid] = a[c];
        b.mass[c * kLongThreads + tid] = mass[a[c]];
      }
    }
    __syncthreads();
    int at = 0;                                                // smalls of the window that have been taken
    // (of rounds behind an event: written again)
    auto pair = [&](int small, int32_t large) {
      if constexpr (kAlone) alias_seq[sh + small] = large;
      else b.row.alias[small] = large;
    };
    while (l > 64 && count - at >= l) {
      const int rounds = min(kBigRounds, (count - at) / l);
      double v[kBigRounds][kBigItems], x[kBigItems];
      int event = kBigRounds;
#pragma unroll
      for (int c = 0; c < kBigItems; ++c) x[c] = m[c];
      const bool busy = wave * (64 * kBigItems) < l;           // (waves without larges leave the issue slots to the others)
      if (busy) {
#pragma unroll
        for (int j = 0; j < kBigRounds; ++j)
#pragma unroll
          for (int c = 0; c < kBigItems; ++c)
            v[j][c] = b.mass[min(at + j * l + mine + c * 64, kSmalls - 1)];
#pragma unroll
        for (int j = 0; j < kBigRounds; ++j) {
          if (j >= rounds) break;
#pragma unroll
          for (int c = 0; c < kBigItems; ++c) {
            x[c] = (x[c] + v[j][c]) - S;
            if (mine + c * 64 < l) {
              if (x[c] < S) event = min(event, j);
              pair(at + j * l + mine + c * 64, id[c]);
            }
          }
        }
      }
      if (event < kBigRounds) atomicMin(&b.first_event[turn & 3], event);
      if (tid == 0) b.first_event[(turn + 2) & 3] = kBigRounds;
      lds_barrier();
      event = __builtin_amdgcn_readfirstlane(b.first_event[turn & 3]);
      ++turn;
      if (event == kBigRounds) {
#pragma unroll
        for (int c = 0; c < kBigItems; ++c) m[c] = x[c];
        at += rounds * l;
        continue;
      }
      // up to and with the round of the event once more; the larges that are left close up
      if (busy) {
#pragma unroll
        for (int j = 0; j < kBigRounds; ++j) {
          if (j > event) break;
#pragma unroll
          for (int c = 0; c < kBigItems; ++c) m[c] = (m[c] + v[j][c]) - S;
        }
      }
      at += (event + 1) * l;
      int demoted;
      l = close_up<kAlone, kBigItems>(b.big_id, b.big_mass, S, l, mine, id, m, st, small_q, mass, mass_seq, tot[votes_turn], demoted);
      votes_turn ^= 1;
      st += demoted;
      lds_barrier();
#pragma unroll
      for (int c = 0; c < kBigItems; ++c)
        if (mine + c * 64 < l) { id[c] = b.big_id[mine + c * 64]; m[c] = b.big_mass[mine + c * 64]; }
    }
    if (l > 0 && l <= 64 && count - at >= l) {
      if (wave == 0) {
        int appended = 0;
        int32_t own = id[0];
        double x = m[0];
        while (l > 0 && count - at >= l) {
          const int rounds = min(kBigRoundsOneWave, (count - at) / l);
          double v[kBigRoundsOneWave];
#pragma unroll
          for (int j = 0; j < kBigRoundsOneWave; ++j) v[j] = b.mass[min(at + j * l + lane, kSmalls - 1)];
          // the chain first, then the votes on all of its rounds, which do not wait for one another
          double y[kBigRoundsOneWave];
          uint32_t events = 0u;
#pragma unroll
          for (int j = 0; j < kBigRoundsOneWave; ++j) y[j] = x = (x + v[j]) - S;
#pragma unroll
          for (int j = 0; j < kBigRoundsOneWave; ++j) events |= __ballot(lane < l && y[j] < S) != 0ull ? 1u << j : 0u;
          const int event = min(rounds, events != 0u ? __builtin_ctz(events) : kBigRoundsOneWave);
          const int taken = min(rounds, event + 1);
#pragma unroll
          for (int j = 0; j < kBigRoundsOneWave; ++j) {
            if (j >= taken) break;
            x = y[j];
            if (lane < l) pair(at + j * l + lane, own);
          }
          at += taken * l;
          if (event == rounds) continue;
          const uint64_t down = __ballot(lane < l && x < S);
          const uint64_t stay = __ballot(lane < l && !(x < S));
          if ((down >> lane) & 1ull) {
            const int64_t to = st + appended + __popcll(down & below);
            small_q[to] = own;
            mass[own] = x;
            if (kAlone) mass_seq[to] = x;
          } else if ((stay >> lane) & 1ull) {
            const int to = __popcll(stay & below);
            b.big_id[to] = own;
            b.big_mass[to] = x;
          }
          appended += __popcll(down);
          l = __popcll(stay);
          wave_fence();
          if (lane < l) { own = b.big_id[lane]; x = b.big_mass[lane]; }
          wave_fence();
        }
        id[0] = own;
        m[0] = x;
        if (lane == 0) { b.state[0] = at; b.state[1] = l; b.state[2] = appended; }
      }
      __syncthreads();
      at = __builtin_amdgcn_readfirstlane(b.state[0]);
      l = __builtin_amdgcn_readfirstlane(b.state[1]);
      st += __builtin_amdgcn_readfirstlane(b.state[2]);
    }
    if constexpr (!kAlone) {
      __syncthreads();
      for (int k = tid; k < at; k += kLongThreads) {
        const int32_t a = b.row.id[k];
        prob[a] = (float)(b.mass[k] / S);
        alias[a] = b.row.alias[k];
      }
    }
    sh += at;
  }
#pragma unroll
  for (int c = 0; c < kBigItems; ++c)
    if (mine + c * 64 < l) {
      large_q[lt + mine + c * 64] = id[c];
      mass[id[c]] = m[c];
    }
  lh = lt;
  lt += l;
}

// Between the chip-wide rounds and the workgroup kernel, which does what these leave.  All for segment 0.
__device__ __forceinline__ bool few_larges(const ListState& at) {
  return at.lt > at.lh && at.lt - at.lh <= (int64_t)kBigAlone && at.lt - at.lh <= at.st - at.sh;
}
template <typename OffT>
__global__ __launch_bounds__(256) void alias_wide_gather_kernel(const OffT* __restrict__ seg_offsets,
                                                                const double* __restrict__ mass_ws,
                                                                const int32_t* __restrict__ small_ws,
                                                                const ListState* __restrict__ states,
                                                                double* __restrict__ mass_seq) {
  const ListState at = states[0];
  if (!few_larges(at)) return;
  const int64_t begin = (int64_t)seg_offsets[0];
  for (int64_t k = at.sh + (int64_t)blockIdx.x * 256 + threadIdx.x; k < at.st; k += (int64_t)gridDim.x * 256)
    mass_seq[k] = mass_ws[begin + small_ws[begin + k]];
}
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_wide_tail_kernel(const OffT* __restrict__ seg_offsets,
                                                                       const double* __restrict__ sum, double* mass_ws,
                                                                       int32_t* small_ws, int32_t* large_ws, double* mass_seq,
                                                                       int32_t* alias_seq, ListState* states) {
  __shared__ BigRounds<true> big;
  __shared__ int tot[2][2][kLongWaves];
  ListState at = states[0];
  if (few_larges(at)) {
    const int64_t begin = (int64_t)seg_offsets[0];
    rounds_of_few_larges<true>(big, *sum, nullptr, nullptr, mass_ws + begin, mass_seq, alias_seq, small_ws + begin,
                               large_ws + 2 * begin, at.sh, at.st, at.lh, at.lt, tot);
  }
  if (threadIdx.x == 0) states[1] = at;
}
// the smalls that the tail took: positions states[0].sh .. states[1].sh of the list
template <typename OffT>
__global__ __launch_bounds__(256) void alias_wide_table_kernel(const OffT* __restrict__ seg_offsets,
                                                               const double* __restrict__ sum,
                                                               const int32_t* __restrict__ small_ws,
                                                               const double* __restrict__ mass_seq,
                                                               const int32_t* __restrict__ alias_seq,
                                                               const ListState* __restrict__ states,
                                                               float* __restrict__ prob_out, int32_t* __restrict__ alias_out) {
#pragma clang fp contract(off)
  const int64_t begin = (int64_t)seg_offsets[0], last = states[1].sh;
  const double S = *sum;
  for (int64_t k = states[0].sh + (int64_t)blockIdx.x * 256 + threadIdx.x; k < last; k += (int64_t)gridDim.x * 256) {
    const int32_t a = small_ws[begin + k];
    prob_out[begin + a] = (float)(mass_seq[k] / S);
    alias_out[begin + a] = alias_seq[k];
  }
}

struct LongShared {
  Runs run_s[kLongWaves];
  uint32_t bad_s[kLongWaves];
  double sum_s;
  int tot[2][2][kLongWaves];                   // (two sets, used in turn: one barrier per use)
  int64_t q_s[4];                              // small head/tail, large head/tail after a narrow stretch
  BigRounds<false> big;
};
// One segment by the workgroup.  resume != null: its sum and lists exist already.
// Scratch per entry of the segment, at the segment's own offsets: mass, the
// small list (n entries), the large list (2n: appended without wrapping).
template <typename OffT>
__device__ __forceinline__ void long_segment(LongShared& shared, const OffT* __restrict__ seg_offsets, int64_t seg,
                                             const float* __restrict__ weights, float* __restrict__ prob_out,
                                             int32_t* __restrict__ alias_out, double* mass_ws, int32_t* small_ws,
                                             int32_t* large_ws, const ListState* __restrict__ resume,
                                             const double* __restrict__ sum) {
#pragma clang fp contract(off)  // every fp64 operation below must round on its own
  auto& run_s = shared.run_s;
  auto& bad_s = shared.bad_s;
  auto& sum_s = shared.sum_s;
  auto& tot = shared.tot;
  auto& q_s = shared.q_s;
  auto& big = shared.big;
  static_assert(kWindow >= 2 * kRing, "the rings lie in the window");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
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
    if (lt - lh <= (int64_t)kBig && lt - lh <= st - sh) {
      rounds_of_few_larges<false>(big, S, prob, alias, mass, nullptr, nullptr, small_q, large_q, sh, st, lh, lt, tot);
      continue;
    }
    if (m < kNarrow) {
      const int64_t popped = sh;               // the smalls from here on are taken in this stretch
      if (wave == 0) {
        Window s = {big.row.id, big.mass, uniform64(sh), uniform64(sh), uniform64(st)};
        Window l = {big.row.id + kRing, big.mass + kRing, uniform64(lh), uniform64(lh), uniform64(lt)};
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

// the single segment 0
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_build_long_kernel(const OffT* __restrict__ seg_offsets,
                                                                        const float* __restrict__ weights,
                                                                        float* __restrict__ prob_out,
                                                                        int32_t* __restrict__ alias_out, double* mass_ws,
                                                                        int32_t* small_ws, int32_t* large_ws,
                                                                        const ListState* __restrict__ resume,
                                                                        const double* __restrict__ sum) {
  __shared__ LongShared shared;
  long_segment<OffT>(shared, seg_offsets, 0, weights, prob_out, alias_out, mass_ws, small_ws, large_ws, resume, sum);
}

// All segments of 33 to 1024 entries and the long ones: the first `long_blocks` workgroups take the long ones, each of the
// others the segments of its size among `per_block` consecutive ones, a wave per segment, whichever wave is free.
// One launch, because the longest row of a skewed graph keeps one compute unit busy while the others wait for work.  R-MAT graphs,
// whole calls, one launch per size against this: 10,000 nodes 145 / 109 us, 100,000 257 / 195, 300,000 (4 M edges) 396 / 296, 1 M
// (10 M edges) 967 / 847.  But a compute unit holds 16 of these waves, and 32 that take 33 to 256 entries alone: without a long
// row (200,000 rows of 100 entries 386 us, 453 from here) the segments are left to launches of their own.  The number of
// long rows is known to the device alone, so both are launched, and the waves of the one that is not to be return.
constexpr int kRowsMiddle = 256, kRowsMost = 1024;
// waves whose lists hold kRowsMost entries; the others' hold kRowsMiddle (7, 11 and 12 of them: 20,000 rows of 500 beside 5 of 3000 268,
// 210, 208 us, 2000 of 1000 beside those 88, 75, 73, R-MAT of 1 M nodes 787, 755, 756; 12 fill the LDS)
constexpr int kRowsWideWaves = 12;
constexpr int kRowsPerBlock = 512;
constexpr int64_t kRowsLongBlocks = 1024;
struct RowsShared {
  WaveLists<kRowsMost> wide[kRowsWideWaves];
  WaveLists<kRowsMiddle> narrow[kLongWaves - kRowsWideWaves];
  uint16_t wide_seg[kRowsPerBlock], narrow_seg[kRowsPerBlock];
  int wide_count, narrow_count, wide_next, narrow_next;
};
static_assert(sizeof(RowsShared) <= 160 * 1024 && sizeof(RowsShared) >= sizeof(LongShared), "LDS of a compute unit");
template <typename OffT>
__global__ __launch_bounds__(kLongThreads) void alias_build_rows_kernel(
    const OffT* __restrict__ seg_offsets, int64_t num_segments, int per_block, const int64_t* __restrict__ long_ids,
    const unsigned long long* __restrict__ long_count, int64_t max_long, int long_blocks, const float* __restrict__ weights,
    float* __restrict__ prob_out, int32_t* __restrict__ alias_out, double* mass_ws, int32_t* small_ws, int32_t* large_ws) {
  __shared__ __attribute__((aligned(16))) char lds[sizeof(RowsShared)];
  if ((int)blockIdx.x < long_blocks) {
    LongShared& shared = *reinterpret_cast<LongShared*>(lds);
    const int64_t count = (int64_t)min(*long_count, (unsigned long long)max_long);
    for (int64_t b = blockIdx.x; b < count; b += long_blocks) {
      long_segment<OffT>(shared, seg_offsets, long_ids[b], weights, prob_out, alias_out, mass_ws, small_ws, large_ws, nullptr,
                         nullptr);
      __syncthreads();
    }
    return;
  }
  if (*long_count == 0ull) return;
  RowsShared& shared = *reinterpret_cast<RowsShared*>(lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int64_t first = (int64_t)((int)blockIdx.x - long_blocks) * per_block; first < num_segments;
       first += (int64_t)((int)gridDim.x - long_blocks) * per_block) {
    __syncthreads();                           // (the last turn's segments have been taken)
    if (threadIdx.x == 0) shared.wide_count = shared.narrow_count = shared.wide_next = shared.narrow_next = 0;
    __syncthreads();
    if ((int)threadIdx.x < per_block && first + threadIdx.x < num_segments) {
      const int64_t n = (int64_t)seg_offsets[first + threadIdx.x + 1] - (int64_t)seg_offsets[first + threadIdx.x];
      if (n > kRowsMiddle && n <= kRowsMost) shared.wide_seg[atomicAdd(&shared.wide_count, 1)] = (uint16_t)threadIdx.x;
      else if (n > kLaneSegment && n <= kRowsMiddle) shared.narrow_seg[atomicAdd(&shared.narrow_count, 1)] = (uint16_t)threadIdx.x;
    }
    __syncthreads();
    int64_t begin;
    int n;
    auto take = [&](int* next, int count, const uint16_t* segs) {
      int at = 0;
      if (lane == 0) at = atomicAdd(next, 1);
      at = __builtin_amdgcn_readfirstlane(at);
      if (at >= count) return false;
      const int64_t seg = first + __builtin_amdgcn_readfirstlane((int)segs[at]);
      begin = (int64_t)seg_offsets[seg];
      n = __builtin_amdgcn_readfirstlane((int)((int64_t)seg_offsets[seg + 1] - begin));
      return true;
    };
    if (wave < kRowsWideWaves)
      while (take(&shared.wide_next, shared.wide_count, shared.wide_seg))
        wave_segment<kRowsMost>(shared.wide[wave], lane, n, weights + begin, prob_out + begin, alias_out + begin);
    // (the lists of a wide wave are its own, and idle by now)
    WaveLists<kRowsMiddle>& lists = wave < kRowsWideWaves ? *reinterpret_cast<WaveLists<kRowsMiddle>*>(&shared.wide[wave])
                                                          : shared.narrow[wave - kRowsWideWaves];
    while (take(&shared.narrow_next, shared.narrow_count, shared.narrow_seg))
      wave_segment<kRowsMiddle>(lists, lane, n, weights + begin, prob_out + begin, alias_out + begin);
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
  double* mass_seq;
  int32_t* alias_seq;
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
  p.states = cv.take<ListState>(kMostWideRounds + 2);
  p.flags = cv.take<uint64_t>(t / 64 + 1);
  p.counts = cv.take<int32_t>(t / kWideTile + 1);
  p.mass_seq = cv.take<double>(t);
  p.alias_seq = cv.take<int32_t>(t);
  p.wide_bytes = cv.used;
  return p;
}

static bool wide_segment(int64_t num_segments, int64_t total_entries) {
  return num_segments == 1 && total_entries >= kWideSegment;
}

template <typename OffT, int kThreads>
static int32_t launch_wide_rounds(const OffT* seg_offsets, int64_t n, const float* weights, float* prob_out,
                                  int32_t* alias_out, const AliasPlan& p, hipStream_t stream) {
  const unsigned tiles = (unsigned)std::min((int64_t)4096, ceil_div(n, kThreads * kLongItems));
  alias_wide_masses_kernel<OffT, kThreads><<<tiles, kThreads, 0, stream>>>(seg_offsets, weights, p.sum, p.mass, p.flags, p.counts);
  alias_wide_append_kernel<OffT, kThreads><<<tiles, kThreads, 0, stream>>>(seg_offsets, p.small_q, p.large_q, p.flags, p.counts,
                                                                           p.states, 1);
  GS_LAUNCH_CHECK();
  const int rounds = wide_rounds(n);
  const unsigned half = (unsigned)std::min((int64_t)2048, ceil_div(n / 2 + 1, kThreads * kLongItems));      // m is at most half of n
  for (int r = 0; r < rounds; ++r) {
    alias_wide_round_kernel<OffT, kThreads><<<half, kThreads, 0, stream>>>(
        seg_offsets, p.sum, prob_out, alias_out, p.mass, p.small_q, p.large_q, p.flags, p.counts, p.states + r);
    alias_wide_append_kernel<OffT, kThreads><<<half, kThreads, 0, stream>>>(seg_offsets, p.small_q, p.large_q, p.flags,
                                                                            p.counts, p.states + r, 0);
    GS_LAUNCH_CHECK();
  }
  return GS_OK;
}

template <typename OffT>
static int32_t launch_alias_wide(const OffT* seg_offsets, int64_t n, const float* weights, float* prob_out,
                                 int32_t* alias_out, const AliasPlan& p, hipStream_t stream) {
  const int64_t chunks = ceil_div(n, kSumChunk);
  alias_wide_chunks_kernel<OffT><<<(unsigned)std::min((int64_t)1024, ceil_div(chunks, kLongWaves)), kLongThreads, 0, stream>>>(
      seg_offsets, weights, p.chunk_sums, p.runs);
  int32_t* summed = p.counts;                  // (the counts come later)
  alias_wide_prefix_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, p.chunk_sums, p.runs, p.sum, summed);
  alias_wide_runs_kernel<OffT><<<(unsigned)std::min((int64_t)8192, ceil_div(chunks, 4)), 256, 0, stream>>>(
      seg_offsets, weights, p.chunk_sums, p.runs, summed);
  alias_wide_sum_kernel<OffT><<<1, 256, 0, stream>>>(seg_offsets, weights, p.runs, p.sum, summed);
  GS_LAUNCH_CHECK();
  const int32_t rc = n <= kWideSmallTiles
      ? launch_wide_rounds<OffT, kWideThreads>(seg_offsets, n, weights, prob_out, alias_out, p, stream)
      : launch_wide_rounds<OffT, kLongThreads>(seg_offsets, n, weights, prob_out, alias_out, p, stream);
  if (rc != GS_OK) return rc;
  ListState* left = p.states + wide_rounds(n);
  const unsigned blocks = (unsigned)std::min((int64_t)4096, ceil_div(n, 256));
  alias_wide_gather_kernel<OffT><<<blocks, 256, 0, stream>>>(seg_offsets, p.mass, p.small_q, left, p.mass_seq);
  alias_wide_tail_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, p.sum, p.mass, p.small_q, p.large_q, p.mass_seq,
                                                               p.alias_seq, left);
  alias_wide_table_kernel<OffT><<<blocks, 256, 0, stream>>>(seg_offsets, p.sum, p.small_q, p.mass_seq, p.alias_seq, left,
                                                            prob_out, alias_out);
  alias_build_long_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, weights, prob_out, alias_out, p.mass, p.small_q,
                                                                p.large_q, left + 1, p.sum);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

template <typename OffT>
static int32_t launch_alias_build(const OffT* seg_offsets, int64_t num_segments, int64_t total_entries,
                                  const float* weights, float* prob_out, int32_t* alias_out,
                                  const AliasPlan& p, hipStream_t stream) {
  if (p.sum != nullptr) return launch_alias_wide(seg_offsets, total_entries, weights, prob_out, alias_out, p, stream);
  if (num_segments == 1 && total_entries > kWaveSegment) {
    alias_build_long_kernel<OffT><<<1, kLongThreads, 0, stream>>>(seg_offsets, weights, prob_out, alias_out, p.mass,
                                                                  p.small_q, p.large_q, nullptr, nullptr);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  // at most this many segments are longer than a wave's
  const int64_t max_long = std::min(num_segments, total_entries / (kWaveSegment + 1));
  const unsigned long long* any_long = nullptr;
  if (max_long > 0) {
    zero_u64_kernel<<<1, 1, 0, stream>>>(p.long_count);
    GS_LAUNCH_CHECK();
    any_long = p.long_count;
  }
  const int threads = 64;
  alias_build_kernel<OffT><<<(unsigned)ceil_div(num_segments, threads), threads, 0, stream>>>(
      seg_offsets, num_segments, weights, prob_out, alias_out, max_long > 0 ? p.long_ids : nullptr, max_long, p.long_count);
  GS_LAUNCH_CHECK();
  // few segments: a wave each; many: up to 64 per wave, so that the short ones cost one look
  const int per_wave = (int)std::max((int64_t)1, std::min((int64_t)64, num_segments / 16384));
  const unsigned waves = (unsigned)ceil_div(num_segments, per_wave);
  if (total_entries > kLaneSegment) {
    alias_build_wave_kernel<OffT, (int)kLaneSegment + 1, kRowsMiddle><<<waves, 64, 0, stream>>>(
        seg_offsets, num_segments, per_wave, any_long, weights, prob_out, alias_out);
    GS_LAUNCH_CHECK();
  }
  // (the LDS of a wave bounds how many there are at a time: 257 .. 2048 entries in one kernel 267 us on the 1 M-node graph)
  if (total_entries > kRowsMiddle) {
    alias_build_wave_kernel<OffT, kRowsMiddle + 1, kRowsMost><<<waves, 64, 0, stream>>>(
        seg_offsets, num_segments, per_wave, any_long, weights, prob_out, alias_out);
    GS_LAUNCH_CHECK();
  }
  if (total_entries > kRowsMost) {
    alias_build_wave_kernel<OffT, kRowsMost + 1, kWaveSegment><<<waves, 64, 0, stream>>>(
        seg_offsets, num_segments, per_wave, nullptr, weights, prob_out, alias_out);
    GS_LAUNCH_CHECK();
  }
  if (max_long > 0) {
    const int long_blocks = (int)std::min(kRowsLongBlocks, max_long);
    // few segments: 16 per workgroup, whose waves then take one or two each
    const int per_block = (int)std::max((int64_t)16, std::min((int64_t)kRowsPerBlock, ceil_div(num_segments, 1024)));
    const int64_t row_blocks = std::min((int64_t)1 << 20, ceil_div(num_segments, per_block));
    alias_build_rows_kernel<OffT><<<(unsigned)(long_blocks + row_blocks), kLongThreads, 0, stream>>>(
        seg_offsets, num_segments, per_block, p.long_ids, p.long_count, max_long, long_blocks, weights, prob_out, alias_out,
        p.mass, p.small_q, p.large_q);
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
