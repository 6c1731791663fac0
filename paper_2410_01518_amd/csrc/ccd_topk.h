// Exact top-k threshold selection inside one workgroup, shared by the NuC slots and the final selection.
//
// Keys are order-preserving 32-bit images of fp32 values.  An MSB-first radix select with digits of up to 10 bits
// (LDS histogram, one atomic per candidate key and pass) over the range the keys actually span yields the threshold
// key tau and the number `need` of keys equal to tau that still belong to the k largest: a token is selected iff
// key > tau, or key == tau and fewer than `need` equal tokens precede it in token order (lowest index wins ties).
//
// What bounds it: nothing but latency.  A row is a few KB, yet every step depends on the step before it, and a barrier
// with the cross-wave bookkeeping around it costs about 0.9 us with 16 waves.  Hence eight waves instead of 16 where the
// kernel has no other use for them (the bookkeeping is per wave), counts by ballots on the scalar unit, and every wave works out digits and thresholds for
// itself from LDS instead of having one wave do it and broadcast: one barrier per histogram pass and one behind the last
// candidates, where three and two were needed.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ccd {

constexpr int kBinBits = 10, kBins = 1 << kBinBits;
constexpr int kCandMax = 256;   // at most this many keys left in the chosen bin: they are ranked directly

constexpr uint32_t kHiFrom = 0xFF800000u;   // score_key(+inf)
constexpr uint32_t kLoUpTo = 0x007FFFFFu;   // score_key(-inf)

// fp32 -> uint32 with the same order; NaN ranks with -inf and -0 equals +0.  No key is 0.
__device__ __forceinline__ uint32_t score_key(float x) {
  if (x != x) x = -INFINITY;
  x += 0.0f;
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
// novelty key: NaN and -inf map to 0, strictly below every token that may take a NuC slot
__device__ __forceinline__ uint32_t novelty_key(float x) {
  if (x != x || x == -INFINITY) return 0u;
  return score_key(x);
}

// Wave-wide inclusive scan in six data-parallel-primitive steps (shifts inside rows of 16 lanes, then the last lane of
// a row broadcast into the following rows): one ALU instruction per step where a cross-lane shuffle takes a round trip
// through the LDS pipeline.  `identity` fills the lanes a step has no source for.
template <class Op>
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, uint32_t identity, Op op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return v;
}
struct OpAdd { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };
struct OpMin { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return min(a, b); } };
struct OpMax { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
// the operation over all 64 lanes, as a scalar
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, uint32_t identity, Op op) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v, identity, op), 63);
}
// the operation over each aligned group of N = 4, 8 or 16 lanes, as a scalar; all groups hold the same values
template <int N, class Op>
__device__ __forceinline__ uint32_t reduce_group(uint32_t v, Op op) {
  static_assert(N == 4 || N == 8 || N == 16, "");
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));    // quad_perm [1,0,3,2]
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));    // quad_perm [2,3,0,1]
  if (N >= 8) v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));    // row_half_mirror
  if (N == 16) v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));   // row_mirror
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// what radix_threshold and its callers share in LDS; two sets of everything, so that the NuC slots and the final
// selection need no barrier between them
template <int THREADS>
struct TopkShared {
  static constexpr int kWaves = THREADS / 64;
  __attribute__((aligned(16))) uint32_t hist[2][kBins];
  __attribute__((aligned(16))) uint32_t cand[2][kCandMax];   // the keys that share all digits fixed so far, once they are few
  uint4 classes[3][kWaves];                                  // per wave: class counts and key range (KeyClasses)
  uint32_t cand_n[2];
  uint32_t found[2][3];                                      // threshold among more than 64 candidates
};
// to be followed by a barrier before the first radix_threshold
template <int THREADS>
__device__ __forceinline__ void topk_clear(TopkShared<THREADS>& sh) {
  for (int i = threadIdx.x; i < 2 * kBins / 4; i += THREADS) reinterpret_cast<uint4*>(&sh.hist[0][0])[i] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < 2 * kCandMax / 4) reinterpret_cast<uint4*>(&sh.cand[0][0])[threadIdx.x] = make_uint4(0, 0, 0, 0);
  if (threadIdx.x < 2) sh.cand_n[threadIdx.x] = 0;
}

// Scores of one row share a few exponents, and a quarter or half of them are the +inf of the NuC slots: the top bits of
// such keys fall into a handful of histogram bins, and a wave's 64 LDS atomics on one address serialise.  So keys are
// split into three classes by fixed bounds - at or above the key of +inf, at or below the key of -inf, ordinary - with
// counts and, for the ordinary ones, the range.  The class that holds the k-th largest is known from the counts; inside
// it - the two outer ones hold a single value each - the digits are taken from key - mn over the range actually spanned.
struct KeyClasses { uint32_t mn, mx, n_mid, n_hi; };

// A thread's keys folded into its wave's classes (counts are wave totals and scalar; mn and mx are per lane)
__device__ __forceinline__ void classify(uint32_t key, KeyClasses& c) {
  const bool hi = key >= kHiFrom, mid = !hi && key > kLoUpTo;
  c.n_hi += (uint32_t)__popcll(__ballot(hi));
  c.n_mid += (uint32_t)__popcll(__ballot(mid));
  c.mn = mid ? min(c.mn, key) : c.mn;
  c.mx = mid ? max(c.mx, key) : c.mx;
}
// set `which` of sh.classes; a barrier, then combine_classes
template <int THREADS>
__device__ __forceinline__ void publish_classes(KeyClasses c, TopkShared<THREADS>& sh, int which) {
  const uint32_t mn = wave_reduce(c.mn, 0xFFFFFFFFu, OpMin{}), mx = wave_reduce(c.mx, 0u, OpMax{});
  if ((threadIdx.x & 63) == 0) sh.classes[which][threadIdx.x >> 6] = make_uint4(mn, mx, c.n_mid, c.n_hi);
}
template <int THREADS>
__device__ __forceinline__ KeyClasses combine_classes(const TopkShared<THREADS>& sh, int which) {
  constexpr int W = THREADS / 64;
  const uint4 v = sh.classes[which][threadIdx.x & (W - 1)];
  return {reduce_group<W>(v.x, OpMin{}), reduce_group<W>(v.y, OpMax{}), reduce_group<W>(v.z, OpAdd{}), reduce_group<W>(v.w, OpAdd{})};
}

struct Threshold { uint32_t tau, need, n_eq; };   // n_eq: keys equal to tau in all; need of them are wanted

// The `remaining`-th largest of the `count` keys of the workgroup that lie in [lo, hi] (1 <= remaining <= count).
// each_key(f): calls f(key) for every key of the thread; keys outside [lo, hi] take no part.  hist[which] must be cleared
// and the clearing visible; ends without a barrier.
template <int THREADS, class EachKey>
__device__ __forceinline__ Threshold radix_threshold(EachKey&& each_key, uint32_t lo, uint32_t hi, uint32_t remaining,
                                                     uint32_t count, TopkShared<THREADS>& sh, int which) {
  const int lane = threadIdx.x & 63;
  uint32_t* hist = sh.hist[which];
  const uint32_t span = hi - lo;
  int rem_bits = 32 - __clz(span);             // bits of key - lo not yet fixed (__clz(0) = 32)
  uint32_t prefix = 0;                         // the fixed high bits of tau - lo, as a value (already shifted down)
  if (rem_bits == 0) return {lo, remaining, count};
  bool first = true;
#pragma unroll 1
  while (true) {
    const int width = min(kBinBits, rem_bits), shift = rem_bits - width;
    const uint32_t dmask = (1u << width) - 1u;
    each_key([&](uint32_t key) {
      const uint32_t rel = key - lo;
      if (rel <= span && (first || (rel >> rem_bits) == prefix)) atomicAdd(&hist[(rel >> shift) & dmask], 1u);
    });
    __syncthreads();
    // Lane 0 owns the highest 16 bins, so inclusive sums in lane order count the keys of larger digits; then the same over
    // the bins of the lane in which the wanted key falls.
    constexpr int kPerLane = kBins / 64;
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kPerLane; i += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(&hist[kBins - kPerLane * (lane + 1) + i]);
      mine += v.x + v.y + v.z + v.w;
    }
    const uint32_t incl = wave_inclusive_scan(mine, 0u, OpAdd{});
    const int owner = __ffsll((unsigned long long)__ballot(incl >= remaining)) - 1;
    remaining -= (uint32_t)__builtin_amdgcn_readlane((int)(incl - mine), owner);
    const int top = kBins - kPerLane * owner - 1;           // the owner's highest bin
    const uint32_t h = lane < kPerLane ? hist[top - lane] : 0u;
    const uint32_t incl2 = wave_inclusive_scan(h, 0u, OpAdd{});
    const int at_bin = __ffsll((unsigned long long)__ballot(incl2 >= remaining)) - 1;
    const uint32_t n_cand = (uint32_t)__builtin_amdgcn_readlane((int)h, at_bin);
    remaining -= (uint32_t)__builtin_amdgcn_readlane((int)incl2, at_bin) - n_cand;
    const uint32_t dig = (uint32_t)(top - at_bin);
    prefix = (prefix << width) | dig;
    rem_bits = shift;
    first = false;
    if (rem_bits == 0) return {lo + prefix, remaining, n_cand};
    if (n_cand <= (uint32_t)kCandMax) {
      // Few keys share the digits fixed so far (the digits are spread over the range, so this is the rule after one
      // pass): gather them and rank them against each other instead of two more histogram passes.
      each_key([&](uint32_t key) {
        const uint32_t rel = key - lo;
        if (rel <= span && (rel >> rem_bits) == prefix) sh.cand[which][atomicAdd(&sh.cand_n[which], 1u)] = key;
      });
      __syncthreads();
      // gt = candidates above mine; the wanted key is the smallest one with fewer than `remaining` above it.  (The list is
      // padded with zeros, which are above nothing; it is read four at a time, all lanes the same address.)
      const uint4* list = reinterpret_cast<const uint4*>(sh.cand[which]);
      if (n_cand <= 64) {
        const uint32_t c = sh.cand[which][lane];
        uint32_t gt = 0;
        for (uint32_t i = 0; i < n_cand; i += 8) {
          const uint4 v = list[i / 4], w = list[i / 4 + 1];
          gt += (v.x > c ? 1u : 0u) + (v.y > c ? 1u : 0u) + (v.z > c ? 1u : 0u) + (v.w > c ? 1u : 0u);
          gt += (w.x > c ? 1u : 0u) + (w.y > c ? 1u : 0u) + (w.z > c ? 1u : 0u) + (w.w > c ? 1u : 0u);
        }
        const uint32_t tau = wave_reduce(gt < remaining && (uint32_t)lane < n_cand ? c : 0xFFFFFFFFu, 0xFFFFFFFFu, OpMin{});
        const uint64_t is = __ballot(c == tau);
        return {tau, remaining - (uint32_t)__builtin_amdgcn_readlane((int)gt, __ffsll((unsigned long long)is) - 1),
                (uint32_t)__popcll(is)};
      }
      if (threadIdx.x < n_cand) {
        const uint32_t c = sh.cand[which][threadIdx.x];
        uint32_t gt = 0, ge = 0;
        for (uint32_t i = 0; i < n_cand; i += 4) {
          const uint4 v = list[i / 4];
          gt += (v.x > c ? 1u : 0u) + (v.y > c ? 1u : 0u) + (v.z > c ? 1u : 0u) + (v.w > c ? 1u : 0u);
          ge += (v.x >= c ? 1u : 0u) + (v.y >= c ? 1u : 0u) + (v.z >= c ? 1u : 0u) + (v.w >= c ? 1u : 0u);
        }
        if (gt < remaining && remaining <= ge) {             // (equal keys write the same values)
          sh.found[which][0] = c;
          sh.found[which][1] = remaining - gt;
          sh.found[which][2] = ge - gt;
        }
      }
      __syncthreads();
      return {sh.found[which][0], sh.found[which][1], sh.found[which][2]};
    }
    __syncthreads();                           // every wave has read the histogram
    for (int i = threadIdx.x; i < kBins / 4; i += THREADS) reinterpret_cast<uint4*>(hist)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
  }
}

// Ranks in token order.  A row is dealt out in chunks of four consecutive tokens: chunk c of thread t starts at token
// 4 (c * THREADS + t), so the 64 chunks of a wave's round c follow each other, and the rounds c * (THREADS / 64) + wave
// follow each other in the row.  `sums` (LDS, MAXCH * THREADS / 64 words): every wave puts the total of each of its rounds there
// (put_round_sum), a barrier, then RoundBases hands out the sum of all rounds before one.
template <int THREADS>
__device__ __forceinline__ void put_round_sum(uint32_t inclusive, uint32_t* sums, int c) {
  if ((threadIdx.x & 63) == 63) sums[c * (THREADS / 64) + (threadIdx.x >> 6)] = inclusive;
}
template <int THREADS, int MAXCH>
struct RoundBases {
  static constexpr int kWaves = THREADS / 64;
  static constexpr int kPer = (MAXCH * kWaves + 63) / 64;   // entry e sits in lane e / kPer
  static_assert(kWaves % kPer == 0, "the place of a wave's entries inside a lane does not depend on c");
  uint32_t s;
  int wave;
  __device__ __forceinline__ RoundBases(const uint32_t* sums, int rounds) {
    const int lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t v[kPer], mine = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = lane * kPer + i;
      v[i] = e < rounds * kWaves ? sums[e] : 0u;
      mine += v[i];
    }
    uint32_t run = wave_inclusive_scan(mine, 0u, OpAdd{}) - mine;
    s = run;
#pragma unroll
    for (int i = 1; i < kPer; ++i) {
      run += v[i - 1];
      s = wave % kPer == i ? run : s;
    }
  }
  __device__ __forceinline__ uint32_t of(int c) const {
    return (uint32_t)__builtin_amdgcn_readlane((int)s, (c * kWaves + wave) / kPer);
  }
};

}  // namespace ccd
