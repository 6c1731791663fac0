// fp32 values as sums of three bf16 values, and what is computed again by fp32 fmas where that fails (elements that round to an
// infinite bf16): shared by the fp32 kernels on the matrix cores and the merge of their statistics.
#pragma once
#include "ccd_score_mfma.h"

namespace ccd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// (bf16(x0), bf16(x1)) packed; x0, x1 <- what the rounding left over
__device__ __forceinline__ uint32_t take_bf16(float& x0, float& x1) {
  const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x0, x1}, bf16x2));
  x0 -= __uint_as_float(p << 16);
  x1 -= __uint_as_float(p & 0xFFFF0000u);
  return p;
}
struct Split8 { bf16x8 s[3]; };              // h, m, l of eight values
__device__ __forceinline__ Split8 split8(const f32x4 (&v)[2]) {
  float x[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
  Split8 out;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = take_bf16(x[2 * i], x[2 * i + 1]);
    out.s[s] = __builtin_bit_cast(bf16x8, (u32x4){w[0], w[1], w[2], w[3]});
  }
  return out;
}

// logit of a query row that is held in registers and a key (times the scale), as the vector-ALU kernels take it
template <int HD>
__device__ __forceinline__ float plain_dot(const float4 (&a)[HD / 4], const float* __restrict__ b) {
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < HD / 4; ++i) {
    const float4 v = load4(b + 4 * i);
    acc = fmaf(a[i].x, v.x, acc);
    acc = fmaf(a[i].y, v.y, acc);
    acc = fmaf(a[i].z, v.z, acc);
    acc = fmaf(a[i].w, v.w, acc);
  }
  return acc;
}
template <int HD>
__device__ __forceinline__ void load_row(float4 (&a)[HD / 4], const float* __restrict__ p) {
#pragma unroll
  for (int i = 0; i < HD / 4; ++i) a[i] = load4(p + 4 * i);
}
// Scores that came out as NaN again, by a chain of fp32 fmas for every logit (the merge kernel does the same for statistics): u[t] =
// sum of 2^(x - lse[q]) over the rows q that see token t (first + q % P and later ones), t in [t0, t1).  By one wave.  Not inlined:
// the kernel around has no registers to spare, and code that is jumped over costs a miss of the instruction cache per launch
// (inlined: 1 us a pass).
template <int HD>
__device__ __noinline__ void scores_again(int GP, int P, int first, int t0, int t1, const float* __restrict__ Q, int64_t q_sh,
                                          const float* __restrict__ Ku, float c, const float* __restrict__ lse, float lse_mul,
                                          float* __restrict__ u) {
  __threadfence_block();
  for (int t = t0 + (int)(threadIdx.x & 63); t < t1; t += 64) {
    if (u[t] == u[t]) continue;
    float4 kr[HD / 4];
    load_row<HD>(kr, Ku + (int64_t)t * HD);
    float sum = 0.f;
    for (int q = 0; q < GP; ++q) {
      const int g = q / P, i = q - g * P;
      if (t < first + i) continue;
      sum += fast_exp2(fmaf(plain_dot<HD>(kr, Q + g * q_sh + (int64_t)i * HD), c, -lse[q] * lse_mul));
    }
    u[t] = sum;
  }
}

// (maximum, sum of 2^(x - maximum)) of a query row over the keys t .. last (a -infinite logit has no part in it), eight keys to a
// load of the row: it would not fit the registers of the small kernel that calls this, which hardly ever happens
template <int HD>
__device__ __noinline__ float2 statistics_of_row(const float* __restrict__ q, const float* __restrict__ Ku, int t, int last, float c) {
  constexpr int kKeys = 8;
  float2 a = make_float2(-INFINITY, 0.f);
  for (; t <= last; t += kKeys) {
    float x[kKeys];
#pragma unroll
    for (int e = 0; e < kKeys; ++e) x[e] = 0.f;
#pragma unroll 1
    for (int i = 0; i < HD; i += 4) {
      const float4 qq = load4(q + i);
#pragma unroll
      for (int e = 0; e < kKeys; ++e) {
        const float4 kk = load4(Ku + (int64_t)min(t + e, last) * HD + i);
        x[e] = fmaf(qq.x, kk.x, x[e]);
        x[e] = fmaf(qq.y, kk.y, x[e]);
        x[e] = fmaf(qq.z, kk.z, x[e]);
        x[e] = fmaf(qq.w, kk.w, x[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < kKeys; ++e) {
      const float y = t + e <= last ? x[e] * c : -INFINITY;
      if (y > a.x) a = make_float2(y, a.y * fast_exp2(a.x - y) + 1.f);
      else if (y != -INFINITY) a.y += fast_exp2(y - a.x);
    }
  }
  return a;
}

// The statistics of a query row (at q; CaP token `cap_pos`, first visible token `first`) over all slices - p[j * GP] - and the CaP
// keys (Kc, null: none; their entry: cap), those of them that came out as NaN taken again.  Not inlined: hardly ever needed, and its
// callers have no registers to spare.
template <int HD>
__device__ __noinline__ float2 statistics_again(const float* __restrict__ q, const float* __restrict__ Ku, const float* __restrict__ Kc,
                                                const float2* __restrict__ p, float2 cap, int GP, int n_slices, int slice, int n,
                                                int first, int cap_pos, float c) {
  float M = -INFINITY, Z = 0.f;
  for (int j = Kc != nullptr ? -1 : 0; j < n_slices; ++j) {            // -1: the CaP keys, of which the row sees 0 .. cap_pos
    const int t = j < 0 ? 0 : max(j * slice, first);
    const int last = j < 0 ? cap_pos : min(n, (j + 1) * slice) - 1;
    float2 v = j < 0 ? cap : p[(int64_t)j * GP];
    if (v.y != v.y) v = statistics_of_row<HD>(q, j < 0 ? Kc : Ku, t, last, c);
    if (v.y == 0.f) continue;
    const float m = fmaxf(M, v.x);
    Z = Z * fast_exp2(M - m) + v.y * fast_exp2(v.x - m);
    M = m;
  }
  return make_float2(M, Z);
}

}  // namespace ccd
