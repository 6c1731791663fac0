// Representative score of Eq. 2 for fp32 caches on the matrix cores, to fp32 accuracy: two passes over token slices, as
// on the vector ALUs (statistics per slice, merge, probabilities), with the logits computed as sums of bf16 products.
//
// gfx950's fp32 matrix instructions run at a sixteenth of the bf16 rate.  An fp32 value x is therefore split into three
// bf16 values, h = bf16(x), m = bf16(x - h), l = bf16(x - h - m) - 24 bits of mantissa, both differences exact - and a
// product taken as qh kh + (qh km + qm kh + qm km + qh kl + ql kh): six bf16 products with fp32 accumulation.  The three
// products left out are below 2^-24 of |q k| together, less than the rounding of one fp32 multiplication; the five small ones
// have a sum of their own, so that only the eight additions of qh kh (four for head dimension 64) round at the logit's
// size, where a chain of fp32 fmas rounds 128 (64) times.
//
// An element that rounds to an infinite bf16 (infinities, and finite values from 3.396e38 on) leaves remainders that are no
// numbers, and every logit it takes part in comes out as NaN, which reaches each sum that such a logit enters.  So the sums
// tell: a row's statistics of a slice (in the merge kernel), or a token's score (at the end of pass 2), that come out as NaN are
// computed again by a chain of fp32 fmas.  Calls without such elements pay 0.2 % (256 units of 4096 tokens) to 1.5 % (short rows).
//
// Bound by the matrix cores: 6 x 2 x 68.7 GFLOP for 256 units of 4096 tokens and 256 query rows of 128 elements.  A workgroup
// of eight waves (two per SIMD: one folds while the other one multiplies) takes one slice of a unit's tokens and up to 256
// query rows: a wave keeps the split fragments of 32 rows in registers and all waves share the K tiles, which are split once
// per workgroup on their way into LDS: fragment by fragment, so that every read is 64 consecutive 16-byte pieces.  Stages of
// 64 tokens, double buffered; the global loads of stage s + 2 are under way while stage s is multiplied.  The waves of a SIMD
// split their share of the next stage at opposite ends of a stage.  With up to 128 query rows two waves share a row block,
// one per tile of the stage.
//
// Measured, 256 units of 4096 fp32 tokens of 128 elements and 256 query rows: 330 us a pass, 5 us the merge, where the
// vector-ALU kernels took 3.2 ms for both passes.  Scores against fp64 (2 to 8 units, 1000 to 8000 tokens, logits
// up to about 10 / 25 / 65 / 160 log2 units): largest relative error 6e-7 / 2.5e-6 / 1.2e-5 / 2.4e-5, on the vector ALUs
// 2e-6 / 7e-6 / 2.5e-5 / 1e-4.
#include <algorithm>

#include "ccd_fp32.h"

namespace ccd {

namespace {

constexpr int kSplitThreads = 512;
constexpr int kSplitWaves = kSplitThreads / 64;
constexpr int kStage = 2 * kStep;            // tokens per stage: two tiles
constexpr int kSplitRows = kSplitWaves * 32; // query rows per sweep

template <int HD>
struct SplitLds {
  static constexpr int KQ = HD / 16;
  bf16x8 k[2][2][3 * KQ][64];                // [buffer][tile][h: 0.., m: KQ.., l: 2 KQ..][lane]
  float ub[4][kSplitWaves][kStage];          // pass 2: token sums of a stage per row block; pass 1: (reference, sum) pairs at the end
  int first[kSplitRows];                     // pass 2 under a window: the first token a query row sees
  int nan_out;                               // pass 2: some token's score is NaN
};

// PASS 1: part[unit, slice, q] = (maximum, sum of 2^(x - maximum)) of the log2-domain logits x of query row q over the slice;
//   slice n_slices1 (causal variant) stands for the CaP tokens' own keys, of which row g * P + i sees 0 .. i.
// PASS 2: u[unit, t] = sum over the query rows of 2^(x - lse2[q]).
template <int HD, int PASS>
__global__ __launch_bounds__(kSplitThreads, 2) void score_split_kernel(Dims D, ScorePlan pl, const float* __restrict__ Q,
                                                                       const float* __restrict__ K,
                                                                       const float* __restrict__ Kcap,
                                                                       float2* __restrict__ part,
                                                                       const float* __restrict__ lse2, float lse_mul,
                                                                       float* __restrict__ u) {
  constexpr int KQ = HD / 16;
  constexpr int kChunks = HD / 64;           // runs of eight elements that a thread stages
  constexpr int kEl = 16 / KQ;               // accumulator elements folded per k-step of the next tile
  __shared__ SplitLds<HD> sm;
  const int slices = PASS == 1 ? pl.n_slices1 + (Kcap != nullptr ? 1 : 0) : pl.n_slices2;
  const int slice = blockIdx.x % slices, unit = D.unit0 + blockIdx.x / slices, tid = threadIdx.x;
  const UnitIdx ui = decode_unit(D, unit);
  if (PASS == 2) clear_sync(D, pl, unit, slice == 0);
  const bool cap = PASS == 1 && slice == pl.n_slices1;
  const float* Ku = cap ? Kcap + (int64_t)unit * D.P * HD : K + kv_offset(D, ui);
  const int t0 = cap ? 0 : slice * pl.slice1, t1 = cap ? D.P : min(D.n, t0 + pl.slice1);
  // stages [it0, it1) of the slice: those before are hidden from every query by the window
  const int it1 = (t1 - t0 + kStage - 1) / kStage;
  const int it0 = cap ? 0 : min(it1, max(0, D.head0 - t0) / kStage);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, col = lane & 31, half = lane >> 5;
  const float c = D.scale_log2;
  if (PASS == 2 && tid == 0) sm.nan_out = 0;   // (set and read by the same wave)

  // staging: eight consecutive threads take the same elements of eight consecutive rows (their LDS writes are contiguous)
  const int st_c = (tid >> 3) % (HD / 8), st_row = (tid / HD) * 8 + (tid & 7);
  f32x4 raw[kChunks][2];
  auto request = [&](int it) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const float* p = Ku + (int64_t)min(t0 + it * kStage + i * kStep + st_row, t1 - 1) * HD + st_c * 8;
      raw[i][0] = *reinterpret_cast<const f32x4*>(p);
      raw[i][1] = *reinterpret_cast<const f32x4*>(p + 4);
    }
  };
  auto stage = [&](int it) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const Split8 x = split8(raw[i]);
      const int row = i * kStep + st_row;
#pragma unroll
      for (int s = 0; s < 3; ++s) sm.k[it & 1][row >> 5][s * KQ + (st_c >> 1)][(st_c & 1) * 32 + (row & 31)] = x.s[s];
    }
  };

  for (int qc = 0; qc < D.GP; qc += kSplitRows) {
    // row blocks of the sweep (1, 2, 4 or 8 waves side by side); up to four: the other waves take the other tile
    const int rows = min(D.GP - qc, kSplitRows), blocks = (rows + 31) / 32;
    const int wide = blocks <= 1 ? 1 : (blocks <= 2 ? 2 : (blocks <= 4 ? 4 : 8));
    const int rb = wave & (wide - 1), group = wave / wide;
    const bool active = rb < blocks && group < 2;
    const int tile0 = wide == 8 ? 0 : group, tile1 = wide == 8 ? 2 : group + 1;
    const int q = qc + rb * 32 + col;

    request(it0);
    // The wave's query rows, split.  Rows past G * P repeat the last one: nobody reads their statistics, and a normaliser of
    // infinity takes them out of the token sums.
    Split8 qf[KQ];
    {
      const float* row = Q + q_offset(D, ui, min(q, D.GP - 1)) + half * 8;
#pragma unroll
      for (int ks = 0; ks < KQ; ++ks)
        qf[ks] = split8({*reinterpret_cast<const f32x4*>(row + ks * 16), *reinterpret_cast<const f32x4*>(row + ks * 16 + 4)});
    }
    // pass 1: first and last key the lane's query sees;  pass 2: normalisers of the 16 query rows a lane holds
    const int lo = PASS == 1 && !cap && D.window > 0 ? D.win_off + q % D.P : 0;
    const int hi = PASS == 1 ? (cap ? q % D.P : t1 - 1) : 0;
    float nl[16];
    if (PASS == 2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qr = qc + rb * 32 + acc_row(r, half);
        const float l = lse2[(int64_t)unit * D.GP + min(qr, D.GP - 1)] * lse_mul;
        nl[r] = qr < D.GP ? -l : -INFINITY;
      }
      // A last CaP token whose window holds no cached token (window == P) takes no part either: a normaliser over cached tokens
      // alone is -infinity for it, and its masked logits would come out as -infinity + infinity.
      if (D.head > 0 && D.win_off + D.P > D.n) {
#pragma unroll 1
        for (int i = D.P - 1; i < D.GP; i += D.P)
#pragma unroll
          for (int r = 0; r < 16; ++r) nl[r] = qc + rb * 32 + acc_row(r, half) == i ? -INFINITY : nl[r];
      }
      if (D.head > 0 && tid < kSplitRows) sm.first[tid] = D.win_off + (qc + tid) % D.P;
    }
    float m = kNegHuge, z0 = 0.f, z1 = 0.f;      // pass 1: running maximum (raw logit) and sum
    floatx16 cur;                                // logits of the tile before, folded while the next one is multiplied
#pragma unroll
    for (int r = 0; r < 16; ++r) cur[r] = -INFINITY;
    float* ub_cur = &sm.ub[(it0 + 3) & 3][wave][0];     // where its token sums go (nobody reads those of the first fold)

    float negm = 0.f;
    auto fold_begin = [&]() {
      if (PASS == 1) {
        float t[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) t[i] = fmaxf(fmaxf(cur[3 * i], cur[3 * i + 1]), cur[3 * i + 2]);
        const float m_new = fmaxf(fmaxf(fmaxf(fmaxf(t[0], t[1]), t[2]), fmaxf(fmaxf(t[3], t[4]), cur[15])), m);
        const float f = fast_exp2((m - m_new) * c);
        z0 *= f;
        z1 *= f;
        m = m_new;
        negm = -m_new * c;
      } else {
        z0 = 0.f;
        z1 = 0.f;
      }
    };
    auto fold_some = [&](int ks) {
      float e[kEl];
#pragma unroll
      for (int i = 0; i < kEl; ++i) e[i] = fast_exp2(fmaf(cur[ks * kEl + i], c, PASS == 1 ? negm : nl[ks * kEl + i]));
#pragma unroll
      for (int i = 0; i < kEl; i += 2) { z0 += e[i]; z1 += e[i + 1]; }
      asm volatile("" : "+v"(z0), "+v"(z1));      // here and now: not sunk behind the matrix instructions
    };
    auto fold_end = [&]() {
      if (PASS == 2) {
        float v = z0 + z1;
        v += __shfl_xor(v, 32);
        if (half == 0) ub_cur[col] = v;
      }
    };
    // one tile: its logits while those of the tile before are folded
    auto multiply = [&](int it, int tile) {
      const bf16x8* kf = &sm.k[it & 1][tile][0][lane];
      floatx16 big, small;
#pragma unroll
      for (int r = 0; r < 16; ++r) { big[r] = 0.f; small[r] = 0.f; }
      auto mma = [](const bf16x8& k, const bf16x8& qv, const floatx16& acc) {
        return PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, qv, acc, 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, k, acc, 0, 0, 0);
      };
      bf16x8 f[2][3];
#pragma unroll
      for (int s = 0; s < 3; ++s) f[0][s] = kf[(s * KQ) * 64];
      fold_begin();
#pragma unroll
      for (int ks = 0; ks < KQ; ++ks) {
        const bf16x8(&k)[3] = f[ks & 1];
        if (ks + 1 < KQ) {
#pragma unroll
          for (int s = 0; s < 3; ++s) f[(ks + 1) & 1][s] = kf[(s * KQ + ks + 1) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
        small = mma(k[2], qf[ks].s[0], small);
        small = mma(k[1], qf[ks].s[1], small);
        small = mma(k[0], qf[ks].s[2], small);
        big = mma(k[0], qf[ks].s[0], big);
        small = mma(k[1], qf[ks].s[0], small);
        small = mma(k[0], qf[ks].s[1], small);
        fold_some(ks);
        __builtin_amdgcn_sched_barrier(0);
      }
      fold_end();
      cur = big + small;
      const int t = t0 + it * kStage + tile * kStep;
      if (PASS == 1) {
        if (cap || t + kStep > t1 || t < D.head) {          // some row may not see some token
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int tok = t + acc_row(r, half);
            if (tok < lo || tok > hi) cur[r] = -INFINITY;
          }
        }
      } else {
        if (t < D.head) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (t + col < sm.first[rb * 32 + acc_row(r, half)]) cur[r] = -INFINITY;
        }
        ub_cur = &sm.ub[it & 3][rb][tile * kStep];
      }
    };
    // pass 2: the token sums of a stage, added up over the row blocks
    auto write_out = [&](int it) {
      const int t = t0 + it * kStage + lane;
      if (wave == 0 && t < t1) {
        float v = sm.ub[it & 3][0][lane];
        for (int b = 1; b < blocks; ++b) v += sm.ub[it & 3][b][lane];
        if (v != v) sm.nan_out = 1;
        float* out = u + (int64_t)unit * D.n + t;
        *out = qc == 0 ? v : *out + v;
      }
    };

    if (it0 < it1) {
      stage(it0);
      request(it0 + 1);
      __syncthreads();
      for (int it = it0; it < it1; ++it) {
        if (wave < kSplitWaves / 2) { stage(it + 1); request(it + 2); }
        if (active)
          for (int tile = tile0; tile < tile1; ++tile) multiply(it, tile);
        if (wave >= kSplitWaves / 2) { stage(it + 1); request(it + 2); }
        // (a stage's last tile is folded in the iteration after it: its sums are complete one barrier later)
        if (PASS == 2 && it - 2 >= it0) write_out(it - 2);
        __syncthreads();
      }
      if (active) {
        fold_begin();
#pragma unroll
        for (int ks = 0; ks < KQ; ++ks) fold_some(ks);
        fold_end();
      }
      __syncthreads();
    }
    if (PASS == 2) {
      for (int it = max(it0, it1 - 2); it < it1; ++it) write_out(it);
      if (qc == 0)                              // tokens nobody sees
        for (int t = t0 + tid; t < min(t1, t0 + it0 * kStage); t += kSplitThreads) u[(int64_t)unit * D.n + t] = 0.f;
    } else {
      // the two lane halves, and the two waves of a row block, hold different tokens of the same query row
      float z = z0 + z1;
      const float m_o = __shfl_xor(m, 32), z_o = __shfl_xor(z, 32), M = fmaxf(m, m_o);
      z = z * fast_exp2((m - M) * c) + z_o * fast_exp2((m_o - M) * c);
      float2* st = reinterpret_cast<float2*>(&sm.ub[0][0][0]);      // [wave][row of the block]
      if (half == 0) st[wave * 32 + col] = make_float2(M, z);
      __syncthreads();
      if (active && group == 0 && half == 0 && q < D.GP) {
        float2 a = st[wave * 32 + col];
        if (wide < 8) {
          const float2 b = st[(wave + wide) * 32 + col];
          const float mm = fmaxf(a.x, b.x);
          a = make_float2(mm, a.y * fast_exp2((a.x - mm) * c) + b.y * fast_exp2((b.x - mm) * c));
        }
        part[cap ? extra_block_index(D, pl, unit, q) : ((int64_t)unit * pl.n_slices1 + slice) * D.GP + q] =
            make_float2(a.x * c, a.y);
      }
    }
    __syncthreads();          // the LDS tables are rewritten by the next sweep
  }
  if (PASS == 2 && wave == 0 && __builtin_expect(__builtin_amdgcn_readfirstlane(sm.nan_out) != 0, 0))
    scores_again<HD>(D.GP, D.P, D.window > 0 ? D.win_off : -D.P, t0, t1, Q + q_offset(D, ui, 0), D.q_sh, Ku, c,
                     lse2 + (int64_t)unit * D.GP, lse_mul, u + (int64_t)unit * D.n);
}

}  // namespace

// Token slices per unit: one workgroup fits a compute unit, so the rounds of the grid times the tokens of a workgroup, plus what
// a workgroup spends before and behind its tokens (about 100 of them), are the time of a pass.
void plan_split(const Dims& D, int compute_units, int min_slice, ScorePlan& pl) {
  const int max_slices = (D.n + min_slice - 1) / min_slice;
  int64_t best = INT64_MAX;
  for (int ns = 1; ns <= max_slices; ++ns) {
    const int slice = std::max(min_slice, ((D.n + ns - 1) / ns + kStage - 1) / kStage * kStage);
    const int64_t rounds = ((int64_t)D.units_run * ((D.n + slice - 1) / slice) + compute_units - 1) / compute_units;
    const int64_t cost = rounds * (slice + 100);
    if (cost < best) {
      best = cost;
      pl.slice1 = pl.slice2 = slice;
    }
  }
  pl.n_slices1 = pl.n_slices2 = (D.n + pl.slice1 - 1) / pl.slice1;
  pl.split_kernel = 1;
}

int64_t time_split(const Dims& D, int compute_units, const ScorePlan& pl, bool cap_keys, bool lse_given) {
  // per sweep; per stage with up to two, four and eight blocks of query rows side by side; the merge kernel and each of its slices
  struct Pass { int sweep, stage[3]; };
  struct Cost { Pass stats, prob; int merge, merge_slice; };
  static constexpr Cost c64{{281, {54, 87, 128}}, {560, {80, 118, 254}}, 87, 35}, c128{{516, {92, 160, 265}}, {844, {154, 239, 475}}, 40, 35};
  const Cost& c = D.d == 64 ? c64 : c128;
  const int sweeps = (D.GP + kSplitRows - 1) / kSplitRows, blocks = (D.GP - (sweeps - 1) * kSplitRows + 31) / 32;
  const int last = blocks <= 2 ? 0 : (blocks <= 4 ? 1 : 2);
  const int64_t stages = (std::min(pl.slice1, D.n) + kStage - 1) / kStage;
  auto pass = [&](const Pass& p, int slices) {
    const int64_t rounds = ((int64_t)D.units_run * slices + compute_units - 1) / compute_units;
    return rounds * (sweeps * p.sweep + stages * ((sweeps - 1) * p.stage[2] + p.stage[last]));
  };
  const int64_t prob = pass(c.prob, pl.n_slices2);
  return lse_given ? prob : prob + pass(c.stats, pl.n_slices1 + (cap_keys ? 1 : 0)) + c.merge + pl.n_slices1 * c.merge_slice;
}

void launch_stats_split(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const void* K_cap, float2* part,
                        hipStream_t s) {
  const dim3 grid((unsigned)(pl.n_slices1 + (K_cap != nullptr ? 1 : 0)) * D.units_run), block(kSplitThreads);
  auto* kernel = D.d == 64 ? score_split_kernel<64, 1> : score_split_kernel<128, 1>;
  launch(kernel, grid, block, s, D, pl, (const float*)Q, (const float*)K, (const float*)K_cap, part, nullptr, 0.f, nullptr);
}

void launch_prob_split(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const float* lse2, float* u,
                       hipStream_t s) {
  const dim3 grid((unsigned)pl.n_slices2 * D.units_run), block(kSplitThreads);
  const float lse_mul = pl.lse_given ? 1.44269504088896340736f : 1.0f;
  auto* kernel = D.d == 64 ? score_split_kernel<64, 2> : score_split_kernel<128, 2>;
  launch(kernel, grid, block, s, D, pl, (const float*)Q, (const float*)K, nullptr, nullptr, lse2, lse_mul, u);
}

}  // namespace ccd
