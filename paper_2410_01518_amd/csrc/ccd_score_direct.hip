// Representative score of Eq. 2 for bf16 caches on the matrix cores, for calls that do not fill the chip: two passes over short
// token slices.
//
// Such a call is bound by latency: the slice kernels of ccd_score_mfma.hip take about 10 us a pass whatever its size - two
// rounds of DMA through the LDS ring with a barrier each, then eight tiles one after the other in a slice of 256 tokens, while
// waves that have no query rows compute zeros.  Here a workgroup requests everything it needs first at once (its query rows and
// two tiles per wave, by DMA in whole lines: fragments loaded straight from memory, 32 bytes of a row at a time, took 1 to 2 us
// longer and twice the time when there was more to do), and the work is cut until it covers the chip:
//
//   pass 1  a workgroup takes (unit, slice of tokens, 64 query rows); its four waves take turns at pairs of tiles, each with a
//           running maximum and sum per row, merged through LDS.  The workgroups that share a slice are placed on one XCD.
//   pass 2  a workgroup takes (unit, slice of tokens); its waves lie side by side over one, two or four blocks of 64 query rows
//           and over the tiles.  It merges the statistics of the unit's slices for itself.
//
// A sliding window and the CaP keys (one more slice of pass 1) are masked in the tiles they touch: no kernels of their own.
// Two workgroups fit a compute unit; while one waits for its tiles the other one multiplies.
//
// Measured per pass, slice kernels against these: 8 units of 2048 tokens, 256 query rows 11.4 / 11.5 -> 5.9 / 8.1 us; 15 units of
// 448 tokens, 48 rows 9.5 / 9.5 -> 5.7 / 6.5 us; 48 units of 800 tokens under a window with CaP keys 4.1 + 9.2 + 10.8 + 4.5 -> 5.3 +
// 6.5 us.  (Steps of one tile per wave with the next ones under way, so that pass 1 can have 256 rows to a workgroup: 2 to 3 us
// slower on these, no faster on longer ones.)  Which calls come here: direct_pays in infinipot_api.hip.
#include "ccd_score_mfma.h"

namespace ccd {

namespace {

constexpr int kRowsPerWave = kQB * 32;       // query rows of a wave: 64
constexpr int kTilesPerWave = 2;             // tiles a wave has in LDS at a time
// Tokens per workgroup at most (pass 2: its token sums lie where the query rows were)
constexpr int kDirectMaxSlice1 = 4096, kDirectMaxSlice2 = 2048;

// The query rows of all waves and the tiles, in the swizzled order of ccd_score_mfma.h: in pass 1, and with up to 64 query rows, 16
// + 64 KiB (head dimension 128); with 128 query rows 32 + 32 KiB; with more 64 + 16 KiB.  No more than half of the LDS of a
// compute unit: what waves tell each other lies where the query rows were, once these are in registers.
template <int HD>
struct DirectLds {
  static_assert(kDirectMaxSlice2 * 4 <= kQB * Tiles<HD>::kSlotBytes, "the sums of a row block fit where its rows were");
  __attribute__((aligned(1024))) uint8_t rows[(kQB + 4 * kTilesPerWave) * Tiles<HD>::kSlotBytes];
};

// 64 x 16 bytes from the lanes' own addresses to consecutive LDS addresses
__device__ __forceinline__ void dma16_at(const void* p, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(p) : "memory");
}
// one 32-row tile by one wave; row(r): address of row r
template <int HD, class RowAt>
__device__ __forceinline__ void stage_tile(RowAt&& row_at, uint32_t lds_addr, int lane) {
  using T = Tiles<HD>;
#pragma unroll
  for (int j = 0; j < T::kInstrPerTile; ++j) {
    const int row = j * T::kRowsPerInstr + lane / T::kChunksPerRow, ch = (lane % T::kChunksPerRow) ^ T::swz(row);
    dma16_at(reinterpret_cast<const char*>(row_at(row)) + ch * 16, lds_addr + j * 1024);
  }
}

template <int HD, int PASS>
__global__ __launch_bounds__(kMT, 2) void score_direct_kernel(Dims D, ScorePlan pl, const uint16_t* __restrict__ Q,
                                                              const uint16_t* __restrict__ K, const uint16_t* __restrict__ Kcap,
                                                              float2* __restrict__ part, const float* __restrict__ lse_given,
                                                              float* __restrict__ u) {
  constexpr int KS = HD / 16;
  constexpr int kSlot = Tiles<HD>::kSlotBytes;
  __shared__ DirectLds<HD> sm;
  const int row_blocks = (D.GP + kRowsPerWave - 1) / kRowsPerWave;
  const int slices = PASS == 1 ? pl.n_slices1 + (Kcap != nullptr ? 1 : 0) : pl.n_slices2;
  // consecutive blocks go to different XCDs: the workgroups of one slice are eight blocks apart
  const int per_item = PASS == 1 ? row_blocks : 1;
  const int item = (int)(blockIdx.x >> 3) / per_item * 8 + (int)(blockIdx.x & 7);
  if (item >= D.units_run * slices) return;
  const int slice = item % slices, unit = D.unit0 + item / slices;
  const UnitIdx ui = decode_unit(D, unit);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const float c = D.scale_log2;
  if (PASS == 2) clear_sync(pl, unit, slice == 0);
  const bool cap = PASS == 1 && slice == pl.n_slices1;
  const uint16_t* Ku = cap ? Kcap + (int64_t)unit * D.P * HD : K + kv_offset(D, ui);
  const int slice_len = PASS == 1 ? pl.slice1 : pl.slice2;
  const int t0 = cap ? 0 : slice * slice_len, t1 = cap ? D.P : min(D.n, t0 + slice_len);
  // tiles [it0, it1) of the slice: those before are hidden from every query by the window
  const int it1 = (t1 - t0 + kStep - 1) / kStep;
  const int it0 = cap ? 0 : min(it1, max(0, D.head0 - t0) / kStep);
  const uint32_t rows_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)sm.rows;
  int koff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) koff[ks] = col * Tiles<HD>::kRowBytes + (((2 * ks + half) ^ Tiles<HD>::swz(col)) << 4);
  auto frags = [&](bf16x8 (&a)[KS], int slot) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) a[ks] = *reinterpret_cast<const bf16x8*>(sm.rows + slot * kSlot + koff[ks]);
  };

  // waves side by side over 64-row blocks (1, 2 or 4 of them; pass 1: one), the others on other tiles
  const int wide = PASS == 1 || row_blocks <= 1 ? 1 : (row_blocks <= 2 ? 2 : 4), groups = 4 / wide;
  const int rb = wave % wide, group = wave / wide;
  const int q_first = PASS == 1 ? (int)(blockIdx.x >> 3) % per_item * kRowsPerWave : 0;
  const int q_last = PASS == 1 ? min(D.GP, q_first + kRowsPerWave) : D.GP;
  float* up = reinterpret_cast<float*>(sm.rows);             // pass 2: token sums per row block
  float m_raw[kQB], Z[kQB];                  // pass 1
  int lo[kQB], hi[kQB];                      // pass 1: first and last key the lane's query rows see
  if (PASS == 1) {
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
      const int q = q_first + qb * 32 + col;
      m_raw[qb] = kNegHuge;
      Z[qb] = 0.f;
      lo[qb] = !cap && D.window > 0 ? D.win_off + q % D.P : 0;
      hi[qb] = cap ? q % D.P : t1 - 1;
    }
  }
  for (int qc = q_first; qc < q_last; qc += kQPerPass) {
    const int q0 = qc + rb * kRowsPerWave;
    // the query rows: 2 wide tiles, dealt to the four waves (rows past G P repeat the last one: nobody reads their statistics,
    // and a normaliser of infinity takes them out of the token sums)
    for (int b = wave; b < kQB * wide; b += 4)
      stage_tile<HD>([&](int r) { return Q + q_offset(D, ui, min(qc + b * 32 + r, D.GP - 1)); }, rows_addr + b * kSlot, lane);
    const int batch = groups * kTilesPerWave;              // tiles in LDS at a time
    const int slot0 = kQB * wide;
    auto stage_keys = [&](int it) {
      for (int b = wave; b < batch; b += 4)
        if (it + b < it1)
          stage_tile<HD>([&](int r) { return Ku + (int64_t)min(t0 + (it + b) * kStep + r, t1 - 1) * HD; },
                         rows_addr + (slot0 + b) * kSlot, lane);
    };
    stage_keys(it0);
    float neg_lse = -INFINITY;                 // pass 2: of row q0 + lane, the statistics of all slices merged
    const int q = q0 + lane;
    if (PASS == 2 && q < D.GP) {
      if (pl.lse_given) {
        neg_lse = -(lse_given[(int64_t)unit * D.GP + q] * 1.44269504088896340736f);
      } else {
        float2 cp = make_float2(kNegHuge, 0.f);
        if (pl.cap_block) cp = part[extra_block_index(D, pl, unit, q)];
        const float2* p = part + (int64_t)unit * pl.n_slices1 * D.GP + q;
        constexpr int kFly = 16;               // loads in flight, the last ones over again past the end
        const int n = pl.n_slices1;
        float M = cp.x, z = cp.y;
        for (int j0 = 0; j0 < n; j0 += kFly) {
          float2 v[kFly];
#pragma unroll
          for (int j = 0; j < kFly; ++j) v[j] = p[(int64_t)min(j0 + j, n - 1) * D.GP];
          float M_new = M;
#pragma unroll
          for (int j = 0; j < kFly; ++j) M_new = fmaxf(M_new, v[j].x);
          z *= fast_exp2(M - M_new);
          M = M_new;
#pragma unroll
          for (int j = 0; j < kFly; ++j)
            if (j0 + j < n) z += v[j].y * fast_exp2(v[j].x - M);
        }
        neg_lse = -(M + __log2f(z));
      }
    }
    float nl[PASS == 2 ? kQB : 1][16];
    if (PASS == 2) {
#pragma unroll
      for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r) nl[qb][r] = __shfl(neg_lse, qb * 32 + acc_row(r, half));
    }
    const int first = D.win_off + q % D.P;     // pass 2 under a window: the first token row q sees
    wait_all_dma();
    __syncthreads();
    const bool active = q0 < q_last;
    bf16x8 bq[kQB][KS];
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) frags(bq[qb], rb * kQB + qb);
    if (PASS == 2) __syncthreads();            // the query rows make room for token sums
    for (int it = it0; it < it1; it += batch) {
      if (it > it0) {
        __syncthreads();
        stage_keys(it);
        wait_all_dma();
        __syncthreads();
      }
#pragma unroll
      for (int i = 0; i < kTilesPerWave; ++i) {
        const int b = group * kTilesPerWave + i, t = t0 + (it + b) * kStep;
        if (active && it + b < it1) {
          bf16x8 a[KS];
          frags(a, slot0 + b);
          floatx16 acc[kQB];
          logits<HD, PASS>(acc, a, bq);
          if constexpr (PASS == 1) {
            if (cap || t + kStep > t1 || t < D.head) {            // some row may not see some key
#pragma unroll
              for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const int tok = t + acc_row(r, half);
                  if (tok < lo[qb] || tok > hi[qb]) acc[qb][r] = -INFINITY;
                }
            }
            fold_stats<false>(acc, m_raw, Z, c, half, kStep);
          } else {
            float us = 0.f;
            if (t < D.head) {
              int f = first;
              asm volatile("" : "+v"(f));               // (32 values that would be kept in registers for all tiles)
#pragma unroll
              for (int qb = 0; qb < kQB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const float p = fast_exp2(fmaf(acc[qb][r], c, nl[qb][r]));
                  us += t + col >= __shfl(f, qb * 32 + acc_row(r, half)) ? p : 0.f;
                }
            } else {
              us = fold_prob(acc, nl, c);
            }
            us += __shfl_xor(us, 32);
            if (half == 0) up[rb * pl.slice2 + (it + b) * kStep + col] = us;
          }
        }
      }
    }
    __syncthreads();
    if constexpr (PASS == 2) {
      const int used = min(wide, (D.GP - qc + kRowsPerWave - 1) / kRowsPerWave);
      float* uu = u + (int64_t)unit * D.n + t0;
      for (int t = threadIdx.x; t < t1 - t0; t += kMT) {
        float v = 0.f;                         // (tokens nobody sees)
        if (t >= it0 * kStep) {
          v = up[t];
          for (int w = 1; w < used; ++w) v += up[w * pl.slice2 + t];
        }
        uu[t] = qc == 0 ? v : uu[t] + v;
      }
      __syncthreads();                         // the next sweep's query rows take the place of the sums
    }
  }
  if constexpr (PASS == 1) {
    // the two lane halves and the four waves hold different tokens of the same query rows
    float2* stat = reinterpret_cast<float2*>(sm.rows);
#pragma unroll
    for (int qb = 0; qb < kQB; ++qb) {
      const float m_o = __shfl_xor(m_raw[qb], 32), z_o = __shfl_xor(Z[qb], 32);
      const float M = fmaxf(m_raw[qb], m_o);
      const float z = Z[qb] * fast_exp2((m_raw[qb] - M) * c) + z_o * fast_exp2((m_o - M) * c);
      if (half == 0) stat[wave * kRowsPerWave + qb * 32 + col] = make_float2(M * c, z);
    }
    __syncthreads();
    const int q = q_first + (int)threadIdx.x;
    if (threadIdx.x < kRowsPerWave && q < D.GP) {
      float2 v[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) v[w] = stat[w * kRowsPerWave + threadIdx.x];
      const float M = fmaxf(fmaxf(v[0].x, v[1].x), fmaxf(v[2].x, v[3].x));
      float z = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) z += v[w].y * fast_exp2(v[w].x - M);
      part[cap ? extra_block_index(D, pl, unit, q) : ((int64_t)unit * pl.n_slices1 + slice) * D.GP + q] = make_float2(M, z);
    }
  }
}

unsigned direct_grid(const Dims& D, int slices, int per_item) {
  return (unsigned)(((int64_t)D.units_run * slices + 7) / 8 * 8 * per_item);
}

}  // namespace

// Slices: two workgroups fit a compute unit, so the rounds of the grid times what one takes - its batches of tiles, and as much as
// three of them before and behind these - are the time of a pass; a workgroup that has its compute unit to itself is an eighth faster.
// (Powers of two with at least 1.25 workgroups per compute unit, before: 45 units of 3001 tokens were 540 workgroups on 512 places,
// two rounds, step by step 52.7 -> 48.3 us; 120 units of 2500 tokens and 256 rows 152 -> 138 us for append + distill.)
void plan_direct(const Dims& D, int compute_units, int min_slice, ScorePlan& pl) {
  const int row_blocks = (D.GP + kRowsPerWave - 1) / kRowsPerWave, groups = row_blocks <= 1 ? 4 : (row_blocks <= 2 ? 2 : 1);
  auto best_slice = [&](int batch, int most, int per_slice) {
    int best = batch;
    int64_t best_cost = INT64_MAX;
    for (int slice = batch; slice <= most; slice += batch) {
      const int64_t wgs = (int64_t)D.units_run * ((D.n + slice - 1) / slice) * per_slice;
      const int64_t rounds = (wgs + 2 * compute_units - 1) / (2 * compute_units);
      const int64_t cost = rounds * (3 + slice / batch) * (wgs <= compute_units ? 7 : 8);
      if (cost < best_cost) { best_cost = cost; best = slice; }
      if (slice >= D.n) break;
    }
    return best;
  };
  pl.slice1 = best_slice(4 * kTilesPerWave * kStep, kDirectMaxSlice1, row_blocks);
  pl.slice2 = best_slice(groups * kTilesPerWave * kStep, kDirectMaxSlice2, 1);
  pl.n_slices1 = (D.n + pl.slice1 - 1) / pl.slice1;
  pl.n_slices2 = (D.n + pl.slice2 - 1) / pl.slice2;
  pl.direct_kernel = 1;
}

void launch_stats_direct(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const void* K_cap, float2* part,
                         hipStream_t s) {
  const int row_blocks = (D.GP + kRowsPerWave - 1) / kRowsPerWave;
  const dim3 grid(direct_grid(D, pl.n_slices1 + (K_cap != nullptr ? 1 : 0), row_blocks)), block(kMT);
  auto* kernel = D.d == 64 ? score_direct_kernel<64, 1> : score_direct_kernel<128, 1>;
  launch(kernel, grid, block, s, D, pl, (const uint16_t*)Q, (const uint16_t*)K, (const uint16_t*)K_cap, part, nullptr, nullptr);
}

void launch_prob_direct(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const float2* part, const float* lse,
                        float* u, hipStream_t s) {
  const dim3 grid(direct_grid(D, pl.n_slices2, 1)), block(kMT);
  auto* kernel = D.d == 64 ? score_direct_kernel<64, 2> : score_direct_kernel<128, 2>;
  launch(kernel, grid, block, s, D, pl, (const uint16_t*)Q, (const uint16_t*)K, nullptr, const_cast<float2*>(part), lse, u);
}

}  // namespace ccd
