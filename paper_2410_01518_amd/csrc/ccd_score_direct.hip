// Representative score of Eq. 2 on the matrix cores for calls that do not fill the chip: two passes over short token slices.  bf16
// caches, and fp32 caches as sums of six bf16 products (ccd_fp32.h, ccd_score_split.hip).
//
// Such a call is bound by latency: the slice kernels of ccd_score_mfma.hip take about 10 us a pass whatever its size - two
// rounds of DMA through the LDS ring with a barrier each, then eight tiles one after the other in a slice of 256 tokens, while
// waves that have no query rows compute zeros - and the six-product kernels 9 to 23 us and another 4 for their merge.  Here a
// workgroup requests everything it needs first at once (its query rows and one or two tiles per wave, by DMA in whole lines: bf16
// fragments loaded straight from memory, 32 bytes of a row at a time, took 1 to 2 us longer and twice the time when there was more
// to do), and the work is cut until it covers the chip:
//
//   pass 1  a workgroup takes (unit, slice of tokens, 64 query rows - fp32: 32, whose three fragments fill the registers); its four
//           waves take turns at the tiles, each with a running maximum and sum per row, merged through LDS.  The workgroups that
//           share a slice are placed on one XCD.
//   pass 2  a workgroup takes (unit, slice of tokens); its waves lie side by side over one, two or four blocks of query rows
//           and over the tiles.  It merges the statistics of the unit's slices for itself.
//
// A sliding window and the CaP keys (one more slice of pass 1) are masked in the tiles they touch: no kernels of their own.
// Two workgroups fit a compute unit; while one waits for its tiles the other one multiplies.
//
// Measured per pass, slice kernels against these: 8 units of 2048 tokens, 256 query rows 11.4 / 11.5 -> 5.9 / 8.1 us; 15 units of
// 448 tokens, 48 rows 9.5 / 9.5 -> 5.7 / 6.5 us; 48 units of 800 tokens under a window with CaP keys 4.1 + 9.2 + 10.8 + 4.5 -> 5.3 +
// 6.5 us.  fp32, append + distill: 4 units of 820 tokens, 100 rows, 64 / 128 elements 39 / 51 -> 28 / 33 us.  (Steps of one tile per wave
// with the next ones under way, so that pass 1 can have 256 rows to a workgroup: 2 to 3 us slower on small calls, no faster on
// longer ones.)  Which calls come here: direct_pays and plan_score in infinipot_api.hip.
#include <algorithm>
#include <type_traits>

#include "ccd_fp32.h"
#include "ccd_select_body.h"

namespace ccd {

namespace {

// Tokens per workgroup at most (pass 2: its token sums lie where the query rows were)
constexpr int kDirectMaxSlice1 = 4096, kDirectMaxSlice2 = 1024;

// Rows of HD elements of type ET (uint16_t: bf16 bits; float) in LDS, in tiles of 32: 16-byte chunk c of row r at c ^ swz(r)
template <int HD, class ET>
struct DirectShape {
  static constexpr bool F32 = std::is_same<ET, float>::value;
  static constexpr int QB = F32 ? 1 : 2;                     // blocks of 32 query rows per wave (fp32: three fragments for one)
  static constexpr int kRows = 32 * QB;                      // query rows of a wave
  static constexpr int kTiles = F32 && HD == 128 ? 1 : 2;    // tiles a wave has in LDS at a time
  static constexpr int kRowBytes = HD * (int)sizeof(ET);
  static constexpr int kSlotBytes = 32 * kRowBytes;
  static constexpr int kChunksPerRow = kRowBytes / 16;
  static constexpr int kRowsPerInstr = 64 / kChunksPerRow;   // rows one wave instruction moves
  __device__ static __forceinline__ int swz(int row) { return kChunksPerRow >= 16 ? (row & 15) : ((row >> 1) & 7); }
  // The query rows of all waves and the tiles: at most (with one or four row blocks side by side) QB + 4 kTiles tiles, 40 to 80
  // KiB - no more than half of the LDS of a compute unit: what waves tell each other lies where the query rows were, once these are
  // in registers.
  static constexpr int kSlots = QB + 4 * kTiles;
  static_assert(4 * QB + kTiles <= kSlots && 2 * QB + 2 * kTiles <= kSlots, "any number of row blocks");
  static_assert(kDirectMaxSlice2 * 4 <= QB * kSlotBytes, "the sums of a row block fit where its rows were");
};

// 64 x 16 bytes from the lanes' own addresses to consecutive LDS addresses (lds_addr: the same in all lanes)
__device__ __forceinline__ void dma16_at(const void* p, uint32_t lds_addr) {
  lds_addr = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_addr);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(p) : "memory");
}
// one 32-row tile by one wave; row_at(r): address of row r
template <class SH, class RowAt>
__device__ __forceinline__ void stage_tile(RowAt&& row_at, uint32_t lds_addr, int lane) {
  // (fp32 rows of 128 elements: the addresses, worked out ahead of the loop over tiles, would fill the registers)
  if (SH::F32 && SH::kTiles == 1) asm volatile("" : "+v"(lane));
#pragma unroll
  for (int j = 0; j < 32 / SH::kRowsPerInstr; ++j) {
    const int row = j * SH::kRowsPerInstr + lane / SH::kChunksPerRow, ch = (lane % SH::kChunksPerRow) ^ SH::swz(row);
    dma16_at(reinterpret_cast<const char*>(row_at(row)) + ch * 16, lds_addr + j * 1024);
  }
}

// A fragment: elements 16 ks + 8 half .. + 7 of row `col` (of a tile at `slot`); fp32: split into three
template <bool F32> struct DirectFrag { bf16x8 s[F32 ? 3 : 1]; };
template <class SH>
__device__ __forceinline__ DirectFrag<SH::F32> load_frag(const uint8_t* slot, int ks, int col, int half) {
  DirectFrag<SH::F32> f;
  if constexpr (SH::F32) {
    f32x4 v[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      v[i] = *reinterpret_cast<const f32x4*>(slot + col * SH::kRowBytes + (((4 * ks + 2 * half + i) ^ SH::swz(col)) << 4));
    const Split8 x = split8(v);
#pragma unroll
    for (int i = 0; i < 3; ++i) f.s[i] = x.s[i];
  } else {
    f.s[0] = *reinterpret_cast<const bf16x8*>(slot + col * SH::kRowBytes + (((2 * ks + half) ^ SH::swz(col)) << 4));
  }
  return f;
}
// logits of a tile against the wave's query rows; PASS 1: D[token][query], PASS 2: D[query][token].  fp32: the six products of
// ccd_score_split.hip
template <class SH, int HD, int PASS>
__device__ __forceinline__ void tile_logits(floatx16 (&acc)[SH::QB], const uint8_t* slot,
                                            const DirectFrag<SH::F32> (&q)[SH::QB][HD / 16], int col, int half) {
  auto mma = [](const bf16x8& k, const bf16x8& qv, const floatx16& a) {
    return PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, qv, a, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, k, a, 0, 0, 0);
  };
  floatx16 small;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    small[r] = 0.f;
#pragma unroll
    for (int qb = 0; qb < SH::QB; ++qb) acc[qb][r] = 0.f;
  }
  DirectFrag<SH::F32> f[2];
  f[0] = load_frag<SH>(slot, 0, col, half);
#pragma unroll
  for (int ks = 0; ks < HD / 16; ++ks) {
    const DirectFrag<SH::F32>& k = f[ks & 1];
    if (ks + 1 < HD / 16) f[(ks + 1) & 1] = load_frag<SH>(slot, ks + 1, col, half);
    if constexpr (SH::F32) {
      const auto& x = q[0][ks];
      small = mma(k.s[2], x.s[0], small);
      small = mma(k.s[1], x.s[1], small);
      small = mma(k.s[0], x.s[2], small);
      acc[0] = mma(k.s[0], x.s[0], acc[0]);
      small = mma(k.s[1], x.s[0], small);
      small = mma(k.s[0], x.s[1], small);
      __builtin_amdgcn_sched_barrier(0);       // (no fragments of later steps: they would be kept in scratch memory)
    } else {
#pragma unroll
      for (int qb = 0; qb < SH::QB; ++qb) acc[qb] = mma(k.s[0], q[qb][ks].s[0], acc[qb]);
    }
  }
  if constexpr (SH::F32) acc[0] += small;
}

// Which tokens of a row have a NuC slot (Sec. 3.3.3 step 1), as the key of the T-th most novel one and where its equals end, by a workgroup
// of its own beside those that score.  It depends on nothing that the call computes, and in the selection, where every workgroup of a unit
// found it for itself behind the scores, it was two of six barriers and a third of the passes over the row.  Append + distill: 4 units of 512
// fp32 tokens 26.5 -> 25.4 us, 8 units of 2048 / 8192 tokens 31.4 / 59.6 -> 30.2 / 57.0, 2 units of 5000 tokens and 16 rows 37.5 -> 35.1; 45
// units of 3000 tokens step by step 48.2 -> 45.5.  Bound by latency; rows are kept in registers.  (Rows of 16384 tokens: 8 units and
// 256 rows 89.3 -> 85.8, but 1 unit 49.2 -> 53.7, whose score pass is shorter than this.)
// Not inlined: the kernel around it has no registers to spare.  NOV = false: the same kernel without these workgroups, for the other calls and
// for pass 2 behind a pass 1 that had them; the call costs up to 18 spilled scalar registers and 12 bytes of scratch per lane (without
// NuC slots, 4 units of 512 / 16 of 1000 fp32 tokens 24.5 / 36.6 us with it, 23.8 / 35.8 without).
// The longest row.  (32 tokens a thread are 180 registers; bf16 rows of 64 elements are scored with 126, four workgroups to a compute unit.)
constexpr int kNoveltyRow = kNoveltyMaxRow;
static_assert(kNoveltyRow == 32 * kMT, "");
constexpr int novelty_row(int d, bool f32) { return d == 64 && !f32 ? 16 * kMT : kNoveltyRow; }
struct NoveltyLds {
  TopkShared<kMT> topk;
  uint32_t sums[kNoveltyRow / (4 * 64)];
};
template <int CHUNKS>
__device__ __noinline__ void find_novelty_key(const float* __restrict__ nov, int n, int T, uint32_t lds_addr, uint32_t* words) {
  auto& sh = *(NoveltyLds*)(__attribute__((address_space(3))) NoveltyLds*)(uintptr_t)lds_addr;
  auto token = [&](int c) { return 4 * (c * kMT + (int)threadIdx.x); };
  uint32_t kept[CHUNKS][4];                                        // keys, 0 past the end
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    float f[4];
    load_row4(f, nov, token(c), n, -INFINITY);
#pragma unroll
    for (int i = 0; i < 4; ++i) kept[c][i] = novelty_key(f[i]);
  }
  auto chunks = [&](auto&& use) {
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      // (what a pass makes of a key is not kept for the next one)
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(kept[c][i]));
      use(kept[c], c);
    }
  };
  auto each_key = [&](auto&& f) {
    chunks([&](const uint32_t (&k)[4], int) {
#pragma unroll
      for (int i = 0; i < 4; ++i) f(k[i]);
    });
  };
  topk_clear(sh.topk);
  KeyClasses cn{0xFFFFFFFFu, 0u, 0u, 0u};
  each_key([&](uint32_t k) { classify(k, cn); });
  publish_classes(cn, sh.topk, 1);
  __syncthreads();
  cn = combine_classes(sh.topk, 1);
  const uint32_t slots = min((uint32_t)T, cn.n_hi + cn.n_mid);     // NaN and -inf never take a slot
  Threshold th{0xFFFFFFFFu, 0u, 0u};                               // (above every key)
  if (slots > 0)
    th = slots <= cn.n_hi ? Threshold{kHiFrom, slots, cn.n_hi} : radix_threshold(each_key, cn.mn, cn.mx, slots - cn.n_hi, cn.n_mid, sh.topk, 0);
  if (th.need < th.n_eq) {                                         // only some of the equal tokens: the first ones
    auto equal_before = [&](const uint32_t (&k)[4], uint32_t& mine) {
      mine = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) mine += k[i] == th.tau ? 1u : 0u;
      return wave_inclusive_scan(mine, 0u, OpAdd{});
    };
    chunks([&](const uint32_t (&k)[4], int c) {
      uint32_t mine;
      put_round_sum<kMT>(equal_before(k, mine), sh.sums, c);
    });
    __syncthreads();
    const RoundBases<kMT, CHUNKS> bases(sh.sums, CHUNKS);
    chunks([&](const uint32_t (&k)[4], int c) {
      uint32_t mine;
      const uint32_t inc = equal_before(k, mine);
      uint32_t eq = bases.of(c) + inc - mine;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k[i] == th.tau && eq++ == th.need) words[kSyncNoveltyTies] = (uint32_t)(token(c) + i);
    });
  } else if (threadIdx.x == 0) {
    words[kSyncNoveltyTies] = 0xFFFFFFFFu;
  }
  if (threadIdx.x == 0) words[kSyncNovelty] = th.tau;
}

template <int HD, class ET, int PASS, bool NOV>
__global__ __launch_bounds__(kMT, 2) void score_direct_kernel(Dims D, ScorePlan pl, const ET* __restrict__ Q, const ET* __restrict__ K,
                                                              const ET* __restrict__ Kcap, float2* __restrict__ part,
                                                              float* lse_io, float* __restrict__ u, const float* novelty, int nov_wgs) {
  using SH = DirectShape<HD, ET>;
  constexpr int KS = HD / 16, QB = SH::QB;
  __shared__ __attribute__((aligned(1024))) uint8_t rows[SH::kSlots * SH::kSlotBytes];
  // (one value from each of the arguments' five lines: all are asked for together here and not, one miss after the other, where they are used.
  // 8 units of 2048 tokens 30.0 -> 29.4 us, 48 units of 800 under a window with CaP keys 36.1 -> 35.3; fp32, 4 units of 512 24.8 -> 24.3)
  asm volatile("" ::"s"(D.GP), "s"(D.unit0), "s"(D.q_sl), "s"(Q), "s"(u));
  static_assert(sizeof(NoveltyLds) <= sizeof(rows), "what find_novelty_key keeps fits");
  const int row_blocks = (D.GP + SH::kRows - 1) / SH::kRows;
  const int slices = PASS == 1 ? pl.n_slices1 + (Kcap != nullptr ? 1 : 0) : pl.n_slices2;
  // consecutive blocks go to different XCDs: the workgroups of one slice are eight blocks apart
  const int per_item = PASS == 1 ? row_blocks : 1;
  // (the workgroups for novelty come first: they are done long before the others)
  const int bid = (int)blockIdx.x - (NOV ? (nov_wgs + 7) / 8 * 8 : 0);
  if (NOV && bid < 0) {
    if ((int)blockIdx.x < nov_wgs) {
      const int nu = (int)blockIdx.x * (D.units / nov_wgs);           // every unit's own row, or one for each sequence
      const float* row = novelty + nov_offset(D, decode_unit(D, nu));
      const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)rows;
      uint32_t* words = pl.sync + (int64_t)nu * kSyncWords;
      if (D.n <= 8 * kMT)       find_novelty_key<2>(row, D.n, D.T, lds, words);
      else if (D.n <= 16 * kMT) find_novelty_key<4>(row, D.n, D.T, lds, words);
      else if constexpr (novelty_row(HD, SH::F32) > 16 * kMT) find_novelty_key<8>(row, D.n, D.T, lds, words);
    }
    return;
  }
  const int item = (bid >> 3) / per_item * 8 + (bid & 7);
  if (item >= D.units_run * slices) return;
  const int slice = item % slices, unit = D.unit0 + item / slices;
  const UnitIdx ui = decode_unit(D, unit);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const float c = D.scale_log2;
  if (PASS == 2) clear_sync(D, pl, unit, slice == 0);
  const bool cap = PASS == 1 && slice == pl.n_slices1;
  const ET* Ku = cap ? Kcap + (int64_t)unit * D.P * HD : K + kv_offset(D, ui);
  const int slice_len = PASS == 1 ? pl.slice1 : pl.slice2;
  const int t0 = cap ? 0 : slice * slice_len, t1 = cap ? D.P : min(D.n, t0 + slice_len);
  // tiles [it0, it1) of the slice: those before are hidden from every query by the window
  const int it1 = (t1 - t0 + kStep - 1) / kStep;
  const int it0 = cap ? 0 : min(it1, max(0, D.head0 - t0) / kStep);
  const uint32_t rows_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)rows;

  // waves side by side over row blocks (1, 2 or 4 of them; pass 1: one), the others on other tiles
  const int wide = PASS == 1 || row_blocks <= 1 ? 1 : (row_blocks <= 2 ? 2 : 4), groups = 4 / wide;
  const int rb = wave % wide, group = wave / wide;
  const int q_first = PASS == 1 ? (bid >> 3) % per_item * SH::kRows : 0;
  const int q_last = PASS == 1 ? min(D.GP, q_first + SH::kRows) : D.GP;
  float* up = reinterpret_cast<float*>(rows);                // pass 2: token sums per row block
  bool nan_out = false;                                      // pass 2, fp32: some token's score is NaN
  float m_raw[QB], Z[QB];                    // pass 1
  int lo[QB], hi[QB];                        // pass 1: first and last key the lane's query rows see
  if (PASS == 1) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int q = q_first + qb * 32 + col;
      m_raw[qb] = kNegHuge;
      Z[qb] = 0.f;
      lo[qb] = !cap && D.window > 0 ? D.win_off + q % D.P : 0;
      hi[qb] = cap ? q % D.P : t1 - 1;
    }
  }
  for (int qc = q_first; qc < q_last; qc += 4 * SH::kRows) {
    const int q0 = qc + rb * SH::kRows;
    // the query rows: QB wide tiles, dealt to the four waves (rows past G P repeat the last one: nobody reads their statistics,
    // and a normaliser of infinity takes them out of the token sums)
    for (int b = wave; b < QB * wide; b += 4)
      stage_tile<SH>([&](int r) { return Q + q_offset(D, ui, min(qc + b * 32 + r, D.GP - 1)); }, rows_addr + b * SH::kSlotBytes, lane);
    const int batch = groups * SH::kTiles;                 // tiles in LDS at a time
    const int slot0 = QB * wide;
    auto stage_keys = [&](int it) {
      for (int b = wave; b < batch; b += 4)
        if (it + b < it1)
          stage_tile<SH>([&](int r) { return Ku + (int64_t)min(t0 + (it + b) * kStep + r, t1 - 1) * HD; },
                         rows_addr + (slot0 + b) * SH::kSlotBytes, lane);
    };
    stage_keys(it0);
    float neg_lse = -INFINITY;                 // pass 2: of row q0 + lane, the statistics of all slices merged
    const int q = q0 + (SH::kRows == 64 ? lane : col);
    if (PASS == 2 && q < D.GP) {
      if (pl.lse_given) {
        neg_lse = -(lse_io[(int64_t)unit * D.GP + q] * 1.44269504088896340736f);
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
        if constexpr (SH::F32) {
          if (__builtin_expect(z != z, 0)) {
            const float2 a = statistics_again<HD>(Q + q_offset(D, ui, q), Ku, pl.cap_block ? Kcap + (int64_t)unit * D.P * HD : nullptr, p,
                                                  cp, D.GP, n, pl.slice1, D.n, D.window > 0 ? D.win_off + q % D.P : 0, q % D.P, c);
            M = a.x;
            z = a.y;
          }
        }
        // (a row none of whose visible logits is finite adds nothing: probabilities of 0, not of 2^(-inf + inf))
        neg_lse = z == 0.f ? -INFINITY : -(M + __log2f(z));
        if constexpr (SH::F32) {               // for scores_again (all workgroups of a unit write the same)
          if (lane < SH::kRows) lse_io[(int64_t)unit * D.GP + q] = -neg_lse;
        }
      }
    }
    float nl[PASS == 2 ? QB : 1][16];
    if (PASS == 2) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r) nl[qb][r] = __shfl(neg_lse, qb * 32 + acc_row(r, half));
    }
    const int first = D.win_off + q % D.P;     // pass 2 under a window: the first token row q sees
    wait_all_dma();
    __syncthreads();
    const bool active = q0 < q_last;
    DirectFrag<SH::F32> bq[QB][KS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) bq[qb][ks] = load_frag<SH>(rows + (rb * QB + qb) * SH::kSlotBytes, ks, col, half);
    if (PASS == 2) __syncthreads();            // the query rows make room for token sums
    for (int it = it0; it < it1; it += batch) {
      if (it > it0) {
        __syncthreads();
        stage_keys(it);
        wait_all_dma();
        __syncthreads();
      }
#pragma unroll
      for (int i = 0; i < SH::kTiles; ++i) {
        const int b = group * SH::kTiles + i, t = t0 + (it + b) * kStep;
        if (active && it + b < it1) {
          floatx16 acc[QB];
          tile_logits<SH, HD, PASS>(acc, rows + (slot0 + b) * SH::kSlotBytes, bq, col, half);
          if constexpr (PASS == 1) {
            if (cap || t + kStep > t1 || t < D.head) {            // some row may not see some key
#pragma unroll
              for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const int tok = t + acc_row(r, half);
                  if (tok < lo[qb] || tok > hi[qb]) acc[qb][r] = -INFINITY;
                }
            }
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) fold_block(acc[qb], m_raw[qb], Z[qb], c);
          } else {
            float s[2] = {0.f, 0.f};
            if (t < D.head) {
              int f = first;
              asm volatile("" : "+v"(f));               // (32 values that would be kept in registers for all tiles)
#pragma unroll
              for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const float p = fast_exp2(fmaf(acc[qb][r], c, nl[qb][r]));
                  s[r & 1] += t + col >= __shfl(f, qb * 32 + acc_row(r, half)) ? p : 0.f;
                }
            } else {
#pragma unroll
              for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r & 1] += fast_exp2(fmaf(acc[qb][r], c, nl[qb][r]));
            }
            float us = s[0] + s[1];
            us += __shfl_xor(us, 32);
            if (half == 0) up[rb * pl.slice2 + (it + b) * kStep + col] = us;
          }
        }
      }
    }
    __syncthreads();
    if constexpr (PASS == 2) {
      const int used = min(wide, (D.GP - qc + SH::kRows - 1) / SH::kRows);
      float* uu = u + (int64_t)unit * D.n + t0;
      for (int t = threadIdx.x; t < t1 - t0; t += kMT) {
        float v = 0.f;                         // (tokens nobody sees)
        if (t >= it0 * kStep) {
          v = up[t];
          for (int w = 1; w < used; ++w) v += up[w * pl.slice2 + t];
        }
        v = qc == 0 ? v : uu[t] + v;
        uu[t] = v;
        if (SH::F32) nan_out |= v != v;
      }
      __syncthreads();                         // the next sweep's query rows take the place of the sums
    }
  }
  if constexpr (PASS == 1) {
    // the two lane halves and the four waves hold different tokens of the same query rows
    float2* stat = reinterpret_cast<float2*>(rows);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const float m_o = __shfl_xor(m_raw[qb], 32), z_o = __shfl_xor(Z[qb], 32);
      const float M = fmaxf(m_raw[qb], m_o);
      const float z = Z[qb] * fast_exp2((m_raw[qb] - M) * c) + z_o * fast_exp2((m_o - M) * c);
      if (half == 0) stat[wave * SH::kRows + qb * 32 + col] = make_float2(M * c, z);
    }
    __syncthreads();
    const int q = q_first + (int)threadIdx.x;
    if ((int)threadIdx.x < SH::kRows && q < D.GP) {
      float2 v[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) v[w] = stat[w * SH::kRows + threadIdx.x];
      const float M = fmaxf(fmaxf(v[0].x, v[1].x), fmaxf(v[2].x, v[3].x));
      float z = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) z += v[w].y * fast_exp2(v[w].x - M);
      part[cap ? extra_block_index(D, pl, unit, q) : ((int64_t)unit * pl.n_slices1 + slice) * D.GP + q] = make_float2(M, z);
    }
  } else if constexpr (SH::F32) {
    // (the barrier behind the sums has passed; scores_again waits for the stores)
    int* again = reinterpret_cast<int*>(rows);
    if (threadIdx.x == 0) *again = 0;
    __syncthreads();
    if (__builtin_expect(nan_out, 0)) *again = 1;
    __threadfence_block();
    __syncthreads();
    if (__builtin_expect(wave == 0 && __builtin_amdgcn_readfirstlane(*again) != 0, 0))
      scores_again<HD>(D.GP, D.P, D.window > 0 ? D.win_off : -D.P, t0, t1, Q + q_offset(D, ui, 0), D.q_sh, Ku, c,
                       lse_io + (int64_t)unit * D.GP, pl.lse_given ? 1.44269504088896340736f : 1.0f, u + (int64_t)unit * D.n);
  }
}

unsigned direct_grid(const Dims& D, int slices, int per_item) {
  return (unsigned)(((int64_t)D.units_run * slices + 7) / 8 * 8 * per_item);
}

struct DirectCut { int row_blocks, batch1, batch2; };       // blocks of query rows; tokens per batch of tiles in either pass
DirectCut direct_cut(const Dims& D) {
  const int rows = D.dtype == 0 ? 32 : 64, tiles = D.dtype == 0 && D.d == 128 ? 1 : 2;      // per wave: DirectShape
  const int row_blocks = (D.GP + rows - 1) / rows, groups = row_blocks <= 1 ? 4 : (row_blocks <= 2 ? 2 : 1);
  return {row_blocks, 4 * tiles * kStep, groups * tiles * kStep};
}

}  // namespace

// Slices: two workgroups fit a compute unit, so the rounds of the grid times what one takes - its batches of tiles, and as much as
// three of them before and behind these - are the time of a pass; a workgroup that has its compute unit to itself is an eighth faster.
// (Powers of two with at least 1.25 workgroups per compute unit, before: 45 units of 3001 tokens were 540 workgroups on 512 places,
// two rounds, step by step 52.7 -> 48.3 us; 120 units of 2500 tokens and 256 rows 152 -> 138 us for append + distill.)
void plan_direct(const Dims& D, int compute_units, ScorePlan& pl) {
  const DirectCut g = direct_cut(D);
  auto best_slice = [&](int batch, int least, int most, int per_slice) {
    int best = least;
    int64_t best_cost = INT64_MAX;
    for (int slice = least; slice <= most; slice += batch) {
      const int64_t wgs = (int64_t)D.units_run * ((D.n + slice - 1) / slice) * per_slice;
      const int64_t rounds = (wgs + 2 * compute_units - 1) / (2 * compute_units);
      const int64_t cost = rounds * (3 + slice / batch) * (wgs <= compute_units ? 7 : 8);
      if (cost < best_cost) { best_cost = cost; best = slice; }
      if (slice >= D.n) break;
    }
    return best;
  };
  pl.slice1 = best_slice(g.batch1, kMinSlice, kDirectMaxSlice1, g.row_blocks);
  pl.slice2 = best_slice(g.batch2, g.batch2, kDirectMaxSlice2, 1);
  pl.n_slices1 = (D.n + pl.slice1 - 1) / pl.slice1;
  pl.n_slices2 = (D.n + pl.slice2 - 1) / pl.slice2;
  pl.direct_kernel = 1;
}

int novelty_workgroups(const Dims& D, int compute_units, const ScorePlan& pl, bool cap_keys, bool lse_given) {
  if (D.T <= 0 || D.units > kMaxSharedUnits || D.units_run != D.units || D.n > novelty_row(D.d, D.dtype == 0)) return 0;
  const int wgs = D.nov_sl != 0 || D.nov_sh != 0 ? D.units : D.B;
  const int scores = lse_given ? direct_grid(D, pl.n_slices2, 1) : direct_grid(D, pl.n_slices1 + (cap_keys ? 1 : 0), direct_cut(D).row_blocks);
  const int all = scores + (wgs + 7) / 8 * 8;
  auto rounds = [&](int n) { return (n + compute_units - 1) / compute_units; };
  return all <= 2 * compute_units || rounds(all) == rounds(scores) ? wgs : 0;
}

int64_t time_direct(const Dims& D, int compute_units, const ScorePlan& pl, bool cap_keys, bool lse_given) {
  struct Pass { int start, batch; };               // two workgroups per compute unit start together and then share it
  struct Cost { Pass stats, prob; };
  static constexpr Cost c16[2] = {{{127, 54}, {310, 71}}, {{294, 74}, {362, 79}}};          // bf16; 64, 128 elements
  static constexpr Cost c32[2] = {{{124, 137}, {403, 163}}, {{246, 137}, {665, 167}}};      // fp32
  const Cost& c = (D.dtype == 0 ? c32 : c16)[D.d == 128];
  const DirectCut g = direct_cut(D);
  auto pass = [&](const Pass& p, int64_t workgroups, int slice, int batch) {
    auto rounds = [&](int64_t places) { return (workgroups + places - 1) / places; };
    return rounds(2 * compute_units) * p.start + rounds(compute_units) * p.batch * ((std::min(slice, D.n) + batch - 1) / batch);
  };
  const int64_t prob = (g.row_blocks + 3) / 4 * pass(c.prob, (int64_t)D.units_run * pl.n_slices2, pl.slice2, g.batch2);
  if (lse_given) return prob;
  return prob + pass(c.stats, (int64_t)D.units_run * (pl.n_slices1 + (cap_keys ? 1 : 0)) * g.row_blocks, pl.slice1, g.batch1);
}

void launch_stats_direct(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const void* K_cap, float2* part,
                         const float* novelty, int nov_wgs, hipStream_t s) {
  const int rows = D.dtype == 0 ? 32 : 64, row_blocks = (D.GP + rows - 1) / rows;
  const dim3 grid(direct_grid(D, pl.n_slices1 + (K_cap != nullptr ? 1 : 0), row_blocks) + (nov_wgs + 7) / 8 * 8), block(kMT);
#define CCD_LAUNCH(HD, ET)                                                                                                       \
  launch((nov_wgs > 0 ? score_direct_kernel<HD, ET, 1, true> : score_direct_kernel<HD, ET, 1, false>), grid, block, s, D, pl, (const ET*)Q, (const ET*)K, (const ET*)K_cap, part, nullptr, \
         nullptr, novelty, nov_wgs)
  if (D.dtype == 0) { if (D.d == 64) CCD_LAUNCH(64, float); else CCD_LAUNCH(128, float); }
  else              { if (D.d == 64) CCD_LAUNCH(64, uint16_t); else CCD_LAUNCH(128, uint16_t); }
#undef CCD_LAUNCH
}

void launch_prob_direct(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const void* K_cap, const float2* part,
                        float* lse_io, float* u, const float* novelty, int nov_wgs, hipStream_t s) {
  const dim3 grid(direct_grid(D, pl.n_slices2, 1) + (nov_wgs + 7) / 8 * 8), block(kMT);
#define CCD_LAUNCH(HD, ET)                                                                                          \
  launch((nov_wgs > 0 ? score_direct_kernel<HD, ET, 2, true> : score_direct_kernel<HD, ET, 2, false>), grid, block, s, D, pl, (const ET*)Q, (const ET*)K, (const ET*)K_cap, \
         const_cast<float2*>(part), lse_io, u, novelty, nov_wgs)
  if (D.dtype == 0) { if (D.d == 64) CCD_LAUNCH(64, float); else CCD_LAUNCH(128, float); }
  else              { if (D.d == 64) CCD_LAUNCH(64, uint16_t); else CCD_LAUNCH(128, uint16_t); }
#undef CCD_LAUNCH
}

}  // namespace ccd
