// NuC slots + pooling + NuC lift + final top-k of one unit (Sec. 3.3.3), as a workgroup-level device function.
#pragma once
#include <float.h>

#include "ccd_common.h"
#include "ccd_topk.h"

namespace ccd {

// four consecutive floats whose address is only known to be a multiple of four bytes
struct __attribute__((packed, aligned(4))) Floats4 { float v[4]; };
__device__ __forceinline__ void store_row4(float* row, int t, int n, const float (&x)[4]) {
  if (t + 3 < n) {
    *reinterpret_cast<Floats4*>(row + t) = Floats4{{x[0], x[1], x[2], x[3]}};
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (t + i < n) row[t + i] = x[i];
  }
}
// elements t .. t + 3 of a row of n values; `fill` past the end
__device__ __forceinline__ void load_row4(float (&out)[4], const float* __restrict__ row, int t, int n, float fill) {
  // (one branch for the whole wave: a chunk loop keeps its vector loads in flight together)
  if (__all(t + 3 < n)) {
    const Floats4 f = *reinterpret_cast<const Floats4*>(row + t);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = f.v[i];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = row[min(t + i, n - 1)];
      out[i] = t + i < n ? v : fill;
    }
  }
}

constexpr int kPoolReach = 4;   // windows of up to 2 * 4 + 1 tokens are pooled from three vector loads

// elements j .. j + 3 of a row, `fill` before its start and past its end
__device__ __forceinline__ void load_clipped4(float (&v)[4], const float* __restrict__ u, int j, int n, float fill) {
  if (__all(j >= 0 && j + 3 < n)) {
    const Floats4 f = *reinterpret_cast<const Floats4*>(u + j);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = f.v[i];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = u[min(max(j + i, 0), n - 1)];
      v[i] = j + i >= 0 && j + i < n ? x : fill;
    }
  }
}
// Pooled scores of tokens t .. t + 3 for windows of more than 2 * kPoolReach + 1: four windows share all but three elements at
// either end, so they are pooled together, four elements a load, each window in the order of its elements.  Bound by these loads
// from the caches, a sixteenth of one load per element and window (select_compact with its score pass, windows of 31 / 255 tokens:
// 256 units of 4096 tokens 91 -> 68 us / 295 -> 99 us; 8 units of 65536 tokens, which pool in every step, 2.8 -> 0.56 ms).
template <bool MAX>
__device__ __forceinline__ void pooled_wide(float (&out)[4], const float* __restrict__ u, int t, int n, int w) {
  const int last = w - 1, first = t - (w >> 1);                // element o of the four: token first + o; window i: o in [i, i + last]
  const float fill = MAX ? __builtin_nanf("") : 0.f;           // (neutral: fmaxf passes over NaN)
  auto put = [&](int i, float v) { out[i] = MAX ? fmaxf(out[i], v) : out[i] + v; };
  float v[4];
  load_clipped4(v, u, first, n, fill);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[i] = fill;
#pragma unroll
    for (int e = i; e < 4; ++e) put(i, v[e]);
  }
  int o = 4;
#pragma unroll 1
  for (; o + 3 <= last; o += 4) {
    load_clipped4(v, u, first + o, n, fill);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) put(i, v[e]);
  }
#pragma unroll 1
  for (; o <= last + 3; o += 4) {
    load_clipped4(v, u, first + o, n, fill);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (o + e <= i + last) put(i, v[e]);
  }
  if (!MAX) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] /= (float)w;
  }
}

// Pooling straight from the row in global memory: the row was written by the kernel before this one and is served by the
// caches; a copy in LDS would cost a barrier and, for the longest rows, 128 KiB.  Two steps, so that a chunk loop can
// have the loads of several chunks in flight: `win` holds tokens t - 4 .. t + 7, the row's ends filled with what is neutral
// for the mode (max clips its window at the ends: a NaN never replaces a number, and a window of NaN stays NaN; avg pads with
// zeros).
struct PoolSpec {
  int n, w, mode;
  bool plain, wide;      // no pooling; a window that does not fit `win`
  __device__ __forceinline__ explicit PoolSpec(const Dims& D)
      : n(D.n), w(D.pool_w), mode(D.pool_mode), plain(D.pool_mode == 0 || D.pool_w <= 1), wide(D.pool_w > 2 * kPoolReach + 1) {}
};
__device__ __forceinline__ void pool_load(float (&win)[12], const float* __restrict__ u, int t, const PoolSpec& P) {
  if (P.wide) return;
  const float fill = P.mode == 1 ? __builtin_nanf("") : 0.f;
  if (__all(t >= 4 && t + 7 < P.n)) {
    const Floats4 a = *reinterpret_cast<const Floats4*>(u + t - 4), b = *reinterpret_cast<const Floats4*>(u + t),
                  c = *reinterpret_cast<const Floats4*>(u + t + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) { win[i] = a.v[i]; win[4 + i] = b.v[i]; win[8 + i] = c.v[i]; }
  } else {
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const int x = t - 4 + i;
      const float v = u[min(max(x, 0), P.n - 1)];
      win[i] = x >= 0 && x < P.n ? v : fill;
    }
  }
}
__device__ __forceinline__ void pool_reduce(float (&out)[4], const float (&win)[12], const float* __restrict__ u, int t,
                                            const PoolSpec& P) {
  if (P.plain) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = win[4 + i];
  } else if (P.wide) {
    if (P.mode == 1) pooled_wide<true>(out, u, t, P.n, P.w);
    else             pooled_wide<false>(out, u, t, P.n, P.w);
  } else {
    const int r = P.w >> 1;
    if (P.mode == 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = fmaxf(fmaxf(win[4 + i], win[3 + i]), win[5 + i]);      // r >= 1
#pragma unroll
      for (int o = 2; o <= kPoolReach; ++o) {
        if (o > r) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = fmaxf(fmaxf(out[i], win[4 + i - o]), win[4 + i + o]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = 0.f;
#pragma unroll
      for (int o = -kPoolReach; o <= kPoolReach; ++o) {
        if (o < -r || o > r) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] += win[4 + i + o];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] /= (float)P.w;
    }
  }
}

// Where the keys of a row live between the steps of its selection, by the length of the row:
//   CH = 1, 2, 4   registers: CH chunks of four tokens per thread (rows of up to 4 CH THREADS tokens)
//   kLdsRow        LDS (up to 32768 tokens: 128 KiB), first the novelty keys, then the score keys.  (In registers such a
//                  row takes hundreds of spilled scalar registers, the comparison masks of the unrolled steps.)
//   kLongRow       nowhere: every step pools the row again (up to 65536 tokens), LDS holds four lift flags per chunk
constexpr int kLdsRow = 0, kLongRow = -1;
constexpr int kLdsRowTokens = 32768, kMaxTokens = 65536;
template <int THREADS, int CH>
struct RowStore {
  static constexpr bool kRegs = CH > 0;
  static constexpr int kMaxChunks = kRegs ? CH : (CH == kLdsRow ? kLdsRowTokens : kMaxTokens) / (4 * THREADS);
  static constexpr int kLdsWords = kRegs ? 4 : (CH == kLdsRow ? kLdsRowTokens : kMaxTokens / 16);
};

template <int THREADS, int CH>
struct SelectShared {
  TopkShared<THREADS> topk;
  uint32_t sums[2][RowStore<THREADS, CH>::kMaxChunks * (THREADS / 64)];
  __attribute__((aligned(16))) uint32_t row[RowStore<THREADS, CH>::kLdsWords];
};

// One workgroup's view of one row: chunk loops, keys, novelty.  nov may be null when D.T == 0 and novelty is not carried.
template <int THREADS, int CH>
struct Row {
  using Store = RowStore<THREADS, CH>;
  static constexpr bool kRegs = Store::kRegs, kLds = CH == kLdsRow;
  const Dims& D;
  SelectShared<THREADS, CH>& sh;
  const float* u;          // raw scores, or null: the scores are given
  const float* given;
  const float* nov;
  const PoolSpec pool;
  int rounds;              // chunks per thread, whole groups
  uint32_t key[kRegs ? 4 * CH : 1];
  float nv[kRegs ? 4 * CH : 1];      // the thread's novelty
  uint64_t slots = 0;                // bit 4 c + i: token i of chunk c has a NuC slot (kLds, or where the slots are known)

  __device__ __forceinline__ Row(const Dims& D_, SelectShared<THREADS, CH>& sh_, int unit, const float* u_, const float* given_,
                                 const float* nov_)
      : D(D_), sh(sh_), u(u_ ? u_ + (int64_t)unit * D_.n : nullptr), given(given_ ? given_ + (int64_t)unit * D_.n : nullptr),
        nov(nov_), pool(D_),
        rounds(kRegs ? CH : (D_.n + 4 * THREADS * kGroup - 1) / (4 * THREADS * kGroup) * kGroup) {}
  __device__ __forceinline__ int token(int c) const { return 4 * (c * THREADS + (int)threadIdx.x); }
  // load(x, c) for kGroup chunks at a time, then use(x, c): a group's loads are in flight together.  Chunks past the end
  // are empty (their keys are 0).
  static constexpr int kGroup = kRegs ? CH : 4;
  static_assert(kRegs || Store::kMaxChunks % kGroup == 0, "whole groups fit");
  template <class X, class Load, class Use>
  __device__ __forceinline__ void chunks(Load&& load, Use&& use) {
    int c0 = 0;
#pragma unroll 1
    do {
      X x[kGroup];
#pragma unroll
      for (int g = 0; g < kGroup; ++g) load(x[g].v, kRegs ? g : c0 + g);
#pragma unroll
      for (int g = 0; g < kGroup; ++g) use(x[g].v, kRegs ? g : c0 + g);
      c0 += kGroup;
    } while (!kRegs && c0 < rounds);
  }
  struct Keys4 { uint32_t v[4]; };
  struct Vals4 { float v[4]; };
  struct Window { float v[12]; };

  // novelty: read once and kept (registers; LDS), or read from memory every time
  template <class Use>
  __device__ __forceinline__ void first_novelty_chunks(Use&& use) {
    if constexpr (kRegs) {
      each_novelty_chunk(use);
    } else {
      chunks<Vals4>([&](float (&f)[4], int c) { load_row4(f, nov, token(c), D.n, -INFINITY); },
                    [&](float (&f)[4], int c) {
                      const uint32_t k[4] = {novelty_key(f[0]), novelty_key(f[1]), novelty_key(f[2]), novelty_key(f[3])};
                      if (kLds) *reinterpret_cast<uint4*>(&sh.row[token(c)]) = make_uint4(k[0], k[1], k[2], k[3]);
                      use(k, c);
                    });
    }
  }
  template <class Use>
  __device__ __forceinline__ void each_novelty_chunk(Use&& use) {
    chunks<Keys4>(
        [&](uint32_t (&k)[4], int c) {
          if constexpr (kLds) {
            const uint4 v = *reinterpret_cast<const uint4*>(&sh.row[token(c)]);
            k[0] = v.x; k[1] = v.y; k[2] = v.z; k[3] = v.w;
          } else {
            float f[4];
            if constexpr (kRegs) {
#pragma unroll
              for (int i = 0; i < 4; ++i) f[i] = nv[4 * c + i];
            } else {
              load_row4(f, nov, token(c), D.n, -INFINITY);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) k[i] = novelty_key(f[i]);    // 0 past the end
          }
        },
        use);
  }
  // slots <- the tokens that the words of find_novelty_key give one
  __device__ __forceinline__ void take_slots(const uint32_t* words) {
    const uint32_t from = max(words[kSyncNovelty], 1u), ties_end = words[kSyncNoveltyTies];      // (the keys past the end are 0)
    auto take = [&](const uint32_t (&k)[4], int c) {
      uint32_t slot = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) slot |= k[i] > from || (k[i] == from && (uint32_t)(token(c) + i) < ties_end) ? 1u << i : 0u;
      slots |= (uint64_t)slot << (4 * c);
    };
    each_novelty_chunk(take);
  }
  __device__ __forceinline__ void load_novelty() {
    if constexpr (kRegs) {
      if (nov == nullptr) return;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        float f[4];
        load_row4(f, nov, token(c), D.n, -INFINITY);
#pragma unroll
        for (int i = 0; i < 4; ++i) nv[4 * c + i] = f[i];
      }
    }
  }
  // scores before the lift, in two steps (see pool_load)
  __device__ __forceinline__ void load_window(float (&win)[12], int c) const {
    if (u != nullptr) {
      pool_load(win, u, token(c), pool);
    } else {
      float f[4];
      load_row4(f, given, token(c), D.n, 0.f);
#pragma unroll
      for (int i = 0; i < 4; ++i) win[4 + i] = f[i];
    }
  }
  __device__ __forceinline__ void values(float (&f)[4], const float (&win)[12], int c) const {
    if (u != nullptr) {
      pool_reduce(f, win, u, token(c), pool);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (fabsf(f[i]) < FLT_MIN) f[i] = 0.f;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) f[i] = win[4 + i];
    }
  }
  // k: the chunk's score keys (0 past the end); lifted ones already hold the key of +inf where kLds
  __device__ __forceinline__ void put_keys(const uint32_t (&k)[4], int c) {
    if constexpr (kRegs) {
#pragma unroll
      for (int i = 0; i < 4; ++i) key[4 * c + i] = k[i];
    } else if constexpr (kLds) {
      *reinterpret_cast<uint4*>(&sh.row[token(c)]) = make_uint4(k[0], k[1], k[2], k[3]);
    } else {
      reinterpret_cast<uint8_t*>(sh.row)[token(c) >> 2] = 0;
    }
  }
  __device__ __forceinline__ void lift(uint32_t slot, int c) {         // bit i: token i of the chunk
    if constexpr (kRegs) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((slot >> i) & 1u) key[4 * c + i] = kHiFrom;
    } else if constexpr (kLds) {
      slots |= (uint64_t)slot << (4 * c);
    } else {
      reinterpret_cast<uint8_t*>(sh.row)[token(c) >> 2] = (uint8_t)slot;
    }
  }
  template <class Use>
  __device__ __forceinline__ void each_key_chunk(Use&& use) {
    chunks<Keys4>(
        [&](uint32_t (&k)[4], int c) {
          if constexpr (kRegs) {
#pragma unroll
            for (int i = 0; i < 4; ++i) k[i] = key[4 * c + i];
          } else if constexpr (kLds) {
            const uint4 v = *reinterpret_cast<const uint4*>(&sh.row[token(c)]);
            k[0] = v.x; k[1] = v.y; k[2] = v.z; k[3] = v.w;
          } else {
            float win[12], f[4];
            load_window(win, c);
            values(f, win, c);
            const uint32_t flags = reinterpret_cast<const uint8_t*>(sh.row)[token(c) >> 2];
#pragma unroll
            for (int i = 0; i < 4; ++i) k[i] = token(c) + i < D.n ? ((flags >> i) & 1u ? kHiFrom : score_key(f[i])) : 0u;
          }
        },
        use);
  }
};

// Executed by a whole workgroup of THREADS threads.
// row.u given: score <- pooled u with +inf at the NuC slots, written to `scores` if that is not null.
// else: score <- row.given.
// SELECT: emit(place, token, c, i) is called by the thread that owns it for every kept token (the top-k of score), in
// ascending order of a thread's tokens; c, i: its chunk and place in it.  Ends without a barrier.
//
// NUC: nuc_words, if not null, are what find_novelty_key has left for the row: the slots are known before the scores are read.
//
// Barriers, when the row's keys are ordinary, no bin holds more than 64 candidates and T > 0: classes (of novelty and
// scores together; one after the other where they take turns in LDS), two per threshold, ranks - six in all, or seven; four with known slots.
template <int THREADS, int CH, bool SELECT, bool NUC, class Emit>
__device__ __forceinline__ void select_row(Row<THREADS, CH>& row, float* scores_row, const uint32_t* nuc_words, Emit&& emit) {
  static_assert(!NUC || CH > 0, "rows in registers");
  using R = Row<THREADS, CH>;
  const Dims& D = row.D;
  SelectShared<THREADS, CH>& sh = row.sh;
  const int n = D.n;
  row.load_novelty();
  topk_clear(sh.topk);

  const bool lift = row.u != nullptr && D.T > 0;
  const bool known = NUC && lift && nuc_words != nullptr, find = lift && !known;
  const bool score_first = !R::kLds || !find;
  KeyClasses cs{0xFFFFFFFFu, 0u, 0u, 0u}, cn{0xFFFFFFFFu, 0u, 0u, 0u};
  auto score_stage = [&]() {
    row.template chunks<typename R::Window>(
        [&](float (&win)[12], int c) { row.load_window(win, c); },
        [&](float (&win)[12], int c) {
          float f[4];
          row.values(f, win, c);
          uint32_t k[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) k[i] = row.token(c) + i < n ? score_key(f[i]) : 0u;
          if (R::kLds || known) {
            const uint32_t slot = (uint32_t)(row.slots >> (4 * c)) & 15u;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if ((slot >> i) & 1u) { k[i] = kHiFrom; f[i] = INFINITY; }
          }
          // (else the slots of the NuC tokens are overwritten below)
          if (row.u != nullptr && scores_row != nullptr) store_row4(scores_row, row.token(c), n, f);
          if constexpr (SELECT) {
            row.put_keys(k, c);
#pragma unroll
            for (int i = 0; i < 4; ++i) classify(k[i], cs);
          }
        });
    if (SELECT) publish_classes(cs, sh.topk, 0);
  };
  if (known) row.take_slots(nuc_words);
  if (score_first) score_stage();
  if (find) {
    row.first_novelty_chunks([&](const uint32_t (&k)[4], int) {
#pragma unroll
      for (int i = 0; i < 4; ++i) classify(k[i], cn);
    });
    publish_classes(cn, sh.topk, 1);
  }
  if (SELECT || find) __syncthreads();

  uint32_t n_slots = 0;
  if (find) {
    cn = combine_classes(sh.topk, 1);
    n_slots = min((uint32_t)D.T, cn.n_hi + cn.n_mid);     // NaN and -inf never take a slot
  }
  if (n_slots > 0) {
    auto each_novelty_key = [&](auto&& f) {
      row.each_novelty_chunk([&](const uint32_t (&k)[4], int) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f(k[i]);
      });
    };
    const Threshold th = n_slots <= cn.n_hi
                             ? Threshold{kHiFrom, n_slots, cn.n_hi}
                             : radix_threshold(each_novelty_key, cn.mn, cn.mx, n_slots - cn.n_hi, cn.n_mid, sh.topk, 0);
    const bool some = th.need < th.n_eq;                  // only some of the equal tokens: by rank in token order
    auto equal_before = [&](const uint32_t (&k)[4], uint32_t& mine) {     // inclusive scan over the wave's round
      mine = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) mine += k[i] == th.tau ? 1u : 0u;
      return wave_inclusive_scan(mine, 0u, OpAdd{});
    };
    if (some) {
      row.each_novelty_chunk([&](const uint32_t (&k)[4], int c) {
        uint32_t mine;
        put_round_sum<THREADS>(equal_before(k, mine), sh.sums[0], c);
      });
      __syncthreads();
    }
    row.each_novelty_chunk([&](const uint32_t (&k)[4], int c) {
      uint32_t slot = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) slot |= k[i] >= th.tau ? 1u << i : 0u;
      if (some) {
        uint32_t mine;
        const uint32_t inc = equal_before(k, mine);
        uint32_t eq = RoundBases<THREADS, RowStore<THREADS, CH>::kMaxChunks>(sh.sums[0], row.rounds).of(c) + inc - mine;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (k[i] == th.tau && eq++ >= th.need) slot &= ~(1u << i);
      }
      if (!R::kLds && scores_row != nullptr) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if ((slot >> i) & 1u) scores_row[row.token(c) + i] = INFINITY;
      }
      if (SELECT || R::kLds) row.lift(slot, c);
    });
  }
  if (!score_first) {
    score_stage();
    if (SELECT) __syncthreads();
  }
  if constexpr (SELECT) {
    auto each_key = [&](auto&& f) {
      row.each_key_chunk([&](const uint32_t (&k)[4], int) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f(k[i]);
      });
    };
    cs = combine_classes(sh.topk, 0);
    if (find && score_first) {
      if (cs.n_mid < (uint32_t)n) {
        // rows with -inf, NaN or +inf among the pooled scores: which of them were lifted is only known now
        KeyClasses c2{0xFFFFFFFFu, 0u, 0u, 0u};
        each_key([&](uint32_t k) { classify(k, c2); });
        publish_classes(c2, sh.topk, 2);
        __syncthreads();
        cs = combine_classes(sh.topk, 2);
      } else {
        cs.n_hi = n_slots;                                // all ordinary before the lift; the range may be a little wide
        cs.n_mid = (uint32_t)n - n_slots;
      }
    }
    const uint32_t k = (uint32_t)D.k;
    Threshold th;
    if (k <= cs.n_hi)                 th = {kHiFrom, k, cs.n_hi};
    else if (k <= cs.n_hi + cs.n_mid) th = radix_threshold(each_key, cs.mn, cs.mx, k - cs.n_hi, cs.n_mid, sh.topk, 1);
    else                              th = {kLoUpTo, k - cs.n_hi - cs.n_mid, (uint32_t)n - cs.n_hi - cs.n_mid};
    // a token's place among the kept ones is the number of larger keys before it plus the number of threshold ties
    // before it, capped at `need`: both counts in one word (at most 65536 tokens, so exclusive counts fit 16 bits)
    auto count = [&](const uint32_t (&k)[4]) {
      uint32_t v = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) v += (k[i] > th.tau ? 0x10000u : 0u) + (k[i] == th.tau ? 1u : 0u);
      return v;
    };
    row.each_key_chunk([&](const uint32_t (&k)[4], int c) {
      put_round_sum<THREADS>(wave_inclusive_scan(count(k), 0u, OpAdd{}), sh.sums[1], c);
    });
    __syncthreads();
    const RoundBases<THREADS, RowStore<THREADS, CH>::kMaxChunks> bases(sh.sums[1], row.rounds);
    row.each_key_chunk([&](const uint32_t (&k)[4], int c) {
      const uint32_t mine = count(k);
      const uint32_t before = bases.of(c) + wave_inclusive_scan(mine, 0u, OpAdd{}) - mine;
      uint32_t gt = before >> 16, eq = before & 0xFFFFu;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool is_gt = k[i] > th.tau, is_eq = k[i] == th.tau;
        if (is_gt || (is_eq && eq < th.need)) emit((int)(gt + min(eq, th.need)), row.token(c) + i, c, i);
        gt += is_gt ? 1u : 0u;
        eq += is_eq ? 1u : 0u;
      }
    });
  }
}

}  // namespace ccd
