// Host side of libinfinipot: argument checks, workspace layout and kernel sequencing for the C ABI
// declared in include/infinipot.h.  Everything here runs before any launch; the kernels live in the
// ccd_*.hip files.
#include <cstdlib>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <vector>

#include "../../include/infinipot.h"
#include "ccd_kernels.h"
#include "ccd_launch.h"

// Workspace of ccd_compress_noalloc: one copy per GPU, held from the moment the library is loaded until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress (scratch_of_current_device below): the address
// it yields is what kernels, copies and memsets take.
static __device__ __align__(256) unsigned char scratch[CCD_NOALLOC_WORKSPACE_BYTES];

namespace ccd {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

enum Need { kNeedQ = 1, kNeedKV = 2, kNeedNov = 4, kNeedFull = 7 };

// Checks the fields a call reads; returns CCD_OK or an error code.
static int check_shape(const ccd_shape_t* s, int need) {
  if (s == nullptr) return CCD_EINVAL;
  if (s->B < 1 || s->L < 1 || s->Hkv < 1) return CCD_EINVAL;
  if (s->n_valid < 1 || s->k < 1 || s->k > s->n_valid) return CCD_EINVAL;
  if ((int64_t)s->B * s->L * s->Hkv > (int64_t)1 << 24) return CCD_EINVAL;
  if (s->n_valid > select_max_tokens()) return CCD_EUNSUPPORTED;
  if (need == 0) return CCD_OK;
  if (s->n_cap < s->n_valid) return CCD_EINVAL;
  if (s->dtype != CCD_FP32 && s->dtype != CCD_BF16) return CCD_EUNSUPPORTED;
  if (s->d != 64 && s->d != 128) return CCD_EUNSUPPORTED;
  const int64_t esz = s->dtype == CCD_FP32 ? 4 : 2;
  if (need & kNeedKV) {
    const int64_t row = (int64_t)s->n_cap * s->d;
    if (s->kv_stride_h < row || s->kv_stride_l < 0 || s->kv_stride_b < 0) return CCD_EINVAL;
    if ((s->kv_stride_b * esz) % 16 || (s->kv_stride_l * esz) % 16 || (s->kv_stride_h * esz) % 16) return CCD_EALIGN;
  }
  if (need & kNeedQ) {
    if (s->Hq < 1 || s->Hq % s->Hkv != 0 || s->P < 1) return CCD_EINVAL;
    if ((int64_t)(s->Hq / s->Hkv) * s->P > (1 << 20)) return CCD_EINVAL;
    if (s->q_stride_h < (int64_t)s->P * s->d || s->q_stride_l < 0 || s->q_stride_b < 0) return CCD_EINVAL;
    if ((s->q_stride_b * esz) % 16 || (s->q_stride_l * esz) % 16 || (s->q_stride_h * esz) % 16) return CCD_EALIGN;
    if (!(s->scale >= 0.f) || isinf(s->scale)) return CCD_EINVAL;
    if (s->pool_mode < CCD_POOL_NONE || s->pool_mode > CCD_POOL_AVG) return CCD_EUNSUPPORTED;
    if (s->pool_w < 1 || s->pool_w % 2 == 0) return CCD_EINVAL;
    if (s->window < 0 || (s->window > 0 && s->window < s->P)) return CCD_EINVAL;
    if (s->score_path < CCD_PATH_AUTO || s->score_path > CCD_PATH_MFMA_UNIT) return CCD_EINVAL;
    if (s->dtype != CCD_BF16 && s->score_path == CCD_PATH_MFMA_SLICES) return CCD_EUNSUPPORTED;
    // fp32 caches on the matrix cores: head dimension 64, no sliding window (and no CaP keys: checked with the call)
    if (s->dtype != CCD_BF16 && s->score_path == CCD_PATH_MFMA_UNIT && (s->d != 64 || s->window > 0)) return CCD_EUNSUPPORTED;
  }
  if (need & kNeedNov) {
    if (s->T < 0 || s->T > s->k) return CCD_EINVAL;
    if (s->nov_stride_b < 0 || s->nov_stride_l < 0 || s->nov_stride_h < 0) return CCD_EINVAL;
    const bool per_head = s->nov_stride_l != 0 || s->nov_stride_h != 0;
    if (per_head && s->nov_stride_h < s->n_cap) return CCD_EINVAL;
    if (!per_head && s->B > 1 && s->nov_stride_b < s->n_valid) return CCD_EINVAL;
  }
  return CCD_OK;
}

static Dims make_dims(const ccd_shape_t* s) {
  Dims D{};
  D.B = s->B; D.L = s->L; D.Hq = s->Hq; D.Hkv = s->Hkv; D.d = s->d;
  D.G = (s->Hq > 0 && s->Hkv > 0) ? s->Hq / s->Hkv : 0;
  D.n = s->n_valid; D.n_cap = s->n_cap; D.k = s->k; D.P = s->P; D.T = s->T;
  D.GP = D.G * s->P;
  D.pool_w = s->pool_w; D.pool_mode = s->pool_mode; D.dtype = s->dtype;
  D.units = s->B * s->L * s->Hkv;
  D.unit0 = 0;
  D.units_run = D.units;
  const double scale = s->scale > 0.f ? (double)s->scale : 1.0 / sqrt((double)(s->d > 0 ? s->d : 1));
  D.scale_log2 = (float)(scale * 1.4426950408889634074);
  D.score_path = s->score_path;
  D.window = s->window;
  D.win_off = s->window > 0 ? s->n_valid + 1 - s->window : 0;
  D.head = 0;
  D.head0 = 0;
  if (s->window > 0 && s->n_valid + s->P > s->window) {
    const int64_t hidden = (int64_t)s->n_valid + s->P - s->window;        // tokens hidden from the last CaP token
    D.head = (int)((hidden + 31) / 32 * 32 < s->n_valid ? (hidden + 31) / 32 * 32 : s->n_valid);
    const int64_t unseen = (int64_t)s->n_valid + 1 - s->window;           // tokens hidden from the first one, so from all
    D.head0 = unseen > 0 ? (int)(unseen / 32 * 32) : 0;
    if (D.head0 > D.head) D.head0 = D.head;
  }
  D.kv_sb = s->kv_stride_b; D.kv_sl = s->kv_stride_l; D.kv_sh = s->kv_stride_h;
  D.q_sb = s->q_stride_b; D.q_sl = s->q_stride_l; D.q_sh = s->q_stride_h;
  D.nov_sb = s->nov_stride_b; D.nov_sl = s->nov_stride_l; D.nov_sh = s->nov_stride_h;
  return D;
}

// compute units of the current device (asked once; the answer of the first device serves all: one GPU model per node)
static int compute_units() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0;
    hipDeviceProp_t prop;
    int n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.multiProcessorCount;
    cus = n > 0 ? n : 256;
  }
  return cus;
}
// workgroup slots for the slice kernels of the score passes (two workgroups per compute unit)
static int score_slots() { return 2 * compute_units(); }

// Token slice per workgroup: the longest of 2048 / 1024 / 512 / 256 that still gives every slot a workgroup.  Long
// slices amortise the per-workgroup prologue, and a grid of exactly one round has no half-empty last round (the
// headline shape: 256 units x 2 slices of 2048 = 512 workgroups on 512 slots, 6 us per pass less than 4 slices of
// 1024 in two rounds).
static int pick_slice(const Dims& D) {
  const int64_t slots = score_slots();
  for (int slice = mfma_max_slice(); slice > kMinSlice; slice /= 2)
    if ((int64_t)D.units_run * ((D.n + slice - 1) / slice) >= slots) return slice;
  return kMinSlice;
}

// What the two passes of the bf16 slice kernels take, in units of 10 ns (as time_direct, with which it is compared): per round of two
// workgroups per compute unit and sweep of 256 query rows, which then share the unit for their tiles of 32 tokens; pass 2 merges the
// statistics of all slices and computes with the CaP keys in every workgroup; a window takes two kernels more.
static int64_t time_mfma(const Dims& D, const ScorePlan& pl, bool cap_keys, bool lse_given) {
  struct Pass { int start, tile; };
  struct Cost { Pass stats, prob; int merge_slice, cap_token, head; };
  static constexpr Cost c64{{260, 13}, {310, 18}, 7, 4, 475}, c128{{480, 13}, {420, 17}, 14, 4, 515};
  const Cost& c = D.d == 64 ? c64 : c128;
  const int64_t wgs = (int64_t)(D.units_run + 7) / 8 * 8 * pl.n_slices1, cus = compute_units();
  const int64_t rounds = (wgs + 2 * cus - 1) / (2 * cus), shares = rounds + (wgs + cus - 1) / cus;
  const int64_t sweeps = (D.GP + 255) / 256, tiles = ((pl.slice1 < D.n ? pl.slice1 : D.n) + 31) / 32;
  int64_t t = rounds * (c.prob.start + (cap_keys ? D.P * c.cap_token : 0)) + shares * tiles * c.prob.tile;
  if (!lse_given) t += rounds * (c.stats.start + pl.n_slices1 * c.merge_slice) + shares * tiles * c.stats.tile;
  return sweeps * t + (D.head > 0 ? (lse_given ? 1 : 2) * c.head : 0);
}

// Calls that do not take the unit kernel: do the direct kernels pay against those that cut by longer slices, which take `other`?  They
// compute query rows by 64 (fp32: 32) instead of 256 and start faster; the others keep the matrix cores busier once their grid
// fills its rounds, and split an fp32 key once for 256 rows.  Both sides were timed on 11000 calls, 1 to 400 units, 256 to 32768 tokens, 4
// to 1600 rows, both types and head dimensions, with every option.  A 25th less is asked for: of those that then go to the direct kernels, 1 in
// 150 is more than 1.5 % slower with them (append + distill; 8 % at most), of those that do not, 1 in 9 would have been that much faster (14 %
// at most).  Append + distill, others against direct, us:
//   bf16, 128 elements, 256 rows   8 units of 2048 tokens 39.7 / 30.7, of 32768 135 / 131; 16 / 64 / 128 units of 16384 / 4096 / 2048 tokens,
//                                  grids of whole rounds, 132 / 113 / 110 against 137 / 122 / 118; 64 units of 2560 tokens, a fifth beyond one
//                                  round, 103 / 89; the same with given normalisers, of 1024 / 2560 tokens 36.5 / 71.0 against 40.5 / 68.6
//   bf16, 64 elements, 132 rows    82 units of 31297 tokens, given normalisers 418 / 446
//   fp32, 128 elements             4 units of 820 tokens, 100 rows 51 / 33; 256 units of 4000, 16 rows 755 / 726; 48 units of 1024, 160 rows 13 %
//                                  slower direct; 4 units of 12000, 160 rows 16 % faster
static bool direct_pays(const Dims& D, const ScorePlan& direct, int64_t other, bool cap_keys, bool lse_given) {
  return 26 * time_direct(D, compute_units(), direct, cap_keys, lse_given) < 25 * other;
}

// Does the unit kernel leave a windowed head to the two head kernels?  It deals the head's tiles of 32 tokens to its four waves one by one,
// masked and not pipelined, once per sweep of query rows; the head kernels run several workgroups per compute unit, but cost two
// launches and the normalisers' way through memory.  Append + distill of 160 to 512 units, 512 to 4096 tokens, head kernels against masks:
//   one sweep of up to 256 rows   up to 128 tokens 1.02 to 1.13 times faster by masks (median 1.05), 160 tokens 0.81 to 1.03, 1900 tokens 0.64 to 1.02
//   several sweeps of 256         96 and 128 tokens 1.02 to 1.08 (medians), 32 and 64 tokens 0.93 to 1.01, 160 tokens 0.81 to 1.00
//   one sweep of 384 to 1024      32 and 64 tokens, 170 to 512 units of 600 to 4096 tokens: 1.02 to 1.21 in all of 76 calls (median 1.05)
//   two sweeps of 1024            64 tokens 0.98 to 1.16 (median 1.06)
// The line for 32 and 64 tokens is the one of sweeps of 256 rows, and on the safe side for wider ones: 257 to 1024 rows could go by masks.
static bool head_apart(const Dims& D) {
  const int head = D.head - D.head0;
  return head > 128 || (head > 0 && head <= 64 && D.GP > 256);
}

static ScorePlan plan_mfma(const Dims& D, bool cap_keys, bool lse_given) {
  ScorePlan pl{};
  pl.use_mfma = 1;
  pl.slice1 = pl.slice2 = pick_slice(D);   // multiples of 32, at most mfma_max_slice()
  pl.n_slices1 = (D.n + pl.slice1 - 1) / pl.slice1;
  pl.n_slices2 = (D.n + pl.slice2 - 1) / pl.slice2;
  pl.cap_block = 0;
  pl.head_block = 0;
  pl.lse_given = 0;
  // One workgroup per unit (both passes in one kernel) when the units fill at least three fifths of the chip (what is left of the
  // units after whole rounds: units_in_whole_rounds); kernels that cut a unit into token slices otherwise.  Unit against slice
  // kernels, measured on the headline shape with 128 / 192 / 256 units: 180 / 223 / 220 us per call against 147 / 246 / 233 us, and with
  // 32 to 128 query rows per unit (the unit kernel then sweeps 64 or 128 rows at a time) it is 15 - 20 % ahead.
  if (D.score_path == CCD_PATH_MFMA_UNIT) {
    pl.unit_kernel = 1;
  } else if (D.score_path == CCD_PATH_AUTO && score_unit_supported(D)) {
    pl.unit_kernel = 5 * D.units_run >= 3 * compute_units() ? 1 : 0;
    // A few units beyond one round that fit one round of the slice kernels: with one slice per unit these are done before a unit
    // kernel and its rest have started.  Append + distill of 257 to 307 units, unit kernel and rest against slice kernels for all, medians by
    // up to 64 / 128 / 256 query rows: up to 256 tokens 0.98 / 1.10 / 1.26 (given normalisers 1.12 / 1.26 / 1.45) times longer, 257 to 512
    // tokens 0.80 / 0.90 / 0.96 (0.96 / 1.05 / 1.13).  Five sweeps of 256 rows: up to 256 tokens 1.06 to 1.25 (1.33 to 1.7), 500 tokens (1.07).  With
    // 264 to 1024 rows in one sweep the unit kernel has overtaken: up to 256 tokens 0.83 to 1.01 (CaP keys and 100 tokens to 1.13; given
    // normalisers 1.04 to 1.25), 257 to 512 tokens (0.80 to 0.97); the line does not make that difference yet.
    const bool one_round = D.units_run > compute_units() && 5 * D.units_run < 6 * compute_units();
    if (one_round && (lse_given ? pl.n_slices1 == 1 || (pl.n_slices1 == 2 && D.GP > 64) : pl.n_slices1 == 1 && D.GP > 64)) {
      pl.unit_kernel = 0;
      return pl;
    }
  }
  if (D.score_path == CCD_PATH_AUTO && !pl.unit_kernel) {
    ScorePlan direct = pl;
    plan_direct(D, compute_units(), direct);
    if (direct_pays(D, direct, time_mfma(D, pl, cap_keys, lse_given), cap_keys, lse_given)) return direct;
  }
  return pl;
}

ScorePlan plan_score(const Dims& D, bool cap_keys, bool lse_given) {
  ScorePlan pl{};
  pl.use_mfma = (D.dtype == CCD_BF16 && D.score_path != CCD_PATH_VALU) ? 1 : 0;
  // a windowed head longer than the head kernels take (about 2000 CaP tokens under a window), which the slice kernels need for any
  // head and the unit kernel for long ones: the vector-ALU kernels mask inside their loops, so the automatic choice goes there (also
  // the few units that the direct kernels, which mask a head of any length, could have)
  if (pl.use_mfma && D.score_path == CCD_PATH_AUTO && D.head - D.head0 > mfma_max_slice()) pl.use_mfma = 0;
  if (pl.use_mfma) {
    return plan_mfma(D, cap_keys, lse_given);
  } else {
    pl.slice1 = kMinSlice;
    pl.slice2 = 256;   // one token per thread
  }
  pl.n_slices1 = (D.n + pl.slice1 - 1) / pl.slice1;
  pl.n_slices2 = (D.n + pl.slice2 - 1) / pl.slice2;
  pl.cap_block = 0;
  pl.head_block = 0;
  pl.lse_given = 0;
  // The unit kernel (fp32 values as sums of three bf16 products, logits good to 2^-16 of sum |q k| only; head dimension 64, plain softmax
  // over the cached tokens) when asked for, and by itself from half of the chip's units on: 140 units of 1200 tokens and 16 rows 78 (direct)
  // against 76 us; 127 units and 256 rows, 7000 / 16384 tokens 525 / 1203 (six products) against 452 / 1016 us.  With more
  // than one block of rows from a third on while the rows are short (120 units of 2500 tokens and 100 / 256 rows 145 / 187 against 134 /
  // 170 us; 64 units 92 / 117 against 105 / 140 us).  Long rows stay with six products there: they are the more accurate ones, and the
  // unit kernel is not faster everywhere (81 / 100 units of 7000 tokens and 64 rows 257 / 318 against 276 / 321 us).  The bound counts in 256 rows, also
  // where the unit kernel sweeps more at once and would be faster with less accurate logits: 384 to 1024 rows, 4000 and 6000 tokens, 81
  // units 0.93 to 0.97, 90 and 100 units 1.05 to 1.16, 115 and 127 units 1.19 to 1.33 times.
  // Every other fp32 call: six bf16 products (256 units of 4096 tokens, 256 query rows of 128 elements: append + distill 1.16 ms
  // against 3.61 ms on the vector ALUs, which stay for those who name them), in the direct kernels for a single block of 32 rows, which leaves
  // the kernels by longer slices mostly empty, and where these do not pay (direct_pays).
  if (D.dtype == CCD_FP32) {
    const int cus = compute_units();
    const int64_t rows = (D.GP + 31) / 32, sweeps = (D.GP + 255) / 256;
    const bool unit = score_unit_supported(D) && !cap_keys && D.window == 0;
    if (unit && D.score_path == CCD_PATH_MFMA_UNIT) {
      pl.unit_kernel = 1;
    } else if (D.score_path == CCD_PATH_AUTO) {
      if (unit && (2 * D.units_run >= cus || (rows > 1 && 16 * D.units_run > 5 * cus && sweeps * D.n <= 6000))) {
        pl.unit_kernel = 1;
        return pl;
      }
      ScorePlan direct = pl;
      plan_direct(D, cus, direct);
      if (rows == 1) return direct;
      plan_split(D, cus, kMinSlice, pl);
      if (direct_pays(D, direct, time_split(D, cus, pl, cap_keys, lse_given), cap_keys, lse_given)) return direct;
    }
  }
  return pl;
}
// a path the caller named that this call cannot take
static bool path_refused(const Dims& D, const ScorePlan& pl) {
  return D.dtype == CCD_FP32 && D.score_path == CCD_PATH_MFMA_UNIT && !pl.unit_kernel;
}

// The leading units of a call that the unit kernel takes; the plan of the others is made for them alone.  One workgroup fits a
// compute unit, so a few units beyond whole rounds cost a round of their own, while kernels that cut them into slices spread them
// over the chip - for two launches, and more time per token: a last round that is half empty runs faster than a full one (more
// bandwidth and clock for those who are there).  Scores of all units by the unit kernel against such a rest by itself, append + distill:
//   rest of 8 / 32 / 64 (at most a quarter of the chip): 1200 tokens and 16 rows 133 / 138 / 145 against 124 / 130 / 140 us, 2500
//   tokens and 256 rows 300 / 321 / 355 against 257 / 294 / 351 us; 300 tokens and 16 rows 58 / 60 / 62 against 61 / 63 / 65 us
//   rest of 128: 2500 tokens and 256 rows 676 against 695 us, 8192 tokens and 256 rows 1798 against 1768 us, 32768 tokens and 1024
//   rows 15.0 against 14.2 ms
//   384 to 1024 rows in one sweep, 300 / 1200 / 4096 / 16384 tokens: rests of 8 and 32 0.88 to 0.95 / 0.78 to 0.92 / 0.75 to 0.85 / 0.69 to 0.90
//   of the time, of 64 1.02 to 1.04 (512 rows 0.98) / 0.94 to 0.98 / 0.88 to 0.93 / 0.80 to 0.91, of 128 and 16384 tokens 0.91 to 0.99
//   fp32 (three products for the whole rounds, six for the rest), 16384 tokens and 256 rows, rest of 64 / 80: 2264 / 2324 against 2122 /
//   2279 us; rest of 100 / 127: 2384 / 2481 against 2437 / 2642 us
static int units_in_whole_rounds(const Dims& D, const ScorePlan& pl, bool cap_keys, bool lse_given) {
  if (!pl.unit_kernel || D.score_path != CCD_PATH_AUTO) return D.units_run;
  const int cus = compute_units(), rest = D.units_run % cus;
  if (rest == 0 || rest == D.units_run) return D.units_run;
  Dims R = D;
  R.units_run = rest;
  const int64_t work = (int64_t)D.n * ((D.GP + 63) / 64) * D.d;
  const bool half = D.dtype == CCD_FP32 && D.GP > 32 ? 16 * rest <= 5 * cus : 2 * rest <= cus;
  const bool pays = 4 * rest <= cus ? work >= 128 * 1000 : (half && work >= 128 * 32768);
  return pays && !plan_score(R, cap_keys, lse_given).unit_kernel ? D.units_run - rest : D.units_run;
}

struct Workspace {
  size_t off_part, off_lse, off_u, off_sync, total;
};

// The layout does not depend on the kernel path, so a workspace sized once serves either.
static Workspace layout_workspace(const Dims& D) {
  Workspace w{};
  size_t off = 0;
  const size_t max_slices = (D.n + kMinSlice - 1) / kMinSlice + 1;   // + the block of the CaP keys (causal variant)
  w.off_part = off;   off = align_up(off + (size_t)D.units * max_slices * D.GP * sizeof(float2), 256);
  w.off_lse = off;    off = align_up(off + (size_t)D.units * D.GP * sizeof(float), 256);
  w.off_u = off;      off = align_up(off + (size_t)D.units * D.n * sizeof(float), 256);
  w.off_sync = off;
  if (D.units <= kMaxSharedUnits) off = align_up(off + (size_t)D.units * kSyncWords * sizeof(uint32_t), 256);   // 8 KiB at most
  w.total = off;
  return w;
}

static int check_workspace(const Workspace& w, const void* ws, size_t ws_bytes) {
  if (ws == nullptr || ws_bytes < w.total) return CCD_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 255u) return CCD_EWORKSPACE;
  return CCD_OK;
}

// ---- optional per-kernel timing of ccd_compress -------------------------------------------------------
enum Stage { kStStats = 0, kStMerge, kStProb, kStSelect, kStCompact, kStSelCompact, kStCapBlock, kStHead, kStUnit, kNumStages };
static const char* const kStageNames[kNumStages] = {"score_stats", "score_merge",    "score_prob", "select",     "compact",
                                                    "select_compact", "cap_block",   "window_head", "score_unit"};

// A timed stage owns two events; the kernels launched while it is open take them along (ccd_launch.h): the first
// kernel's begin stamp and the last kernel's end stamp are what the stage reports.
StageTimer* g_stage_timer = nullptr;
struct Profiler {
  bool on = false;
  std::vector<hipEvent_t> pool;       // every event ever created
  size_t used = 0;                    // events handed out since the last collect
  std::vector<int> stage_of;          // stage of the span that starts at event 2*i
  int64_t calls = 0;
  StageTimer timer{nullptr, nullptr, false};
  hipEvent_t next() {
    if (used == pool.size()) {
      hipEvent_t e;
      // (no system-scope fence with these events: cache write-backs and invalidations at every kernel boundary would
      // change the very durations being measured)
      if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
      pool.push_back(e);
    }
    return pool[used++];
  }
  void begin(int stage, hipStream_t) {
    if (!on) return;
    timer.start = next();
    timer.stop = next();
    timer.first = true;
    stage_of.push_back(stage);
    if (timer.start && timer.stop) g_stage_timer = &timer;
  }
  void end(hipStream_t) { g_stage_timer = nullptr; }
};
static Profiler g_prof;

static int launch_status() { return hipGetLastError() == hipSuccess ? CCD_OK : CCD_ELAUNCH; }

// Raw CaP score u[unit, t] (Eq. 2, before pooling).  With K_cap the CaP tokens' own keys join the softmax (causally): their
// statistics become one more entry per unit of `part` (vector ALUs, six-product and direct kernels; the bf16 slice and unit kernels
// compute them in pass 2).
// lse (nullable): the caller's natural-log-sum-exp of every CaP query row [units, G*P]: the statistics pass (and
// with it K_cap) is not needed, the probabilities follow from one pass over K.
// novelty (nullable): the tokens with a NuC slot (Sec. 3.3.3 step 1) are found along the way where a kernel does that; returns whether.  (Else
// the selection kernels find them from the novelty row.)
static bool run_cap_scores(const Dims& D, ScorePlan pl, const Workspace& w, const void* Q, const void* K,
                           const void* K_cap, const float* lse, const float* novelty, char* ws, hipStream_t st) {
  const int lead = units_in_whole_rounds(D, pl, K_cap != nullptr, lse != nullptr);
  if (lead < D.units_run) {
    Dims part = D;
    part.units_run = lead;
    run_cap_scores(part, pl, w, Q, K, K_cap, lse, nullptr, ws, st);
    part.unit0 = D.unit0 + lead;
    part.units_run = D.units_run - lead;
    ScorePlan rest = plan_score(part, K_cap != nullptr, lse != nullptr);
    rest.sync = pl.sync;             // (a partition of few compute units: the rest of a call whose units are shared has words to clear too)
    run_cap_scores(part, rest, w, Q, K, K_cap, lse, nullptr, ws, st);
    return false;
  }
  const int nov_wgs = pl.direct_kernel && pl.sync != nullptr && novelty != nullptr
                          ? novelty_workgroups(D, compute_units(), pl, K_cap != nullptr && lse == nullptr, lse != nullptr) : 0;
  float2* part = reinterpret_cast<float2*>(ws + w.off_part);
  float* lse2 = reinterpret_cast<float*>(ws + w.off_lse);
  float* u = reinterpret_cast<float*>(ws + w.off_u);
  if (pl.unit_kernel) {
    // statistics, merge and probabilities of every unit in one kernel; a windowed head inside, or before and behind it by two small kernels
    pl.lse_given = lse != nullptr ? 1 : 0;
    pl.head_apart = head_apart(D) ? 1 : 0;
    pl.head_block = pl.head_apart && lse == nullptr ? 1 : 0;
    float* lse_io = lse != nullptr ? const_cast<float*>(lse) : lse2;   // only read when pl.lse_given
    if (pl.head_block) {
      g_prof.begin(kStHead, st);
      launch_head_stats_mfma(D, pl, Q, K, part, st);
      g_prof.end(st);
    }
    g_prof.begin(kStUnit, st);
    launch_score_unit(D, pl, Q, K, K_cap, part, u, lse_io, st);
    g_prof.end(st);
    if (pl.head_apart) {
      g_prof.begin(kStHead, st);
      launch_head_prob_mfma(D, pl, Q, K, lse_io, u, st);
      g_prof.end(st);
    }
    return false;
  }
  if (lse != nullptr) {
    pl.lse_given = 1;
    float* lse_rw = const_cast<float*>(lse);   // only read when pl.lse_given
    g_prof.begin(kStProb, st);
    if (pl.direct_kernel)     launch_prob_direct(D, pl, Q, K, nullptr, part, lse_rw, u, novelty, nov_wgs, st);
    else if (pl.use_mfma)     launch_prob_mfma(D, pl, Q, K, nullptr, part, u, lse_rw, st);
    else if (pl.split_kernel) launch_prob_split(D, pl, Q, K, lse, u, st);
    else                      launch_prob_valu(D, pl, Q, K, lse, u, st);
    g_prof.end(st);
    if (pl.use_mfma && !pl.direct_kernel && D.head > 0) {
      g_prof.begin(kStHead, st);
      launch_head_prob_mfma(D, pl, Q, K, lse, u, st);
      g_prof.end(st);
    }
    return nov_wgs > 0;
  }
  if (K_cap != nullptr && (!pl.use_mfma || pl.direct_kernel)) pl.cap_block = 1;   // (launch_prob_mfma takes the CaP keys in its prologue)
  if (pl.direct_kernel) {
    g_prof.begin(kStStats, st);
    launch_stats_direct(D, pl, Q, K, K_cap, part, novelty, nov_wgs, st);
    g_prof.end(st);
    g_prof.begin(kStProb, st);
    launch_prob_direct(D, pl, Q, K, K_cap, part, lse2, u, nullptr, 0, st);
    g_prof.end(st);
    return nov_wgs > 0;
  }
  if (pl.cap_block && !pl.split_kernel) {
    g_prof.begin(kStCapBlock, st);
    launch_cap_block_stats_valu(D, pl, Q, K_cap, part, st);
    g_prof.end(st);
  }
  if (pl.use_mfma) {
    if (D.head > 0) {                        // sliding window: the tokens some CaP token does not see
      pl.head_block = 1;
      g_prof.begin(kStHead, st);
      launch_head_stats_mfma(D, pl, Q, K, part, st);
      g_prof.end(st);
    }
    g_prof.begin(kStStats, st);
    launch_stats_mfma(D, pl, Q, K, part, st);
    g_prof.end(st);
    g_prof.begin(kStProb, st);
    launch_prob_mfma(D, pl, Q, K, K_cap, part, u, lse2, st);
    g_prof.end(st);
    if (D.head > 0) {
      g_prof.begin(kStHead, st);
      launch_head_prob_mfma(D, pl, Q, K, lse2, u, st);
      g_prof.end(st);
    }
  } else {
    g_prof.begin(kStStats, st);
    if (pl.split_kernel) launch_stats_split(D, pl, Q, K, K_cap, part, st);
    else                 launch_stats_valu(D, pl, Q, K, part, st);
    g_prof.end(st);
    g_prof.begin(kStMerge, st);
    launch_merge(D, pl, Q, K, K_cap, part, lse2, st);
    g_prof.end(st);
    g_prof.begin(kStProb, st);
    if (pl.split_kernel) launch_prob_split(D, pl, Q, K, lse2, u, st);
    else                 launch_prob_valu(D, pl, Q, K, lse2, u, st);
    g_prof.end(st);
  }
  return false;
}

}  // namespace ccd

using namespace ccd;

extern "C" {

size_t ccd_workspace_bytes(const ccd_shape_t* shape) {
  if (check_shape(shape, kNeedFull) != CCD_OK) return 0;
  const Dims D = make_dims(shape);
  return layout_workspace(D).total;
}

static int score_impl(const ccd_shape_t* shape, const void* Q_cat, const void* K, const void* K_cap, const float* lse,
                      const float* novelty, float* scores, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_shape(shape, kNeedFull);
  if (rc != CCD_OK) return rc;
  if (Q_cat == nullptr || K == nullptr || scores == nullptr) return CCD_EINVAL;
  if (novelty == nullptr && shape->T > 0) return CCD_EINVAL;
  if (!aligned16(Q_cat) || !aligned16(K) || !aligned16(K_cap) || !aligned16(lse)) return CCD_EALIGN;
  const Dims D = make_dims(shape);
  ScorePlan pl = plan_score(D, K_cap != nullptr, lse != nullptr);
  if (path_refused(D, pl)) return CCD_EUNSUPPORTED;
  if (pl.use_mfma && D.head - D.head0 > mfma_max_slice()) return CCD_EUNSUPPORTED;   // (a matrix-core path was named)
  const Workspace w = layout_workspace(D);
  rc = check_workspace(w, workspace, workspace_bytes);
  if (rc != CCD_OK) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  pl.sync = D.units <= kMaxSharedUnits ? reinterpret_cast<uint32_t*>(ws + w.off_sync) : nullptr;
  const bool nuc_known = run_cap_scores(D, pl, w, Q_cat, K, K_cap, lse, novelty, ws, st);
  launch_finalize_select(D, reinterpret_cast<const float*>(ws + w.off_u), novelty, scores, nullptr, nuc_known ? pl.sync : nullptr, st);
  return launch_status();
}

int ccd_score(const ccd_shape_t* shape, const void* Q_cat, const void* K, const float* novelty, float* scores,
              void* workspace, size_t workspace_bytes, void* hip_stream) {
  return score_impl(shape, Q_cat, K, nullptr, nullptr, novelty, scores, workspace, workspace_bytes, hip_stream);
}

int ccd_score_kcat(const ccd_shape_t* shape, const void* Q_cat, const void* K, const void* K_cap, const float* novelty,
                   float* scores, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (K_cap == nullptr) return CCD_EINVAL;
  return score_impl(shape, Q_cat, K, K_cap, nullptr, novelty, scores, workspace, workspace_bytes, hip_stream);
}

int ccd_score_lse(const ccd_shape_t* shape, const void* Q_cat, const void* K, const float* lse, const float* novelty,
                  float* scores, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (lse == nullptr) return CCD_EINVAL;
  return score_impl(shape, Q_cat, K, nullptr, lse, novelty, scores, workspace, workspace_bytes, hip_stream);
}

int ccd_select(const ccd_shape_t* shape, const float* scores, int32_t* keep_idx, void* hip_stream) {
  int rc = check_shape(shape, 0);
  if (rc != CCD_OK) return rc;
  if (scores == nullptr || keep_idx == nullptr) return CCD_EINVAL;
  const Dims D = make_dims(shape);
  launch_finalize_select(D, nullptr, nullptr, const_cast<float*>(scores), keep_idx, nullptr,
                         static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

int ccd_compact(const ccd_shape_t* shape, const void* K_src, const void* V_src, const int32_t* keep_idx, void* K_dst,
                void* V_dst, float* novelty_inout, void* hip_stream) {
  int rc = check_shape(shape, kNeedKV | (novelty_inout ? kNeedNov : 0));
  if (rc != CCD_OK) return rc;
  if (K_src == nullptr || V_src == nullptr || K_dst == nullptr || V_dst == nullptr || keep_idx == nullptr)
    return CCD_EINVAL;
  if (!aligned16(K_src) || !aligned16(V_src) || !aligned16(K_dst) || !aligned16(V_dst)) return CCD_EALIGN;
  const Dims D = make_dims(shape);
  const bool per_head = shape->nov_stride_l != 0 || shape->nov_stride_h != 0;
  launch_compact(D, K_src, V_src, keep_idx, K_dst, V_dst, per_head ? novelty_inout : nullptr,
                 static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

int ccd_append(const ccd_shape_t* shape, void* K, void* V, float* novelty, const void* K_new, const void* V_new,
               const float* novelty_new, int32_t count, void* hip_stream) {
  if (shape == nullptr) return CCD_EINVAL;
  if (shape->B < 1 || shape->L < 1 || shape->Hkv < 1) return CCD_EINVAL;
  if ((int64_t)shape->B * shape->L * shape->Hkv > (int64_t)1 << 24) return CCD_EINVAL;
  if (shape->n_valid < 0 || shape->n_cap < 1 || count < 0 || (int64_t)shape->n_valid + count > shape->n_cap) return CCD_EINVAL;
  if (shape->dtype != CCD_FP32 && shape->dtype != CCD_BF16) return CCD_EUNSUPPORTED;
  if (shape->d != 64 && shape->d != 128) return CCD_EUNSUPPORTED;
  const int64_t esz = shape->dtype == CCD_FP32 ? 4 : 2;
  if (shape->kv_stride_h < (int64_t)shape->n_cap * shape->d || shape->kv_stride_l < 0 || shape->kv_stride_b < 0) return CCD_EINVAL;
  if ((shape->kv_stride_b * esz) % 16 || (shape->kv_stride_l * esz) % 16 || (shape->kv_stride_h * esz) % 16) return CCD_EALIGN;
  if (K == nullptr || V == nullptr) return CCD_EINVAL;
  if (count == 0) return CCD_OK;                      // an empty chunk (its pointers may be null): nothing to do
  if (K_new == nullptr || V_new == nullptr) return CCD_EINVAL;
  if ((novelty == nullptr) != (novelty_new == nullptr)) return CCD_EINVAL;
  if (!aligned16(K) || !aligned16(V) || !aligned16(K_new) || !aligned16(V_new)) return CCD_EALIGN;
  const bool per_head = shape->nov_stride_l != 0 || shape->nov_stride_h != 0;
  if (novelty != nullptr) {
    if (shape->nov_stride_b < 0 || shape->nov_stride_l < 0 || shape->nov_stride_h < 0) return CCD_EINVAL;
    if (per_head && shape->nov_stride_h < shape->n_cap) return CCD_EINVAL;
    if (!per_head && shape->B > 1 && shape->nov_stride_b < (int64_t)shape->n_valid + count) return CCD_EINVAL;
  }
  const Dims D = make_dims(shape);
  launch_append(D, count, K, V, K_new, V_new, novelty, novelty_new, per_head, static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

// ccd_compress, optionally with CR-RoPE of the kept keys on the side (K_rot != nullptr), other keys to attend to
// (K_score != nullptr) and the CaP tokens' own keys in the softmax (K_cap != nullptr)
static int compress_impl(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, float* novelty, float* scores_opt,
                         int32_t* keep_idx, const void* K_score, const void* K_cap, const float* lse,
                         const float* rope_cos, const float* rope_sin, void* K_rot, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
  int rc = check_shape(shape, kNeedFull);
  if (rc != CCD_OK) return rc;
  if (Q_cat == nullptr || K == nullptr || V == nullptr || keep_idx == nullptr) return CCD_EINVAL;
  if (novelty == nullptr && shape->T > 0) return CCD_EINVAL;
  if (!aligned16(Q_cat) || !aligned16(K) || !aligned16(V)) return CCD_EALIGN;
  if (K_rot != nullptr) {
    if (rope_cos == nullptr || rope_sin == nullptr || K_rot == K || K_rot == V) return CCD_EINVAL;
    if (!aligned16(K_rot) || !aligned16(rope_cos) || !aligned16(rope_sin)) return CCD_EALIGN;
  }
  if (K_score != nullptr && (K_score == V || !aligned16(K_score))) return K_score == V ? CCD_EINVAL : CCD_EALIGN;
  if (K_cap != nullptr && (K_cap == K || K_cap == V || K_cap == K_rot)) return CCD_EINVAL;
  if (!aligned16(K_cap)) return CCD_EALIGN;
  if (lse != nullptr && K_cap != nullptr) return CCD_EINVAL;     // the normalisers already account for the CaP keys
  if (!aligned16(lse)) return CCD_EALIGN;
  const void* K_attn = K_score != nullptr ? K_score : K;     // the keys the CaP queries attend to
  const Dims D = make_dims(shape);
  ScorePlan pl = plan_score(D, K_cap != nullptr, lse != nullptr);
  if (path_refused(D, pl)) return CCD_EUNSUPPORTED;
  if (pl.use_mfma && D.head - D.head0 > mfma_max_slice()) return CCD_EUNSUPPORTED;   // (a matrix-core path was named)
  const Workspace w = layout_workspace(D);
  rc = check_workspace(w, workspace, workspace_bytes);
  if (rc != CCD_OK) return rc;
  if (shape->n_valid < shape->n_cap || shape->n_valid <= shape->k) return CCD_NOOP;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  char* ws = static_cast<char*>(workspace);
  const float* u = reinterpret_cast<const float*>(ws + w.off_u);
  const bool per_head = shape->nov_stride_l != 0 || shape->nov_stride_h != 0;
  if (g_prof.on) ++g_prof.calls;
  uint32_t* sync = D.units <= kMaxSharedUnits ? reinterpret_cast<uint32_t*>(ws + w.off_sync) : nullptr;
  pl.sync = sync;
  // (units that are not shared would not take the slots: 8 units of 4096 tokens and 30 kept rows 33.5 us with a search for them, 32.6 without)
  const float* nov_slots = select_compact_shares_units(D, K_rot != nullptr) ? novelty : nullptr;
  const bool nuc_known = run_cap_scores(D, pl, w, Q_cat, K_attn, K_cap, lse, nov_slots, ws, st);
  if (select_compact_supported(D)) {
    g_prof.begin(kStSelCompact, st);
    launch_select_compact(D, u, novelty, per_head, scores_opt, keep_idx, K, V, rope_cos, rope_sin, K_rot, sync, nuc_known, st);
    g_prof.end(st);
    return launch_status();
  }
  g_prof.begin(kStSelect, st);
  launch_finalize_select(D, u, novelty, scores_opt, keep_idx, nullptr, st);
  g_prof.end(st);
  g_prof.begin(kStCompact, st);
  launch_compact(D, K, V, keep_idx, K, V, per_head ? novelty : nullptr, st);
  if (K_rot != nullptr) launch_rope_rows(D, K, rope_cos, rope_sin, D.k, K_rot, st);
  g_prof.end(st);
  return launch_status();
}

int ccd_compress(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, float* novelty, float* scores_opt,
                 int32_t* keep_idx, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return compress_impl(shape, Q_cat, K, V, novelty, scores_opt, keep_idx, nullptr, nullptr, nullptr, nullptr, nullptr,
                       nullptr, workspace, workspace_bytes, hip_stream);
}

// Device address of `scratch` on the current GPU, asked once per GPU (each GPU holds its own copy at its own address).
static int scratch_of_current_device(void** out) {
  constexpr int kMaxDevices = 64;
  static void* ptrs[kMaxDevices] = {};      // racing first calls on one GPU store the same value
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CCD_ELAUNCH;
  if (ptrs[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return CCD_ELAUNCH;
    ptrs[dev] = p;
  }
  *out = ptrs[dev];
  return CCD_OK;
}

int ccd_compress_noalloc(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, float* novelty, float* scores_opt,
                         int32_t* keep_idx, void* hip_stream) {
  int rc = check_shape(shape, kNeedFull);
  if (rc != CCD_OK) return rc;
  if (layout_workspace(make_dims(shape)).total > (size_t)CCD_NOALLOC_WORKSPACE_BYTES) return CCD_EWORKSPACE;
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc != CCD_OK) return rc;
  return compress_impl(shape, Q_cat, K, V, novelty, scores_opt, keep_idx, nullptr, nullptr, nullptr, nullptr, nullptr,
                       nullptr, ws, (size_t)CCD_NOALLOC_WORKSPACE_BYTES, hip_stream);
}

int ccd_compress_lse(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, const float* lse, float* novelty,
                     float* scores_opt, int32_t* keep_idx, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (lse == nullptr) return CCD_EINVAL;
  return compress_impl(shape, Q_cat, K, V, novelty, scores_opt, keep_idx, nullptr, nullptr, lse, nullptr, nullptr, nullptr,
                       workspace, workspace_bytes, hip_stream);
}

int ccd_compress_kcat(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, const void* K_cap, float* novelty,
                      float* scores_opt, int32_t* keep_idx, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (K_cap == nullptr) return CCD_EINVAL;
  return compress_impl(shape, Q_cat, K, V, novelty, scores_opt, keep_idx, nullptr, K_cap, nullptr, nullptr, nullptr,
                       nullptr, workspace, workspace_bytes, hip_stream);
}

int ccd_compress_rope(const ccd_shape_t* shape, const void* Q_cat, void* K, void* V, float* novelty, float* scores_opt,
                      int32_t* keep_idx, const void* K_score, const void* K_cap, const float* lse, const float* rope_cos,
                      const float* rope_sin, void* K_rot, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (K_rot == nullptr) return CCD_EINVAL;
  return compress_impl(shape, Q_cat, K, V, novelty, scores_opt, keep_idx, K_score, K_cap, lse, rope_cos, rope_sin, K_rot,
                       workspace, workspace_bytes, hip_stream);
}

int ccd_cr_rope(const ccd_shape_t* shape, const void* K, const float* rope_cos, const float* rope_sin, int32_t count,
                void* K_rot, void* hip_stream) {
  int rc = check_shape(shape, kNeedKV);
  if (rc != CCD_OK) return rc;
  if (K == nullptr || K_rot == nullptr || rope_cos == nullptr || rope_sin == nullptr || K_rot == K) return CCD_EINVAL;
  if (count < 0 || count > shape->n_cap) return CCD_EINVAL;
  if (!aligned16(K) || !aligned16(K_rot) || !aligned16(rope_cos) || !aligned16(rope_sin)) return CCD_EALIGN;
  if (count == 0) return CCD_OK;
  const Dims D = make_dims(shape);
  launch_rope_rows(D, K, rope_cos, rope_sin, count, K_rot, static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

int ccd_nuc_from_logits(const void* logits, const int32_t* labels, float* novelty, int64_t rows, int32_t V,
                        int64_t row_stride, int32_t dtype, void* hip_stream) {
  if (logits == nullptr || labels == nullptr || novelty == nullptr) return CCD_EINVAL;
  if (rows < 0 || rows > 0x7FFFFFFF || V < 1 || row_stride < V) return CCD_EINVAL;
  if (dtype != CCD_FP32 && dtype != CCD_BF16) return CCD_EUNSUPPORTED;
  if (!aligned16(logits) || (row_stride * (dtype == CCD_FP32 ? 4 : 2)) % 16) return CCD_EALIGN;
  if (rows == 0) return CCD_OK;
  launch_nuc_from_logits(logits, labels, novelty, rows, V, row_stride, dtype, static_cast<hipStream_t>(hip_stream));
  return launch_status();
}

int ccd_profile_enable(int on) {
  g_prof.on = on != 0;
  return CCD_OK;
}

int ccd_profile_stages(void) { return kNumStages; }

const char* ccd_profile_stage_name(int stage) {
  return (stage >= 0 && stage < kNumStages) ? kStageNames[stage] : "";
}

int ccd_profile_collect(double* stage_ms, int64_t* calls) {
  if (stage_ms == nullptr || calls == nullptr) return CCD_EINVAL;
  for (int i = 0; i < kNumStages; ++i) stage_ms[i] = 0.0;
  *calls = g_prof.calls;
  int rc = CCD_OK;
  for (size_t i = 0; i + 1 < g_prof.used && i / 2 < g_prof.stage_of.size(); i += 2) {
    if (hipEventSynchronize(g_prof.pool[i + 1]) != hipSuccess) { rc = CCD_ELAUNCH; break; }
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, g_prof.pool[i], g_prof.pool[i + 1]) == hipSuccess) stage_ms[g_prof.stage_of[i / 2]] += ms;
  }
  (void)hipGetLastError();    // a stage that launched nothing leaves two unused events and an error of the query
  g_prof.used = 0;
  g_prof.stage_of.clear();
  g_prof.calls = 0;
  return rc;
}

const char* ccd_strerror(int code) {
  switch (code) {
    case CCD_OK: return "ok";
    case CCD_NOOP: return "pot not full or nothing to drop: nothing done";
    case CCD_EINVAL: return "invalid argument (null pointer or shape field out of range)";
    case CCD_EUNSUPPORTED:
      return "unsupported: head dimension not 64 or 128, unknown dtype or pool mode, more than 65536 tokens, a matrix-core "
             "score path that an fp32 cache cannot take (token slices; units with a head dimension other than 64, a window "
             "or CaP keys), or a matrix-core score path named for a bf16 cache and a window with more than about 2000 CaP tokens";
    case CCD_EALIGN: return "pointer or stride not 16-byte aligned";
    case CCD_EWORKSPACE:
      return "workspace null, misaligned or too small (ccd_compress_noalloc: the shape needs more than the built-in "
             "CCD_NOALLOC_WORKSPACE_BYTES)";
    case CCD_ELAUNCH: return "HIP kernel launch failed";
    default: return "unknown code";
  }
}

}  // extern "C"
