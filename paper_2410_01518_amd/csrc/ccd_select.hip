// Per-unit selection kernels: NuC slots (Sec. 3.3.3 step 1), pooling + NuC lift, and the final top-k (Sec. 3.3.3 step 2 /
// App. B "Final Token Selection").  One workgroup of 1024 threads per unit; every thread looks after chunks of four
// consecutive tokens.  Prefix counts taken in token order give both the lowest-index
// tie-break and the output slot of every kept token, so keep_idx comes out ascending without a sort.  The machinery is in
// ccd_select_body.h and ccd_topk.h.
#include "ccd_select_body.h"

namespace ccd {

namespace {

constexpr int kSelThreads = 1024;

// GIVEN: the scores come from the caller (ccd_select), else from the raw scores u.  Known at compile time: asked at run time it put
// a row's windows into scratch memory and took 74 registers, one workgroup per compute unit, where 58 hold two (ccd_select, 1024
// units of 4096 tokens 22.0 -> 14.8 us, 256 units of 65536 tokens 114 -> 83 us).
// NUC: the units' words say which tokens have a NuC slot (as in ccd_compact.hip)
template <int CH, bool SELECT, bool GIVEN, bool NUC>
__global__ __launch_bounds__(kSelThreads) void finalize_select_kernel(Dims D, const float* __restrict__ u,
                                                                      const float* __restrict__ novelty, float* scores,
                                                                      int32_t* __restrict__ keep_idx, const uint32_t* nuc_words) {
  __shared__ SelectShared<kSelThreads, CH> sh;
  const int unit = D.unit0 + blockIdx.x;
  const float* nov = (!GIVEN && D.T > 0) ? novelty + nov_offset(D, decode_unit(D, unit)) : nullptr;
  Row<kSelThreads, CH> row(D, sh, unit, GIVEN ? nullptr : u, GIVEN ? scores : nullptr, nov);
  int32_t* out = SELECT ? keep_idx + (int64_t)unit * D.k : nullptr;
  const uint32_t* words = NUC ? nuc_words + (int64_t)novelty_unit(D, unit) * kSyncWords : nullptr;
  select_row<kSelThreads, CH, SELECT, NUC>(row, scores != nullptr ? scores + (int64_t)unit * D.n : nullptr, words,
                         [&](int pos, int t, int, int) {
                           // (a row that is pooled anew in every step may be overwritten meanwhile by a call that overlaps on
                           // the workspace: the list is undefined then, but stays in its place)
                           if (CH != kLongRow || pos < D.k) out[pos] = t;
                         });
}

}  // namespace

int select_max_tokens() { return kMaxTokens; }

void launch_finalize_select(const Dims& D, const float* u, const float* novelty, float* scores, int32_t* keep_idx,
                            const uint32_t* nuc_words, hipStream_t s) {
  const dim3 grid(D.units_run), block(kSelThreads);
  // (raw scores and a kept list: long rows only, others go through launch_select_compact)
#define CCD_LAUNCH(CH)                                                                                                     \
  if (u == nullptr) launch((finalize_select_kernel<CH, true, true, false>), grid, block, s, D, u, novelty, scores, keep_idx, nullptr);       \
  else              launch((finalize_select_kernel<CH, false, false, false>), grid, block, s, D, u, novelty, scores, keep_idx, nullptr)
  static_assert(kNoveltyMaxRow <= 8 * kSelThreads, "");
  if (nuc_words != nullptr) {          // (scores only)
    if (D.n <= 4 * kSelThreads) launch((finalize_select_kernel<1, false, false, true>), grid, block, s, D, u, novelty, scores, keep_idx, nuc_words);
    else                        launch((finalize_select_kernel<2, false, false, true>), grid, block, s, D, u, novelty, scores, keep_idx, nuc_words);
  } else if (D.n <= 4 * kSelThreads) { CCD_LAUNCH(1); }
  else if (D.n <= 8 * kSelThreads)  { CCD_LAUNCH(2); }
  else if (D.n <= kLdsRowTokens)    { CCD_LAUNCH(kLdsRow); }
  else if (u != nullptr && keep_idx != nullptr)
    launch((finalize_select_kernel<kLongRow, true, false, false>), grid, block, s, D, u, novelty, scores, keep_idx, nullptr);
  else                              { CCD_LAUNCH(kLongRow); }
#undef CCD_LAUNCH
}

}  // namespace ccd
