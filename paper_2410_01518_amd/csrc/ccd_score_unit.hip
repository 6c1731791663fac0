// Launches of the unit kernel (ccd_score_unit.h): sweeps of 64 and 128 query rows, and which form of the kernel a call takes.
#include "ccd_score_unit.h"

namespace ccd {

// (fp32 caches: head dimension 64 only - the split rows of 128 would need twice the fragment registers - and neither
// CaP keys in the softmax nor a sliding window, whose side kernels exist for bf16 only: the caller checks those)
bool score_unit_supported(const Dims& D) { return D.dtype == 1 ? (D.d == 64 || D.d == 128) : D.d == 64; }

// The rows of a sweep: those for which the sweeps of a call hold the fewest rows, and among these the most, since every sweep reads K anew.
// 256 units of 4096 tokens, append + distill, against sweeps of 256 rows: 192 rows 377 -> 358 us, 384 rows 509 -> 433, 512 rows 516 -> 473,
// 768 rows 643 -> 587, 1024 rows 770 -> 694; 600 tokens and 1024 rows 172 -> 127; 640 units of 32768 tokens and 1024 rows 15.9 -> 14.1 ms.
void launch_score_unit(const Dims& D, const ScorePlan& pl, const void* Q, const void* K, const void* K_cap,
                       const float2* part, float* u, float* lse_io, hipStream_t s) {
  int rows = 0, all = 1 << 30;
  for (int r : {1024, 768, 512, 384, 256, 192, 128, 64}) {
    const int of_all_sweeps = (D.GP + r - 1) / r * r;
    if (of_all_sweeps < all && (r >= 256 || D.GP <= r)) { rows = r; all = of_all_sweeps; }
  }
  if (rows == 64)       launch_score_unit_as<1, 1>(D, pl, Q, K, K_cap, part, u, lse_io, s);
  else if (rows == 128) launch_score_unit_as<2, 1>(D, pl, Q, K, K_cap, part, u, lse_io, s);
  else if (rows <= 256) launch_score_unit_1(D, pl, rows == 192, Q, K, K_cap, part, u, lse_io, s);
  else if (rows <= 512) launch_score_unit_2(D, pl, rows == 384, Q, K, K_cap, part, u, lse_io, s);
  else                  launch_score_unit_4(D, pl, rows == 768, Q, K, K_cap, part, u, lse_io, s);
}

}  // namespace ccd
