// Launches of the unit kernel (ccd_score_unit.h) with 4 row groups: sweeps of 768 or 1024 query rows.
#include "ccd_score_unit.h"

namespace ccd {

void launch_score_unit_4(const Dims& D, const ScorePlan& pl, bool narrow, const void* Q, const void* K, const void* K_cap,
                         const float2* part, float* u, float* lse_io, hipStream_t s) {
  if (narrow) launch_score_unit_as<3, 4>(D, pl, Q, K, K_cap, part, u, lse_io, s);
  else        launch_score_unit_as<4, 4>(D, pl, Q, K, K_cap, part, u, lse_io, s);
}

}  // namespace ccd
