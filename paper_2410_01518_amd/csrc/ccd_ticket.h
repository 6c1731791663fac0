// Tickets by which the workgroups that share a unit deal out its destination rows (select_compact_kernel).
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define CCD_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define CCD_HOST_DEVICE inline
#endif

namespace ccd {

// First row of the chunk that a ticket stands for, or k: there is no such chunk.  The ticket comes out of the caller's
// workspace, where a call that overlaps this one may have left any 32 bits.
CCD_HOST_DEVICE int chunk_first_row(uint32_t ticket, int chunks, int chunk_rows, int k) {
  return ticket < (uint32_t)chunks ? (int)ticket * chunk_rows : k;
}

}  // namespace ccd
