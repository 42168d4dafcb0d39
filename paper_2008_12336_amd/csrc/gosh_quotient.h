// Shared by the translation units of the rebuild of a level (gosh_quotient.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gosh_device_pool.h"

namespace gosh {

constexpr uint32_t kInside = 0xFFFFFFFFu;  // an entry inside its cluster: above every cluster id
constexpr int kGatherTile = 4096;          // entries per workgroup of the gather

// Largest row r in [lo, hi] with pos[r] <= e, i.e. the row that holds entry e (empty rows
// share their place with the next row and are skipped).
template <typename PosT>
__device__ inline int32_t row_of_entry(const PosT *pos, int32_t lo, int32_t hi, PosT e) {
  while (lo < hi) {
    const int32_t mid = lo + (hi - lo + 1) / 2;
    if (pos[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Merges the segments list[0 .. count) in place by sorting their entries as (segment, column) keys;
// length[a] becomes the length of a merged segment.  Queued on the null stream.  GOSH_ENOMEM, with
// nothing changed, if there is no room for the keys.  Its code lies in units of its own, one per
// width of the sums: a process loads it when a graph needs it (12 ms), not with its first coarsening.
template <typename WT, bool WEIGHTED>
int merge_by_radix(Pool &pool, const int64_t *segment, const int32_t *list, int64_t count, int64_t columns,
                   uint32_t *column, WT *weight, int64_t *length);

}  // namespace gosh
