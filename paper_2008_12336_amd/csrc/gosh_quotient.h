// Shared by the translation units of the rebuild of a level (gosh_quotient.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include <rocprim/rocprim.hpp>

#include "gosh_device_pool.h"

namespace gosh {

// The sorts of vertices, by degree and by cluster.  They are of few bits, so a radix pass per eight of them pays from
// fewer elements on than the 2^20 below which rocPRIM merges by default: whole coarsenings, merged / by radix from here
// on, ms: power law of 1 M 2.62 / 2.48, R-MAT of 600,000 1.36 / 1.26, uniform of 400,000 2.14 / 2.04, power law of 300,000
// 1.70 / 1.60, of 200,000 1.46 / 1.49; uniform of 65,000 by radix 1.24 / 1.39.
constexpr size_t kRadixFrom = 3 << 16;
using SortConfig = rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config, rocprim::default_config,
                                              kRadixFrom>;

constexpr uint32_t kInside = 0xFFFFFFFFu;  // an entry inside its cluster: above every cluster id

// An entry in cluster order is one word: its column above `shift` bits of weight, as many as the columns of a
// level leave.  A weight that does not fit them is held apart, at the entry's place, and the word says so with
// `top`, all of its weight bits set.  (shift = 0: a column alone.)
struct Packing {
  uint32_t shift, top;  // top = 2^shift - 1
  static Packing for_columns(int64_t columns) {
    uint32_t bits = 1;
    while (bits < 32 && columns > (int64_t{1} << bits) - 1) ++bits;  // no column has all of them set: kInside does
    if (const int64_t most = seam(kSeamWeightBits)) bits = std::max(bits, 32 - static_cast<uint32_t>(most));
    return Packing{32 - bits, static_cast<uint32_t>((uint64_t{1} << (32 - bits)) - 1)};
  }
  __device__ __forceinline__ uint32_t column(uint32_t word) const { return word == kInside ? kInside : word >> shift; }
  template <typename WT>
  __device__ __forceinline__ uint32_t entry(uint32_t column, WT w) const {
    return column << shift | static_cast<uint32_t>(w < top ? w : static_cast<WT>(top));
  }
  template <typename WT>
  __device__ __forceinline__ WT weight(uint32_t word, const WT *apart, int64_t at) const {
    const uint32_t w = word & top;
    return w < top ? static_cast<WT>(w) : apart[at];
  }
};

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

// Raises *word to the largest `mine` of the workgroup: one atomic, and only if that is above
// what is read there (the word only grows, so a stale value costs an atomic at most).
__device__ inline void raise_by_block(unsigned int *word, unsigned int mine, unsigned int *block_top) {
  if (mine) atomicMax(block_top, mine);
  __syncthreads();
  if (threadIdx.x == 0 && *block_top > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(word, *block_top);
}

// Merges the segments list[0 .. count) in place by sorting their entries as (segment, column) keys (not
// WEIGHTED: they are held as columns alone);
// length[a] becomes the length of a merged segment.  Queued on the null stream.  GOSH_ENOMEM, with
// nothing changed, if there is no room for the keys.  Its code lies in units of its own, one per
// width of the sums: a process loads it when a graph needs it (12 ms), not with its first coarsening.
template <typename WT, bool WEIGHTED>
int merge_by_radix(Pool &pool, const int64_t *segment, const int32_t *list, int64_t count, int64_t columns,
                   Packing pack, uint32_t *entry, WT *weight, int64_t *length);

}  // namespace gosh
