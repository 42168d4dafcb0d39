// The radix way of merging long coarse rows (see gosh_quotient.hip).  Included by the two units that
// instantiate it and by nothing else.
#pragma once

#include <algorithm>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "gosh_common.h"
#include "gosh_quotient.h"

namespace gosh {
namespace {

// size[i] = entries of the i-th segment, size[count] = 0.
__global__ __launch_bounds__(256) void radix_sizes_kernel(const int64_t *__restrict__ segment,
                                                          const int32_t *__restrict__ list, int64_t count,
                                                          int64_t *__restrict__ size) {
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i <= count; i += gridDim.x * 256LL)
    size[i] = i < count ? segment[list[i] + 1LL] - segment[list[i]] : 0;
}

// key = (place in the list, column); an entry inside its cluster gets the largest column of its row.
template <typename WT, bool WEIGHTED>
__global__ __launch_bounds__(256) void radix_keys_kernel(const int64_t *__restrict__ segment,
                                                         const int32_t *__restrict__ list, int64_t count,
                                                         const int64_t *__restrict__ from, int64_t entries,
                                                         unsigned column_bits, Packing pack,
                                                         const uint32_t *__restrict__ entry,
                                                         const WT *__restrict__ weight, uint64_t *__restrict__ key,
                                                         WT *__restrict__ value) {
  __shared__ int32_t first_row;
  const uint64_t inside = (uint64_t{1} << column_bits) - 1;
  for (int64_t tile = blockIdx.x * static_cast<int64_t>(kGatherTile); tile < entries;
       tile += gridDim.x * static_cast<int64_t>(kGatherTile)) {
    __syncthreads();  // the previous tile's row has been read
    if (threadIdx.x == 0) first_row = row_of_entry<int64_t>(from, 0, static_cast<int32_t>(count - 1), tile);
    __syncthreads();
    int32_t r = first_row;
    for (int64_t e = tile + threadIdx.x; e < std::min(tile + kGatherTile, entries); e += 256) {
      while (r + 1 < count && from[r + 1] <= e) ++r;  // a tile spans a few rows: all are long
      const int64_t at = segment[list[r]] + (e - from[r]);
      const uint32_t word = entry[at], c = WEIGHTED ? pack.column(word) : word;
      key[e] = (static_cast<uint64_t>(r) << column_bits) | (c == kInside ? inside : c);
      if constexpr (WEIGHTED) value[e] = c == kInside ? WT(0) : pack.weight(word, weight, at);
    }
  }
}

__device__ inline int64_t first_not_below(const uint64_t *keys, int64_t count, uint64_t key) {
  int64_t lo = 0, hi = count;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (keys[mid] < key) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// first[i] = place of the first merged entry of the i-th segment; the lengths without what lies
// inside the clusters.
__global__ __launch_bounds__(256) void radix_lengths_kernel(const int32_t *__restrict__ list, int64_t count,
                                                            unsigned column_bits, const uint64_t *__restrict__ merged,
                                                            const unsigned long long *__restrict__ merged_count,
                                                            int64_t *__restrict__ first, int64_t *__restrict__ length) {
  const int64_t n = static_cast<int64_t>(*merged_count);
  const uint64_t inside = (uint64_t{1} << column_bits) - 1;
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < count; i += gridDim.x * 256LL) {
    const uint64_t row = static_cast<uint64_t>(i) << column_bits;
    first[i] = first_not_below(merged, n, row);
    length[list[i]] = first_not_below(merged, n, row | inside) - first[i];
  }
}

// The merged entries go to the front of their segments, as the sorting networks leave them.
template <typename WT>
__global__ __launch_bounds__(256) void radix_place_kernel(const int64_t *__restrict__ segment,
                                                          const int32_t *__restrict__ list, unsigned column_bits,
                                                          const uint64_t *__restrict__ merged,
                                                          const WT *__restrict__ sums,
                                                          const unsigned long long *__restrict__ merged_count,
                                                          const int64_t *__restrict__ first, Packing pack,
                                                          uint32_t *__restrict__ entry, WT *__restrict__ weight) {
  const int64_t n = static_cast<int64_t>(*merged_count);
  const uint64_t inside = (uint64_t{1} << column_bits) - 1;
  for (int64_t u = blockIdx.x * 256LL + threadIdx.x; u < n; u += gridDim.x * 256LL) {
    const uint64_t key = merged[u], c = key & inside;
    if (c == inside) continue;
    const int64_t i = static_cast<int64_t>(key >> column_bits), at = segment[list[i]] + (u - first[i]);
    entry[at] = pack.entry(static_cast<uint32_t>(c), sums[u]);
    if (sums[u] >= pack.top) weight[at] = sums[u];
  }
}

}  // namespace

template <typename WT, bool WEIGHTED>
int merge_by_radix(Pool &pool, const int64_t *segment, const int32_t *list, int64_t count, int64_t columns,
                   Packing pack, uint32_t *entry, WT *weight, int64_t *length) {
  Buffers buf(pool);
  int64_t *size = nullptr, *from = nullptr;
  uint64_t *keys = nullptr, *sorted = nullptr;
  WT *values = nullptr, *sorted_values = nullptr;
  unsigned long long *merged_count = nullptr;
  if (gosh::denied(gosh::kDenyRadix)) return GOSH_ENOMEM;
  unsigned column_bits = 1, row_bits = 1;
  while (((int64_t{1} << column_bits) - 1) < columns) ++column_bits;
  while ((count >> row_bits) != 0) ++row_bits;
  if (int rc = buf.alloc(&size, static_cast<size_t>(count) + 1, "long coarse rows")) return rc;
  if (int rc = buf.alloc(&from, static_cast<size_t>(count) + 1, "long coarse rows")) return rc;
  if (int rc = buf.alloc(&merged_count, 1, "merged count")) return rc;
  const int row_blocks = blocks_for(count + 1, 256);
  hipLaunchKernelGGL(radix_sizes_kernel, dim3(row_blocks), dim3(256), 0, nullptr, segment, list, count, size);
  size_t scan_bytes = 0, sort_bytes = 0, reduce_bytes = 0;
  char *temp = nullptr;
  GOSH_TRY_HIP(rocprim::exclusive_scan(nullptr, scan_bytes, size, from, int64_t(0), static_cast<size_t>(count) + 1,
                                       rocprim::plus<int64_t>(), nullptr),
               "long row scan (size query)");
  if (int rc = buf.alloc(&temp, scan_bytes, "scan workspace")) return rc;
  GOSH_TRY_HIP(rocprim::exclusive_scan(temp, scan_bytes, size, from, int64_t(0), static_cast<size_t>(count) + 1,
                                       rocprim::plus<int64_t>(), nullptr),
               "long row scan");
  int64_t entries = 0;
  GOSH_TRY_HIP(hipMemcpy(&entries, from + count, 8, hipMemcpyDeviceToHost), "read long row entries");
  buf.release(temp);
  const size_t total = static_cast<size_t>(entries);
  if (int rc = buf.alloc(&keys, total, "keys of long rows")) return rc;
  if (int rc = buf.alloc(&sorted, total, "sorted keys of long rows")) return rc;
  if (int rc = buf.alloc(&values, total, "multiplicities of long rows")) return rc;
  if constexpr (WEIGHTED)
    if (int rc = buf.alloc(&sorted_values, total, "sorted multiplicities of long rows")) return rc;
  auto sort = [&]() -> hipError_t {
    if constexpr (WEIGHTED)
      return rocprim::radix_sort_pairs(temp, sort_bytes, keys, sorted, values, sorted_values, total, 0u,
                                       column_bits + row_bits, nullptr);
    else
      return rocprim::radix_sort_keys(temp, sort_bytes, keys, sorted, total, 0u, column_bits + row_bits, nullptr);
  };
  auto reduce = [&]() -> hipError_t {  // where the unsorted ones were
    if constexpr (WEIGHTED)
      return rocprim::reduce_by_key(temp, reduce_bytes, sorted, sorted_values, total, keys, values, merged_count,
                                    rocprim::plus<WT>(), rocprim::equal_to<uint64_t>(), nullptr);
    else
      return rocprim::reduce_by_key(temp, reduce_bytes, sorted, rocprim::constant_iterator<WT>(1), total, keys, values,
                                    merged_count, rocprim::plus<WT>(), rocprim::equal_to<uint64_t>(), nullptr);
  };
  temp = nullptr;  // asks for the sizes
  GOSH_TRY_HIP(sort(), "long row sort (size query)");
  GOSH_TRY_HIP(reduce(), "long row merge (size query)");
  if (int rc = buf.alloc(&temp, std::max(sort_bytes, reduce_bytes), "sort workspace")) return rc;
  hipLaunchKernelGGL((radix_keys_kernel<WT, WEIGHTED>), dim3(blocks_for(entries, kGatherTile)), dim3(256), 0, nullptr,
                     segment, list, count, from, entries, column_bits, pack, entry, weight, keys, values);
  if (int rc = gosh::check_launch("radix_keys_kernel")) return rc;
  GOSH_TRY_HIP(sort(), "long row sort");
  GOSH_TRY_HIP(reduce(), "long row merge");
  hipLaunchKernelGGL(radix_lengths_kernel, dim3(row_blocks), dim3(256), 0, nullptr, list, count, column_bits, keys,
                     merged_count, size, length);
  hipLaunchKernelGGL(radix_place_kernel<WT>, dim3(blocks_for(entries, 1024)), dim3(256), 0, nullptr, segment, list,
                     column_bits, keys, values, merged_count, size, pack, entry, weight);
  return gosh::check_launch("radix_place_kernel");
}

}  // namespace gosh
