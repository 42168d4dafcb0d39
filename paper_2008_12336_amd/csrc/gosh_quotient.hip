// "Coarsen(G_i, map_i)" on the device: the quotient graph of a level under its map.
//
// Every coarse row is the union of the fine rows of its members, so the entries of a coarse
// row are brought together by moving whole fine rows, not by sorting entries: the vertices are
// sorted by cluster, a scan of their degrees in that order gives every fine row its place, and
// one pass over the entries writes the cluster of each neighbour there.  What is left is to
// sort each coarse row ("segment") by itself and to merge equal entries.  Three ways, by the
// length S of the segment:
//   S <= 1,024          one wavefront or, up to 32, a part of one, bitonic in registers
//   S <= bitmap_from()  one workgroup, the same
//   longer              no comparisons: a bitmap in LDS with a bit per possible neighbour, 2^18
//                       ("piece") at a time, whose set bits are the merged row in order
// The first two merge in place and are copied out once the length of every coarse row is
// known.  The bitmap is made to count a row and made again to write it where it belongs; the
// number of bits below an entry is the place of its sum.  Rows longer than dense_from(), whose
// sums would fill the LDS many times over, are counted instead: a word of a table per possible
// neighbour, added up by workgroups that each take a slice of the row and 2^14 columns ("strip").
// Both grow with the number of columns; where there are many, the entries of the long rows are
// radix-sorted as (row, column) keys, equal ones added up, and the rest is as after a merge in place.
//
// An entry is one word, its weight beside its column (Packing), from the gather to the copy.
//
// Sorted distinct entries with summed multiplicities are unique, so the arrays are those of
// the sequential algorithm.  128 M entries of a 4 M-vertex R-MAT graph and the 117 M weighted ones of its
// second level take 5.0 ms together (7.5 with weights in arrays of their own, pairs sorted by compare and select, and
// a wavefront per segment to copy; 19.4 as a radix sort of 64-bit (row, column) keys of all entries).
// 8 (wide sums: 12) bytes of scratch per entry, 16 more per entry of a row that is counted and 24 (wide sums: 32)
// of one that is sorted by radix.  A third of it is the gather.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include <rocprim/rocprim.hpp>

#include "gosh_coarsen_internal.h"
#include "gosh_common.h"
#include "gosh_device_pool.h"
#include "gosh_quotient.h"

namespace {

using gosh::blocks_for;
using gosh::persistent;

using gosh::kGatherTile;
using gosh::kInside;
using gosh::Packing;
using gosh::raise_by_block;
using gosh::row_of_entry;

constexpr int kGatherRows = 1024;          // rows of a tile that are looked up in LDS,
constexpr int kTileRows = 4096;            // among at most so many
constexpr int64_t kNarrowFrom = 1 << 19;   // vertices whose map no L2 holds beside the streams
// Longest segments that are sorted in the registers of a quarter, a half or a whole wavefront, one per lane, of a
// wavefront, 2, 4, 8 or 16 per lane, and in those of a workgroup, 8 or 16 per lane.
constexpr int kSortClasses = 9;
constexpr int kSortMax[kSortClasses] = {16, 32, 64, 128, 256, 512, 1024, 2048, 4096};
enum : int { kBitmap = kSortClasses, kDense, kRadix, kWays };
constexpr int kPieceBits = 18, kPieceWords = 1 << (kPieceBits - 5);
constexpr int kStripBits = 14, kStripsPerPiece = 1 << (kPieceBits - kStripBits);
constexpr int64_t kSlice = 1 << 16;  // entries of a counted segment that one workgroup takes
// Columns up to which long segments are worth ranking (each reads its entries once per piece and
// pays for a bitmap per piece, twice) and counting (once per strip).  Beyond, all are sorted, which does
// not grow with the columns.  Rebuilds, ms, with ranks / counters, by sort, with all entries sorted as
// keys (the radix sort this file replaced), all of them before entries were one word:
//   2.0 M columns, 288 M entries 19.0, 16.7, 21.7     2.4 M, 535 M 27.9, 29.9, 38.8
//   3.4 M, 308 M 27.8, 22.3, 22.7                     21.8 M, 536 M 67.7, 35.0, 42.7
//   8.4 M, 3.6 G 336, 202, 264
// twenty segments of millions of entries (counted): 0.8 M columns 6.3, 6.6, 6.6; 6.7 M 57, 18, 18
constexpr int64_t kRankColumns = int64_t{10} << kPieceBits, kCountColumns = int64_t{4} << kPieceBits;
constexpr int kSumBytes = 30 << 10;  // LDS for the columns and sums of a piece, as many at a time as fit

// Number of segments per way of merging, 1 + the largest column met, slices of the counted ones; of the
// coarse graph: its longest row and its entries.
struct Classes {
  unsigned int count[kWays], columns, slices, longest;
  int64_t entries;
};

__host__ __device__ inline int64_t pieces_of(int64_t columns) {
  return std::max<int64_t>((columns + (int64_t{1} << kPieceBits) - 1) >> kPieceBits, 1);
}

// Longest segment that is sorted: the bitmap costs a fixed time per 2^14 columns, as much as
// sorting about 300 entries, and longer ones have no network.  (7,300 segments of 2,049 to 4,096 entries among
// 280,000 or 500,000 columns: about 0.4 ms as bitmaps, written included, 0.15 to 0.19 sorted.)
__host__ __device__ inline int64_t bitmap_from(int64_t columns) {
  return std::min<int64_t>(kSortMax[kSortClasses - 1], std::max<int64_t>(512, ((columns >> kStripBits) + 1) * 300));
}

// Longest segment whose sums are placed by rank.  Every kSumBytes of sums read the segment again,
// in one workgroup; the counters of a longer one take at most 16 bytes per entry.
__host__ __device__ inline int64_t dense_from(int64_t columns, int sum_bytes) {
  const int64_t strips = (columns + (1 << kStripBits) - 1) >> kStripBits;
  return std::max<int64_t>(1 << 15, (strips << kStripBits) * sum_bytes / 16);
}

// How the long segments of a graph are merged: the bounds above, as far as they are not forced.
struct Ways {
  int64_t rank_columns, count_columns;
  int sum_bytes;
};
__host__ __device__ inline int way_of_long(int64_t size, int64_t columns, const Ways &w) {
  if (size <= dense_from(columns, w.sum_bytes)) return columns > w.rank_columns ? kRadix : kBitmap;
  return columns > w.count_columns ? kRadix : kDense;
}
// Segments longer than this are sorted by radix.
inline int64_t radix_above(int64_t columns, const Ways &w) {
  if (columns > w.rank_columns) return bitmap_from(columns);
  return columns > w.count_columns ? dense_from(columns, w.sum_bytes) : INT64_MAX;
}

// A slice of a counted segment: its place in the list, and which of its slices.
struct Slice {
  int32_t row, part;
};

// len[t] = degree of the t-th vertex in cluster order, len[n] = 0; begin[t] = its first entry.
template <typename OffT>
__global__ __launch_bounds__(256) void row_lengths_kernel(const OffT *__restrict__ xadj,
                                                          const int32_t *__restrict__ order, int64_t n,
                                                          int64_t *__restrict__ len, OffT *__restrict__ begin) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t <= n; t += gridDim.x * 256LL) {
    const int64_t v = t < n ? order[t] : 0;
    const OffT first = xadj[v];
    len[t] = t < n ? static_cast<int64_t>(xadj[v + 1] - first) : 0;
    if (t < n) begin[t] = first;
  }
}

// segment[a] = place of the first entry of cluster a (segment[n_coarse] = nnz); tile_row[k] =
// row that holds entry k * kGatherTile, and behind the last tile's the last row with entries (vertices without
// are clusters of their own, the last ones).  pos is the scan of the row lengths.
__global__ __launch_bounds__(256) void segments_kernel(const int32_t *__restrict__ cluster,
                                                       const int64_t *__restrict__ pos, int64_t n, int64_t nnz,
                                                       int64_t n_coarse, int64_t *__restrict__ segment,
                                                       int32_t *__restrict__ tile_row) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL) {
    const int64_t a = cluster[t], lo = pos[t], hi = pos[t + 1];
    // every cluster has a member, so each of these loops writes one entry or none
    for (int64_t c = t == 0 ? 0 : cluster[t - 1] + 1LL; c <= a; ++c) segment[c] = lo;
    if (t == n - 1)
      for (int64_t c = a + 1; c <= n_coarse; ++c) segment[c] = nnz;
    for (int64_t k = (lo + kGatherTile - 1) / kGatherTile; k * kGatherTile < hi; ++k)
      tile_row[k] = static_cast<int32_t>(t);
    if (lo < hi && hi == nnz) tile_row[(nnz + kGatherTile - 1) / kGatherTile] = static_cast<int32_t>(t);
  }
}

// What the gather looks clusters up in: `stride` bytes per vertex, of which `mask` keeps the cluster.
struct ClusterTable {
  const char *base;
  uint32_t stride, mask;
  __device__ __forceinline__ uint32_t of(int32_t v) const {
    uint32_t word;  // need not lie at a multiple of its size
    __builtin_memcpy(&word, base + static_cast<uint64_t>(static_cast<uint32_t>(v)) * stride, 4);
    return word & mask;
  }
};

// The map in three bytes per vertex, four vertices a thread.
__global__ __launch_bounds__(256) void narrow_map_kernel(const int32_t *__restrict__ map, int64_t n,
                                                         uint32_t *__restrict__ narrow) {
  const int64_t quads = (n + 3) / 4;
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < quads; i += gridDim.x * 256LL) {
    uint32_t m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) m[q] = static_cast<uint32_t>(map[std::min<int64_t>(i * 4 + q, n - 1)]);
    narrow[i * 3] = m[0] | m[1] << 24;
    narrow[i * 3 + 1] = m[1] >> 8 | m[2] << 16;
    narrow[i * 3 + 2] = m[2] >> 16 | m[3] << 8;
  }
}

// Which row the entries of a tile lie in: a bit per entry at which a row starts (the tile's first entry counts).
// 64 consecutive entries, a wavefront's, share one word, and the bits up to a lane count its row.
constexpr int kTileWords = kGatherTile / 64;
struct RowStarts {
  unsigned long long after[kTileWords];  // the word without its first bit, shifted down by it
  int32_t before[kTileWords];            // number of the row at a word's first entry
  int32_t met;                           // rows of the tile
  // Number of the row at entry 64 * word + lane.
  __device__ __forceinline__ int32_t row(int word) const {
    const unsigned long long w = after[word];
    return before[word] + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                              static_cast<uint32_t>(w >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(w), 0)));
  }
};

// Fills the table for the entries [e0, e1) of the rows row0 .. row1, which start at pos, and calls
// fill(number, row, pos[row]) for each of them.  Rows without entries share their place with the next row and
// are no rows of the tile.  False if there are too many for tables of kGatherRows, or so many without entries
// that one search per entry costs less: fill has not been called.  The whole workgroup of 256 threads.
template <class Fill>
__device__ __forceinline__ bool lay_out_rows(RowStarts &t, const int64_t *__restrict__ pos, int32_t row0, int32_t row1,
                                             int64_t e0, int64_t e1, Fill fill) {
  static_assert(kTileWords == 64, "the first wavefront scans a word per lane");
  const int lane = threadIdx.x & 63;
  __syncthreads();  // the tables of the previous tile have been used
  if (row1 - row0 >= kTileRows) return false;
  if (threadIdx.x < kTileWords) t.after[threadIdx.x] = 0;
  __syncthreads();
  auto for_rows = [&](auto body) {
    for (int32_t r = row0 + static_cast<int32_t>(threadIdx.x); r <= row1; r += 256) {
      const int64_t p = pos[r];
      if (p < e1 && pos[r + 1] > p) body(r, p, static_cast<uint32_t>(std::max<int64_t>(p - e0, 0)));
    }
  };
  for_rows([&](int32_t, int64_t, uint32_t place) { atomicOr(&t.after[place >> 6], 1ull << (place & 63)); });
  __syncthreads();
  if (threadIdx.x < 64) {
    const unsigned long long mine = t.after[lane];
    int32_t upto = __popcll(mine);
    for (int step = 1; step < 64; step <<= 1) {
      const int32_t x = __shfl_up(upto, step, 64);
      if (lane >= step) upto += x;
    }
    t.after[lane] = mine >> 1;
    t.before[lane] = upto - __popcll(mine >> 1) - 1;
    if (lane == 63) t.met = upto;
  }
  __syncthreads();
  if (t.met > kGatherRows) return false;
  for_rows([&](int32_t r, int64_t p, uint32_t place) {
    fill(t.before[place >> 6] + __popcll(t.after[place >> 6] & ((1ull << (place & 63)) - 1)), r, p);
  });
  __syncthreads();
  return true;
}

// Entry e in cluster order: the cluster of its neighbour (kInside if that is its own) and its
// multiplicity.  A workgroup takes kGatherTile consecutive entries, so hub rows are no long
// tail and the writes are coalesced.  Bound by the lookups: where the table is larger than an L2, most read a
// line from the memory side (7 TB/s of lines).  Hence the narrow table, and streams that pass the L2 by: 128 M
// entries of 4.2 M vertices 1.35 ms without both, now 1.21 (1.43 with a binary search per entry besides).  Eight
// entries of a thread are requested together, as many as leave eight wavefronts to a SIMD: 117 M weighted
// entries of 2.3 M vertices 0.66 ms by fours, now 0.53.
template <typename OffT, typename WT, bool WEIGHTED>
__global__ __launch_bounds__(256) void gather_kernel(const int32_t *__restrict__ adj,
                                                     const WT *__restrict__ mult,
                                                     ClusterTable clusters,
                                                     const OffT *__restrict__ begin,
                                                     const int32_t *__restrict__ cluster,
                                                     const int64_t *__restrict__ pos,
                                                     const int32_t *__restrict__ tile_row, int64_t nnz, Packing pack,
                                                     uint32_t *__restrict__ entry,
                                                     WT *__restrict__ weight, Classes *__restrict__ classes) {
  constexpr int kUnits = 8;
  __shared__ unsigned int block_top;
  if (threadIdx.x == 0) block_top = 0;
  unsigned int top = 0;
  __shared__ RowStarts rows;
  __shared__ int64_t from[kGatherRows];  // fine entry of place 0 of the row, were it that long
  __shared__ int32_t owner[kGatherRows];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t tiles = (nnz + kGatherTile - 1) / kGatherTile;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t e0 = tile * kGatherTile, e1 = std::min(e0 + kGatherTile, nnz);
    const int32_t row0 = tile_row[tile], row1 = tile_row[tile + 1];
    const bool in_lds = lay_out_rows(rows, pos, row0, row1, e0, e1, [&](int32_t k, int32_t r, int64_t p) {
      from[k] = static_cast<int64_t>(begin[r]) - p;
      owner[k] = cluster[r];
    });
    for (int step = 0; step < kGatherTile / 256; step += kUnits) {
      const int64_t first = e0 + step * 256 + threadIdx.x;
      if (first >= e1) break;
      int64_t at[kUnits];
      int32_t own[kUnits], y[kUnits];
      WT w[WEIGHTED ? kUnits : 1];
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        const int64_t e = std::min(first + q * 256, e1 - 1);
        if (in_lds) {
          const int32_t r = rows.row((step + q) * 4 + wave);
          at[q] = from[r] + e;
          own[q] = owner[r];
        } else {
          const int32_t r = row_of_entry<int64_t>(pos, row0, row1, e);
          at[q] = static_cast<int64_t>(begin[r]) - pos[r] + e;
          own[q] = cluster[r];
        }
      }
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        y[q] = __builtin_nontemporal_load(adj + at[q]);
        if constexpr (WEIGHTED) w[q] = __builtin_nontemporal_load(mult + at[q]);
      }
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        const int64_t e = first + q * 256;
        const uint32_t b = clusters.of(y[q]);
        if (e < e1) {
          top = max(top, b + 1);
          uint32_t word = b;
          if constexpr (WEIGHTED) {
            word = pack.entry(b, w[q]);
            if (w[q] >= pack.top) weight[e] = w[q];
          }
          __builtin_nontemporal_store(b == static_cast<uint32_t>(own[q]) ? kInside : word, entry + e);
        }
      }
    }
  }
  raise_by_block(&classes->columns, top, &block_top);
}

// Sorts the segments into kWays lists (list + 0, + n_coarse, ...) and clears the
// lengths that are not set by assignment.  One atomic per workgroup and list.
__global__ __launch_bounds__(1024) void classify_segments_kernel(const int64_t *__restrict__ segment, int64_t n_coarse,
                                                                 int32_t *__restrict__ list,
                                                                 int64_t *__restrict__ length,
                                                                 Slice *__restrict__ slices, Ways ways,
                                                                 Classes *__restrict__ classes) {
  __shared__ unsigned int count[kWays], base[kWays];
  const int64_t columns = classes->columns, longest_sorted = bitmap_from(columns);
  for (int64_t first = blockIdx.x * 1024LL; first < n_coarse; first += gridDim.x * 1024LL) {
    if (threadIdx.x < kWays) count[threadIdx.x] = 0;
    __syncthreads();
    const int64_t a = first + threadIdx.x;
    int cls = -1;
    unsigned int mine = 0;
    if (a < n_coarse) {
      const int64_t s = segment[a + 1] - segment[a];
      if (s > longest_sorted) cls = way_of_long(s, columns, ways);
      else if (s > 0)
        for (cls = 0; s > kSortMax[cls];) ++cls;
      if (cls < 0 || cls >= kBitmap) length[a] = 0;  // (the radix sort assigns, its stand-in adds)
    }
    if (cls >= 0) mine = atomicAdd(&count[cls], 1u);
    __syncthreads();
    if (threadIdx.x < kWays && count[threadIdx.x]) 
      base[threadIdx.x] = atomicAdd(&classes->count[threadIdx.x], count[threadIdx.x]);
    __syncthreads();
    if (cls >= 0) list[cls * n_coarse + base[cls] + mine] = static_cast<int32_t>(a);
    if (cls == kDense) {
      const int32_t parts = static_cast<int32_t>((segment[a + 1] - segment[a] + kSlice - 1) / kSlice);
      const unsigned int at = atomicAdd(&classes->slices, static_cast<unsigned int>(parts));
      for (int32_t q = 0; q < parts; ++q) slices[at + q] = Slice{static_cast<int32_t>(base[cls] + mine), q};
    }
    __syncthreads();
  }
}

// The value of lane ^ MASK.
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  const int v = static_cast<int>(x);
  if constexpr (MASK == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);       // quad_perm [1,0,3,2]
  else if constexpr (MASK == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
  else if constexpr (MASK == 4) return __builtin_amdgcn_ds_swizzle(v, 0x101F);
  else if constexpr (MASK == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);  // row_ror 8
  else if constexpr (MASK == 16) return __builtin_amdgcn_ds_swizzle(v, 0x401F);
  else return __shfl_xor(v, 32, 64);
}

// Median of three: the smaller of a and b beside 0, the larger beside ~0.
__device__ __forceinline__ uint32_t med3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));  // one instruction, which the compiler may place (as asm 10 to 20 % slower)
}

// ~0 where the bit is set in `index`, else 0.
template <int BIT>
__device__ __forceinline__ uint32_t spread(uint32_t index) {
  static_assert(BIT > 0 && (BIT & (BIT - 1)) == 0, "one bit");
  return static_cast<uint32_t>(static_cast<int32_t>(index << __builtin_clz(BIT)) >> 31);
}

// One stage (distance J, in blocks of K of TOP) of a bitonic network over the elements index * R + r,
// r < R, of consecutive lanes; distances below 64 R.  Which of two elements stays is the third operand of a
// median, so a stage costs an instruction per element, and one more to fetch the other from another lane.
template <int K, int J, int TOP, int R>
__device__ __forceinline__ void key_stage(uint32_t (&key)[R], uint32_t index) {
  if constexpr (J >= R) {
    uint32_t larger = spread<J / R>(index);
    if constexpr (K < TOP) larger ^= spread<K / R>(index);
    uint32_t other[R];
#pragma unroll
    for (int r = 0; r < R; ++r) other[r] = lane_xor<J / R>(key[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) key[r] = med3(key[r], other[r], larger);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if ((r & J) == 0) {
        const uint32_t x = key[r], y = key[r | J];
        if constexpr (K >= TOP || K < R) {
          const bool up = K >= TOP || (r & K) == 0;
          key[r] = up ? min(x, y) : max(x, y);
          key[r | J] = up ? max(x, y) : min(x, y);
        } else {
          const uint32_t larger = spread<K / R>(index);
          key[r] = med3(x, y, larger);
          key[r | J] = med3(x, y, ~larger);
        }
      }
  }
}
template <int K, int J, int TOP, int R>
__device__ __forceinline__ void key_merge(uint32_t (&key)[R], uint32_t index) {
  key_stage<K, J, TOP>(key, index);
  if constexpr (J > 1) key_merge<K, J / 2, TOP>(key, index);
}
template <int K, int LAST, int TOP, int R>
__device__ __forceinline__ void key_blocks(uint32_t (&key)[R], uint32_t index) {
  key_merge<K, K / 2, TOP>(key, index);
  if constexpr (K < LAST) key_blocks<K * 2, LAST, TOP>(key, index);
}

// Inclusive sum over the lanes below and this one.
__device__ __forceinline__ uint32_t sum_upto_lane(uint32_t x, int) {
  auto step = [&](auto move) { x += static_cast<uint32_t>(move(static_cast<int>(x))); };
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false); });  // row_shr 1
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false); });
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false); });
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false); });
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false); });  // row_bcast 15
  step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false); });  // row_bcast 31
  return x;
}
__device__ __forceinline__ unsigned long long sum_upto_lane(unsigned long long x, int lane) {
#pragma unroll
  for (int step = 1; step < 64; step <<= 1) {
    const unsigned long long y = __shfl_up(x, step, 64);
    if (lane >= step) x += y;
  }
  return x;
}
__device__ __forceinline__ int32_t lanes_below(unsigned long long mask) {
  return static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0)));
}

// Inclusive sum over the lanes of the group of LANES below and this one.
template <int LANES, typename WT>
__device__ __forceinline__ WT sum_upto_in_group(WT x, int gl) {
  if constexpr (LANES == 64) {
    return sum_upto_lane(x, gl);
  } else if constexpr (sizeof(WT) == 4) {
    auto step = [&](auto move) { x += static_cast<uint32_t>(move(static_cast<int>(x))); };
    step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false); });  // row_shr 1
    step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false); });
    step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false); });
    step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false); });
    if constexpr (LANES == 32) step([](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false); });
    return x;
  } else {
#pragma unroll
    for (int step = 1; step < LANES; step <<= 1) {
      const WT y = __shfl_up(x, step, LANES);
      if (gl >= step) x += y;
    }
    return x;
  }
}

// Segments of at most LANES entries, one per lane, 64 / LANES segments side by side in a wavefront; otherwise as
// merge_sorted_kernel below.  Bound by the chain of reads before the entries, so several share it: 1.5 M segments
// of up to 64 entries, 12 on average, one to a wavefront, took 438 us, now 190.
template <int LANES, typename WT, bool WEIGHTED>
__global__ __launch_bounds__(256) void merge_small_kernel(const int64_t *__restrict__ segment,
                                                          const int32_t *__restrict__ list, int64_t count, Packing pack,
                                                          uint32_t *__restrict__ entries, WT *__restrict__ weight,
                                                          int64_t *__restrict__ length) {
  constexpr int kPerWave = 64 / LANES;
  __shared__ WT extra[256];
  const int lane = threadIdx.x & 63, gl = lane & (LANES - 1), group = lane & ~(LANES - 1);
  const uint64_t of_group = ~uint64_t{0} >> (64 - LANES) << group, below = (uint64_t{1} << lane) - 1;
  const int64_t wave = (blockIdx.x * 256LL + threadIdx.x) >> 6, waves = (gridDim.x * 256LL) >> 6;
  for (int64_t base = wave * kPerWave; base < count; base += waves * kPerWave) {
    const int64_t i = base + lane / LANES;
    const bool live = i < count;
    const int32_t a = list[live ? i : base];
    const int64_t lo = segment[a];
    const int size = live ? static_cast<int>(segment[a + 1] - lo) : 0;
    const uint32_t word = gl < size ? entries[lo + gl] : kInside;
    uint32_t key[1] = {word};
    key_blocks<2, LANES, LANES>(key, static_cast<uint32_t>(gl));
    const uint32_t column = WEIGHTED ? pack.column(key[0]) : key[0];
    const uint32_t before = __shfl_up(column, 1, LANES);
    const bool starts = gl == 0 || column != before, head = starts && column != kInside;
    const uint64_t changes = __ballot(starts) & of_group & ~below & ~(uint64_t{1} << lane);
    const uint64_t heads = __ballot(head) & of_group;
    const int end = changes != 0 ? __builtin_ctzll(changes) : group + LANES;  // lane behind the run
    WT sum = static_cast<WT>(end - lane);
    if constexpr (WEIGHTED) {
      const WT mine = key[0] != kInside ? static_cast<WT>(key[0] & pack.top) : WT(0);
      const WT upto = sum_upto_in_group<LANES, WT>(mine, gl);
      sum = __shfl(upto, end - 1, 64) - upto + mine;
      const bool apart = word != kInside && (word & pack.top) == pack.top;
      if (__ballot(apart) != 0) {  // what the words left out, to the first lane of its run
        extra[threadIdx.x] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        int to = -1;
        for (int q = LANES - 1; q >= 0; --q)
          if (__shfl(column, q, LANES) == pack.column(word)) to = q;
        if (apart) atomicAdd(&extra[threadIdx.x - gl + to], static_cast<WT>(weight[lo + gl] - pack.top));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        sum += extra[threadIdx.x];
      }
    }
    if (head) {
      const int rank = __popcll(heads & below);
      entries[lo + rank] = pack.entry(column, sum);
      if (sum >= pack.top) weight[lo + rank] = sum;
    }
    if (live && gl == 0) length[a] = __popcll(heads);
  }
}

// Segments of at most WAVES * 64 * R entries, WAVES wavefronts each: a bitonic network over the
// registers of the lanes (R consecutive elements per lane; between wavefronts through LDS),
// then equal columns are merged in place.  The sum of a run is the difference of the running
// sums at its end and at the end of the run before.  An entry is sorted as the word it is held in, weight
// included; what a word does not hold of a weight is added to the sum of its column afterwards.  Bound by the network's
// instructions: 74 M entries in segments of up to 2,048 take 0.36 ms, 65 M weighted ones 0.30 (0.66 and 1.00 with
// columns and weights sorted as pairs by compare and select).
template <int R, int WAVES, typename WT, bool WEIGHTED>
__global__ __launch_bounds__(256) void merge_sorted_kernel(const int64_t *__restrict__ segment,
                                                           const int32_t *__restrict__ list, int64_t count,
                                                           Packing pack, uint32_t *__restrict__ entries,
                                                           WT *__restrict__ weight, int64_t *__restrict__ length) {
  static_assert(WAVES == 1 || WAVES == 4, "a wavefront or a workgroup");
  constexpr int kWave = 64 * R, kAll = kWave * WAVES;
  constexpr int kTeams = 4 / WAVES;  // segments a workgroup works at
  __shared__ uint32_t run_column[kTeams][kAll];  // of each run; between wavefronts: what they exchange
  __shared__ WT run_end[kTeams][kAll];           // running sum at the end of each run
  __shared__ int wave_heads[4];
  __shared__ WT wave_sum[4];
  __shared__ uint32_t wave_last[4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), team = wave / WAVES;
  const int member = wave % WAVES;  // wavefront within the team
  const uint32_t index = member * 64 + lane, first = index * R;
  // a team takes the segments team, team + teams, ...; with several teams there are no barriers
  auto team_sync = [] {
    if constexpr (WAVES > 1) {
      __syncthreads();
    } else {  // LDS accesses of a wavefront take effect in their order; the compiler must keep it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kTeams + team; i < count;
       i += static_cast<int64_t>(gridDim.x) * kTeams) {
    const int32_t a = list[i];
    const int64_t lo = segment[a];
    const uint32_t size = static_cast<uint32_t>(segment[a + 1] - lo);
    uint32_t *const entry = entries + lo;
    uint32_t key[R];
    WT w[R];
    bool held_apart = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // lane-consecutive loads; where an element starts does not matter to a sort
      const uint32_t e = member * kWave + r * 64 + lane;
      key[r] = e < size ? entry[e] : kInside;
      if constexpr (WEIGHTED) held_apart |= key[r] != kInside && (key[r] & pack.top) == pack.top;
    }
    bool apart = false;  // whether the segment has weights that its words do not hold
    if constexpr (WEIGHTED) {
      if constexpr (WAVES == 1) apart = __ballot(held_apart) != 0;
      else apart = __syncthreads_or(held_apart) != 0;
    }
    key_blocks<2, kWave, kAll>(key, index);
    if constexpr (WAVES == 4) {
      uint32_t *const swap = run_column[0];
      auto across = [&](uint32_t larger, int partner) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) swap[r * 256 + threadIdx.x] = key[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) key[r] = med3(key[r], swap[r * 256 + partner], larger);
      };
      across(spread<64>(index) ^ spread<128>(index), threadIdx.x ^ 64);
      key_merge<2 * kWave, kWave / 2, kAll>(key, index);
      across(spread<128>(index), threadIdx.x ^ 128);
      across(spread<64>(index), threadIdx.x ^ 64);
      key_merge<4 * kWave, kWave / 2, kAll>(key, index);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      w[r] = WEIGHTED ? static_cast<WT>(key[r] & pack.top) : WT(1);
      if constexpr (WEIGHTED) key[r] = pack.column(key[r]);
    }
    // heads of runs: a column that differs from the one before; what lies inside the cluster is at the end
    if constexpr (WAVES == 4) {
      if (lane == 63) wave_last[wave] = key[R - 1];
      __syncthreads();
    }
    uint32_t before = __shfl_up(key[R - 1], 1, 64);
    if (lane == 0) before = member > 0 ? wave_last[wave - 1] : kInside;
    int rank = -1, distinct = 0;  // of the run that the element before belongs to
    WT sum = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const unsigned long long heads = __ballot(key[r] != kInside && key[r] != (r == 0 ? before : key[r - 1]));
      rank += lanes_below(heads);
      distinct += __popcll(heads);
      if constexpr (WEIGHTED) sum += key[r] != kInside ? w[r] : WT(0);
    }
    WT running = static_cast<WT>(first);  // of the entries before; ones, unless they have weights
    if constexpr (WEIGHTED) {
      const WT upto = sum_upto_lane(sum, lane);
      running = upto - sum;
      if constexpr (WAVES == 4)
        if (lane == 63) wave_sum[wave] = upto;
    }
    if constexpr (WAVES == 4) {
      if (lane == 63) wave_heads[wave] = distinct;
      __syncthreads();
      distinct = 0;
      for (int q = 0; q < 4; ++q) {
        if (q < wave) {
          rank += wave_heads[q];
          if constexpr (WEIGHTED) running += wave_sum[q];
        }
        distinct += wave_heads[q];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (key[r] != (r == 0 ? before : key[r - 1])) {
        if (rank >= 0) run_end[team][rank] = running;  // the run before ends here
        if (key[r] != kInside) run_column[team][++rank] = key[r];
      }
      running += key[r] != kInside ? w[r] : WT(0);
    }
    // the team's last lane knows the end of the last run, if nothing inside the cluster follows it
    if (first + R == kAll && key[R - 1] != kInside) run_end[team][rank] = running;
    team_sync();
    if (WEIGHTED && apart) {  // the sums themselves in place of their ends, and what the words left out
      WT sums[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int c = r * 64 * WAVES + index;
        sums[r] = c < distinct ? run_end[team][c] - (c > 0 ? run_end[team][c - 1] : WT(0)) : WT(0);
      }
      team_sync();
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r * 64 * WAVES + static_cast<int>(index) < distinct) run_end[team][r * 64 * WAVES + index] = sums[r];
      team_sync();
      for (uint32_t e = index; e < size; e += 64 * WAVES) {  // the segment is as it was until the loop below
        const uint32_t word = entry[e];
        if (word == kInside || (word & pack.top) != pack.top) continue;
        const int c = row_of_entry<uint32_t>(run_column[team], 0, distinct - 1, pack.column(word));
        atomicAdd(&run_end[team][c], static_cast<WT>(weight[lo + e] - pack.top));
      }
      team_sync();
    }
    for (int c = index; c < distinct; c += 64 * WAVES) {
      const WT total = run_end[team][c] - (c > 0 && !apart ? run_end[team][c - 1] : WT(0));
      entry[c] = pack.entry(run_column[team][c], total);
      if (total >= pack.top) weight[lo + c] = total;
    }
    if (first == 0) length[a] = distinct;
    team_sync();
  }
}

// Calls body(entry, word, column) for the entries [lo, hi) with the workgroup's threads side by side,
// eight requested before the first is used: a workgroup has its compute unit nearly to itself
// and would otherwise wait for memory once per entry and thread (counting 55 M entries in 9,000
// segments: 110 us, 690 us one by one).
template <class Body>
__device__ __forceinline__ void for_entries(const uint32_t *__restrict__ entry, Packing pack, int64_t lo, int64_t hi,
                                            Body body) {
  constexpr int kAhead = 8;
  const int64_t step = blockDim.x;
  for (int64_t first = lo + threadIdx.x; first < hi; first += kAhead * step) {
    uint32_t b[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) b[q] = entry[std::min(first + q * step, hi - 1)];
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
      if (first + q * step < hi) body(first + q * step, b[q], pack.column(b[q]));
  }
}

// Marks the columns of a piece of a segment in the bitmap.  Returns the number of its words.
__device__ inline int mark_piece(const uint32_t *__restrict__ entry, Packing pack, int64_t lo, int64_t hi, int64_t piece,
                                 int64_t columns, uint32_t *bits) {
  const uint32_t base = static_cast<uint32_t>(piece << kPieceBits);
  const int words = static_cast<int>(std::min<int64_t>(kPieceWords, (columns - base + 31) / 32));
  const uint32_t width = static_cast<uint32_t>(words) * 32u;
  for (int w = threadIdx.x; w < kPieceWords; w += blockDim.x) bits[w] = 0;
  __syncthreads();
  for_entries(entry, pack, lo, hi, [&](int64_t, uint32_t, uint32_t b) {
    b -= base;  // columns of other pieces, and kInside, are past the bitmap
    if (b < width) atomicOr(&bits[b >> 5], 1u << (b & 31));
  });
  __syncthreads();
  return words;
}

// Distinct columns of every strip of the segments of a list, and of the segments.
__global__ __launch_bounds__(512) void count_pieces_kernel(const int64_t *__restrict__ segment,
                                                           const int32_t *__restrict__ list, int64_t count,
                                                           int64_t pieces, int64_t columns,
                                                           const uint32_t *__restrict__ entry, Packing pack,
                                                           uint32_t *__restrict__ in_strip,
                                                           int64_t *__restrict__ length) {
  constexpr int kStripWords = kPieceWords / kStripsPerPiece;
  __shared__ uint32_t bits[kPieceWords];
  __shared__ uint32_t total;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t job = blockIdx.x; job < count * pieces; job += gridDim.x) {
    const int32_t a = list[job / pieces];
    if (threadIdx.x == 0) total = 0;
    mark_piece(entry, pack, segment[a], segment[a + 1], job % pieces, columns, bits);
    for (int strip = wave; strip < kStripsPerPiece; strip += 8) {
      uint32_t mine = 0;
      for (int w = lane; w < kStripWords; w += 64) mine += __popc(bits[strip * kStripWords + w]);
      for (int off = 32; off >= 1; off >>= 1) mine += __shfl_xor(mine, off, 64);
      if (lane == 0) {
        in_strip[job * kStripsPerPiece + strip] = mine;
        if (mine) atomicAdd(&total, mine);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && total)
      atomicAdd(reinterpret_cast<unsigned long long *>(length + a), static_cast<unsigned long long>(total));
    __syncthreads();  // bits and total are rewritten in the next round
  }
}

// Distinct columns in the strips [0, upto) of a segment, added to *sum (which is clear).
__device__ inline void add_strips(const uint32_t *__restrict__ in_strip, int64_t upto, unsigned long long *sum) {
  unsigned long long mine = 0;
  for (int64_t p = threadIdx.x; p < upto; p += blockDim.x) mine += in_strip[p];
  if (mine) atomicAdd(sum, mine);
}

// Writes the pieces of the segments of a list where they belong: the number of set bits below
// an entry's column is the place of that column and of its sum (40 M entries of 8,900 segments:
// 0.68 ms; walking the set bits instead, where the rows are dense in small ids, 1.21 ms).
template <typename WT, bool WEIGHTED>
__global__ __launch_bounds__(1024) void write_pieces_kernel(const int64_t *__restrict__ segment,
                                                            const int32_t *__restrict__ list, int64_t count,
                                                            int64_t pieces, int64_t columns,
                                                            const uint32_t *__restrict__ entry, Packing pack,
                                                            const WT *__restrict__ weight,
                                                            const uint32_t *__restrict__ in_strip,
                                                            const int64_t *__restrict__ xadj_out,
                                                            int32_t *__restrict__ adj_out,
                                                            WT *__restrict__ mult_out) {
  constexpr uint32_t kSums = kSumBytes / (sizeof(WT) + 4);
  constexpr int kPairs = kPieceWords / 2, kPerThread = kPairs / 1024;
  __shared__ unsigned long long bits[kPairs];
  __shared__ uint32_t below[kPairs];  // set bits in the pairs of words before
  __shared__ WT sums[kSums];
  __shared__ uint32_t found[kSums];
  __shared__ uint32_t wave_total[16];
  __shared__ unsigned long long earlier;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t job = blockIdx.x; job < count * pieces; job += gridDim.x) {
    const int64_t which = job / pieces, piece = job % pieces;
    const int32_t a = list[which];
    const int64_t lo = segment[a], hi = segment[a + 1];
    __syncthreads();  // the previous piece is done with the LDS
    if (threadIdx.x == 0) earlier = 0;
    const uint32_t width = 32u * mark_piece(entry, pack, lo, hi, piece, columns, reinterpret_cast<uint32_t *>(bits));
    add_strips(in_strip + which * pieces * kStripsPerPiece, piece * kStripsPerPiece, &earlier);
    // exclusive scan of the set bits: kPerThread pairs per thread, then over the workgroup
    const int p0 = threadIdx.x * kPerThread;
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < kPerThread; ++q) mine += __popcll(bits[p0 + q]);
    uint32_t upto = mine;
    for (int step = 1; step < 64; step <<= 1) {
      const uint32_t x = __shfl_up(upto, step, 64);
      if (lane >= step) upto += x;
    }
    if (lane == 63) wave_total[wave] = upto;
    __syncthreads();
    uint32_t rank = upto - mine, distinct = 0;
    for (int q = 0; q < 16; ++q) {
      if (q < wave) rank += wave_total[q];
      distinct += wave_total[q];
    }
    const int64_t out = xadj_out[a] + static_cast<int64_t>(earlier);
    const uint32_t base = static_cast<uint32_t>(piece << kPieceBits);
    for (int q = 0; q < kPerThread; ++q) {
      below[p0 + q] = rank;
      rank += __popcll(bits[p0 + q]);
    }
    for (uint32_t first = 0; first < distinct; first += kSums) {
      const uint32_t here = std::min(kSums, distinct - first);
      for (uint32_t c = threadIdx.x; c < here; c += 1024) sums[c] = 0;
      __syncthreads();
      for_entries(entry, pack, lo, hi, [&](int64_t e, uint32_t word, uint32_t b) {
        b -= base;
        if (b < width) {
          const uint32_t c = below[b >> 6] + __popcll(bits[b >> 6] & ((1ull << (b & 63)) - 1)) - first;
          if (c < here) {
            found[c] = base + b;  // by every entry of that column alike
            atomicAdd(&sums[c], WEIGHTED ? pack.weight(word, weight, e) : WT(1));
          }
        }
      });
      __syncthreads();
      for (uint32_t c = threadIdx.x; c < here; c += 1024) {
        adj_out[out + first + c] = static_cast<int32_t>(found[c]);
        mult_out[out + first + c] = sums[c];
      }
      __syncthreads();
    }
  }
}

__global__ __launch_bounds__(256) void clear_table_kernel(uint4 *__restrict__ table, int64_t units) {
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < units; i += gridDim.x * 256LL) table[i] = uint4{0, 0, 0, 0};
}

// Counts the entries of the longest segments by column: a workgroup takes a slice of a segment and
// a strip of columns, counts in LDS and adds what it has to the segment's row of the table.  (With
// one workgroup per strip of a segment, which read all of it, the second and third level of a
// graph of 535 M entries, a few segments of tens of millions over two strips, took 60 and 28 ms.)
template <typename WT, bool WEIGHTED>
__global__ __launch_bounds__(1024) void count_dense_kernel(const int64_t *__restrict__ segment,
                                                           const int32_t *__restrict__ list,
                                                           const Slice *__restrict__ slices, int64_t first_strip,
                                                           int64_t strips,
                                                           const uint32_t *__restrict__ entry, Packing pack,
                                                           const WT *__restrict__ weight, WT *__restrict__ table) {
  constexpr int kWidth = 1 << kStripBits;
  __shared__ WT sums[kWidth];
  const Slice slice = slices[blockIdx.x];
  const int64_t strip = first_strip + blockIdx.y;
  const int32_t a = list[slice.row];
  const int64_t lo = segment[a] + slice.part * kSlice, hi = std::min(lo + kSlice, segment[a + 1]);
  const uint32_t base = static_cast<uint32_t>(strip << kStripBits);
  for (int c = threadIdx.x; c < kWidth; c += 1024) sums[c] = 0;
  __syncthreads();
  for_entries(entry, pack, lo, hi, [&](int64_t e, uint32_t word, uint32_t b) {
    b -= base;  // columns of other strips, and kInside, are past the counters
    if (b < static_cast<uint32_t>(kWidth)) atomicAdd(&sums[b], WEIGHTED ? pack.weight(word, weight, e) : WT(1));
  });
  __syncthreads();
  WT *const row = table + (slice.row * strips + strip) * kWidth;
  for (int c = threadIdx.x; c < kWidth; c += 1024)
    if (sums[c] != 0) atomicAdd(row + c, sums[c]);
}

// The number of columns met in every strip of the counted segments (WRITE = false), or those
// columns and their sums where they belong.  One workgroup per segment and strip.
template <typename WT, bool WRITE>
__global__ __launch_bounds__(1024) void dense_strips_kernel(const int32_t *__restrict__ list, int64_t strips,
                                                            const WT *__restrict__ table,
                                                            uint32_t *__restrict__ in_strip,
                                                            int64_t *__restrict__ length,
                                                            const int64_t *__restrict__ xadj_out,
                                                            int32_t *__restrict__ adj_out,
                                                            WT *__restrict__ mult_out) {
  constexpr int kWidth = 1 << kStripBits, kPerWave = kWidth / 16;
  __shared__ uint32_t wave_total[16];
  __shared__ unsigned long long earlier;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t job = blockIdx.x, which = job / strips, strip = job % strips;
  const int32_t a = list[which];
  const WT *const mine = table + job * kWidth + wave * kPerWave;
  uint32_t met = 0;
  for (int c = lane; c < kPerWave; c += 64) met += __popcll(__ballot(mine[c] != 0));
  if (lane == 0) wave_total[wave] = met;
  if (threadIdx.x == 0) earlier = 0;
  __syncthreads();
  if constexpr (!WRITE) {
    if (threadIdx.x == 0) {
      uint32_t total = 0;
      for (int q = 0; q < 16; ++q) total += wave_total[q];
      in_strip[job] = total;
      if (total) atomicAdd(reinterpret_cast<unsigned long long *>(length + a), static_cast<unsigned long long>(total));
    }
  } else {
    add_strips(in_strip + which * strips, strip, &earlier);
    __syncthreads();
    int64_t out = xadj_out[a] + static_cast<int64_t>(earlier);
    for (int q = 0; q < wave; ++q) out += wave_total[q];
    for (int c = lane; c < kPerWave; c += 64) {
      const WT sum = mine[c];
      const unsigned long long set = __ballot(sum != 0);
      if (sum != 0) {
        const int64_t at = out + __popcll(set & ((1ull << lane) - 1));
        adj_out[at] = static_cast<int32_t>((strip << kStripBits) + wave * kPerWave + c);
        mult_out[at] = sum;
      }
      out += __popcll(set);
    }
  }
}

// tile_row[k] = coarse row that holds entry k * kGatherTile of the coarse graph, and behind the last tile's the last
// row with entries.
__global__ __launch_bounds__(256) void coarse_tiles_kernel(const int64_t *__restrict__ xadj_out, int64_t n_coarse,
                                                           int64_t nnz_coarse, int32_t *__restrict__ tile_row) {
  for (int64_t a = blockIdx.x * 256LL + threadIdx.x; a < n_coarse; a += gridDim.x * 256LL) {
    const int64_t lo = xadj_out[a], hi = xadj_out[a + 1];
    for (int64_t k = (lo + kGatherTile - 1) / kGatherTile; k * kGatherTile < hi; ++k)
      tile_row[k] = static_cast<int32_t>(a);
    if (lo < hi && hi == nnz_coarse) tile_row[(nnz_coarse + kGatherTile - 1) / kGatherTile] = static_cast<int32_t>(a);
  }
}

// Copies the segments that were merged in place, those of up to `sorted_to` or more than `radix_from`
// entries, to the coarse graph.  A workgroup takes kGatherTile consecutive entries of that: with a wavefront per
// segment, bound by the chain of reads before its first entry, 96 M entries took 500 us, now 297.
template <typename WT>
__global__ __launch_bounds__(256) void copy_merged_kernel(const int64_t *__restrict__ segment, int64_t sorted_to,
                                                          int64_t radix_from, const int32_t *__restrict__ tile_row,
                                                          int64_t nnz_coarse,
                                                          const uint32_t *__restrict__ entry, Packing pack,
                                                          const WT *__restrict__ weight,
                                                          const int64_t *__restrict__ xadj_out,
                                                          int32_t *__restrict__ adj_out,
                                                          WT *__restrict__ mult_out) {
  constexpr int kUnits = 8;
  constexpr int64_t kElsewhere = INT64_MIN;
  __shared__ RowStarts rows;
  __shared__ int64_t from[kGatherRows];  // entry of place 0 of the row, were it that long
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto start_of = [&](int32_t a, int64_t p) -> int64_t {
    const int64_t lo = segment[a], size = segment[a + 1] - lo;
    return size <= sorted_to || size > radix_from ? lo - p : kElsewhere;
  };
  const int64_t tiles = (nnz_coarse + kGatherTile - 1) / kGatherTile;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t e0 = tile * kGatherTile, e1 = std::min(e0 + kGatherTile, nnz_coarse);
    const int32_t row0 = tile_row[tile], row1 = tile_row[tile + 1];
    const bool in_lds = lay_out_rows(rows, xadj_out, row0, row1, e0, e1,
                                     [&](int32_t k, int32_t a, int64_t p) { from[k] = start_of(a, p); });
    for (int step = 0; step < kGatherTile / 256; step += kUnits) {
      const int64_t first = e0 + step * 256 + threadIdx.x;
      if (first >= e1) break;
      int64_t at[kUnits];
      uint32_t word[kUnits];
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        const int64_t e = std::min(first + q * 256, e1 - 1);
        int64_t start;
        if (in_lds) {
          start = from[rows.row((step + q) * 4 + wave)];
        } else {
          const int32_t a = row_of_entry<int64_t>(xadj_out, row0, row1, e);
          start = start_of(a, xadj_out[a]);
        }
        at[q] = start == kElsewhere || first + q * 256 >= e1 ? -1 : start + e;
      }
#pragma unroll
      for (int q = 0; q < kUnits; ++q) word[q] = __builtin_nontemporal_load(entry + std::max<int64_t>(at[q], 0));
#pragma unroll
      for (int q = 0; q < kUnits; ++q)
        if (at[q] >= 0) {
          const int64_t e = first + q * 256;
          __builtin_nontemporal_store(static_cast<int32_t>(pack.column(word[q])), adj_out + e);
          __builtin_nontemporal_store(pack.weight(word[q], weight, at[q]), mult_out + e);
        }
    }
  }
}

// What is to be known of the coarse rows before there is room for them.
__global__ __launch_bounds__(256) void coarse_shape_kernel(const int64_t *__restrict__ length,
                                                           const int64_t *__restrict__ xadj_out, int64_t n_coarse,
                                                           Classes *__restrict__ classes) {
  __shared__ unsigned int block_top;
  if (threadIdx.x == 0) block_top = 0;
  __syncthreads();
  unsigned int top = 0;
  for (int64_t a = blockIdx.x * 256LL + threadIdx.x; a < n_coarse; a += gridDim.x * 256LL)
    top = max(top, static_cast<unsigned int>(length[a]));
  raise_by_block(&classes->longest, top, &block_top);
  if (blockIdx.x == 0 && threadIdx.x == 0) classes->entries = xadj_out[n_coarse];
}

__global__ void clear_classes_kernel(Classes *classes) { *classes = Classes{}; }

template <typename OffT, typename WT, bool WEIGHTED>
int quotient(gosh::DeviceCoarsener *dc, const gosh::DeviceLevel &fine, int64_t n_coarse, gosh::DeviceLevel &coarse,
             int64_t *xadj_out) {
  const int64_t n = fine.n, nnz = fine.nnz;
  const OffT *xadj = static_cast<const OffT *>(fine.xadj);
  const Packing pack = Packing::for_columns(n_coarse), held = WEIGHTED ? pack : Packing{0, 0};  // merged, and before
  gosh::Buffers buf(dc->pool);
  uint32_t *entry = nullptr;
  WT *weight = nullptr;
  int64_t *segment = nullptr, *length = nullptr;
  int32_t *list = nullptr;
  Classes *classes = nullptr;
  if (int rc = buf.alloc(&entry, static_cast<size_t>(nnz), "entries")) return rc;
  if (int rc = buf.alloc(&weight, static_cast<size_t>(nnz), "multiplicities")) return rc;
  if (int rc = buf.alloc(&segment, static_cast<size_t>(n_coarse) + 1, "coarse rows")) return rc;
  if (int rc = buf.alloc(&length, static_cast<size_t>(n_coarse) + 1, "coarse row lengths")) return rc;
  if (int rc = buf.alloc(&list, static_cast<size_t>(n_coarse) * kWays, "lists of coarse rows")) return rc;
  if (int rc = buf.alloc(&classes, 1, "counters")) return rc;
  Slice *slices = nullptr;  // of segments longer than 2^15 entries, at most 1 + S / kSlice each
  if (int rc = buf.alloc(&slices, static_cast<size_t>(nnz / (1 << 14)) + 1, "slices")) return rc;
  hipLaunchKernelGGL(clear_classes_kernel, dim3(1), dim3(1), 0, nullptr, classes);
  const int flat_blocks = blocks_for(n + 1, 256);

  {  // the fine rows in cluster order
    int32_t *order = nullptr, *cluster = nullptr, *tile_row = nullptr;
    OffT *begin = nullptr;
    int64_t *lengths = nullptr, *pos = nullptr;
    const int64_t tiles = (nnz + kGatherTile - 1) / kGatherTile;
    const rocprim::counting_iterator<int32_t> ids(0);
    if (int rc = buf.alloc(&order, static_cast<size_t>(n), "cluster order")) return rc;
    if (int rc = buf.alloc(&cluster, static_cast<size_t>(n), "sorted clusters")) return rc;
    if (int rc = buf.alloc(&lengths, static_cast<size_t>(n) + 1, "row lengths")) return rc;
    if (int rc = buf.alloc(&pos, static_cast<size_t>(n) + 1, "row places")) return rc;
    if (int rc = buf.alloc(&begin, static_cast<size_t>(n), "row starts")) return rc;
    if (int rc = buf.alloc(&tile_row, static_cast<size_t>(tiles) + 1, "tile rows")) return rc;
    unsigned bits = 1;
    while (bits < 31 && (n_coarse >> bits) != 0) ++bits;
    size_t sort_bytes = 0, scan_bytes = 0;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs<gosh::SortConfig>(nullptr, sort_bytes, fine.map, cluster, ids, order,
                                                             static_cast<size_t>(n), 0u, bits, nullptr),
                 "cluster sort (size query)");
    GOSH_TRY_HIP(rocprim::exclusive_scan(nullptr, scan_bytes, lengths, pos, int64_t(0), static_cast<size_t>(n) + 1,
                                         rocprim::plus<int64_t>(), nullptr),
                 "row scan (size query)");
    char *temp = nullptr;
    if (int rc = buf.alloc(&temp, std::max(sort_bytes, scan_bytes), "sort workspace")) return rc;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs<gosh::SortConfig>(temp, sort_bytes, fine.map, cluster, ids, order,
                                                             static_cast<size_t>(n), 0u, bits, nullptr),
                 "cluster sort");
    hipLaunchKernelGGL(row_lengths_kernel<OffT>, dim3(flat_blocks), dim3(256), 0, nullptr, xadj, order, n, lengths,
                       begin);
    GOSH_TRY_HIP(rocprim::exclusive_scan(temp, scan_bytes, lengths, pos, int64_t(0), static_cast<size_t>(n) + 1,
                                         rocprim::plus<int64_t>(), nullptr),
                 "row scan");
    hipLaunchKernelGGL(segments_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, cluster, pos, n, nnz, n_coarse,
                       segment, tile_row);
    ClusterTable table{reinterpret_cast<const char *>(fine.map), 4, ~0u};
    uint32_t *narrow = nullptr;  // and a word for what is read past the last vertex; without room the map itself does
    if (n >= kNarrowFrom && n_coarse <= (int64_t{1} << 24) && !gosh::denied(gosh::kDenyNarrow) &&
        buf.alloc(&narrow, static_cast<size_t>((n + 3) / 4) * 3 + 1, "narrow map") == GOSH_OK) {
      hipLaunchKernelGGL(narrow_map_kernel, dim3(blocks_for((n + 3) / 4, 256)), dim3(256), 0, nullptr, fine.map, n,
                         narrow);
      table = ClusterTable{reinterpret_cast<const char *>(narrow), 3, 0xFFFFFFu};
    }
    hipLaunchKernelGGL((gather_kernel<OffT, WT, WEIGHTED>), dim3(blocks_for(nnz, kGatherTile)), dim3(256), 0, nullptr,
                       fine.adj, static_cast<const WT *>(fine.mult), table, begin, cluster, pos, tile_row, nnz, pack,
                       entry, weight, classes);
    if (int rc = gosh::check_launch("gather_kernel")) return rc;
    for (void *p : {static_cast<void *>(order), static_cast<void *>(cluster), static_cast<void *>(lengths),
                    static_cast<void *>(begin), static_cast<void *>(pos), static_cast<void *>(tile_row),
                    static_cast<void *>(temp), static_cast<void *>(narrow)})
      buf.release(p);  // what takes them up again is on the same stream
  }
  const int64_t radix_from = gosh::seam(gosh::kSeamRadixFrom);
  const Ways ways{radix_from ? radix_from : kRankColumns, radix_from ? radix_from : kCountColumns,
                  static_cast<int>(sizeof(WT))};
  hipLaunchKernelGGL(classify_segments_kernel, dim3(blocks_for(n_coarse, 1024)), dim3(1024), 0, nullptr, segment,
                     n_coarse, list, length, slices, ways, classes);
  if (int rc = gosh::check_launch("classify_segments_kernel")) return rc;
  Classes c{};
  GOSH_TRY_HIP(hipMemcpy(&c, classes, sizeof(c), hipMemcpyDeviceToHost), "read segment classes");

  // merge: in place, or counted
  bool radix_merged = false;  // the segments of the kRadix list are merged in place
  if (c.count[kRadix] > 0) {
    const int rc = gosh::merge_by_radix<WT, WEIGHTED>(dc->pool, segment, list + kRadix * n_coarse, c.count[kRadix],
                                                c.columns, pack, entry, weight, length);
    if (rc != GOSH_OK && rc != GOSH_ENOMEM) return rc;
    radix_merged = rc == GOSH_OK;
  }
  const int32_t *dense_list = list + kDense * n_coarse;
  const int64_t pieces = pieces_of(c.columns), strips = pieces * kStripsPerPiece;
  const int64_t dense_strips = (static_cast<int64_t>(c.columns) + (1 << kStripBits) - 1) >> kStripBits;
  int64_t denses = c.count[kDense];
  const int64_t dense_jobs = denses * dense_strips;
  uint32_t *in_dense_strip = nullptr;
  WT *table = nullptr;
  const int64_t counters = dense_jobs << kStripBits;
  if (denses > 0 && (gosh::denied(gosh::kDenyTable) ||
                     buf.alloc(&table, static_cast<size_t>(counters), "counters of coarse rows") != GOSH_OK))
    denses = 0;
  if (denses > 0) {
    if (int rc = buf.alloc(&in_dense_strip, static_cast<size_t>(dense_jobs), "strips of coarse rows")) return rc;
    const int64_t units = counters * static_cast<int64_t>(sizeof(WT)) / 16;
    hipLaunchKernelGGL(clear_table_kernel, dim3(blocks_for(units, 256)), dim3(256), 0, nullptr,
                       reinterpret_cast<uint4 *>(table), units);
    // at most 2^17 strips: columns are below 2^31
    for (int64_t first = 0; first < dense_strips; first += 65535)
      hipLaunchKernelGGL((count_dense_kernel<WT, WEIGHTED>),
                         dim3(c.slices, static_cast<unsigned>(std::min<int64_t>(dense_strips - first, 65535))), dim3(1024), 0,
                         nullptr, segment, dense_list, slices, first, dense_strips, entry, held, weight, table);
    hipLaunchKernelGGL((dense_strips_kernel<WT, false>), dim3(static_cast<unsigned>(dense_jobs)), dim3(1024), 0, nullptr,
                       dense_list, dense_strips, table, in_dense_strip, length, xadj_out, nullptr, nullptr);
  }
  // the bitmap also takes the segments that there was no memory to sort or to count
  struct Ranked {
    const int32_t *list;
    int64_t count;
    uint32_t *in_strip;
  } ranked[3] = {{list + kBitmap * n_coarse, c.count[kBitmap], nullptr},
                 {dense_list, denses > 0 ? 0 : c.count[kDense], nullptr},
                 {list + kRadix * n_coarse, radix_merged ? 0 : c.count[kRadix], nullptr}};
  for (Ranked &r : ranked) {
    if (r.count == 0) continue;
    if (int rc = buf.alloc(&r.in_strip, static_cast<size_t>(r.count * strips), "strips of coarse rows")) return rc;
    hipLaunchKernelGGL(count_pieces_kernel, dim3(blocks_for(r.count * pieces, 1)), dim3(512), 0, nullptr, segment,
                       r.list, r.count, pieces, static_cast<int64_t>(c.columns), entry, held, r.in_strip, length);
  }
  auto merge_sorted = [&](auto kernel, int cls, int teams) {
    if (c.count[cls] > 0)
      hipLaunchKernelGGL(kernel, dim3(blocks_for(c.count[cls], teams)), dim3(256), 0, nullptr, segment,
                         list + cls * n_coarse, static_cast<int64_t>(c.count[cls]), pack, entry, weight, length);
  };
  merge_sorted(merge_sorted_kernel<16, 4, WT, WEIGHTED>, 8, 1);
  merge_sorted(merge_sorted_kernel<8, 4, WT, WEIGHTED>, 7, 1);
  merge_sorted(merge_sorted_kernel<16, 1, WT, WEIGHTED>, 6, 4);
  merge_sorted(merge_sorted_kernel<8, 1, WT, WEIGHTED>, 5, 4);
  merge_sorted(merge_sorted_kernel<4, 1, WT, WEIGHTED>, 4, 4);
  merge_sorted(merge_sorted_kernel<2, 1, WT, WEIGHTED>, 3, 4);
  merge_sorted(merge_small_kernel<64, WT, WEIGHTED>, 2, 4);
  merge_sorted(merge_small_kernel<32, WT, WEIGHTED>, 1, 8);
  merge_sorted(merge_small_kernel<16, WT, WEIGHTED>, 0, 16);
  if (int rc = gosh::check_launch("merge of the coarse rows")) return rc;

  // offsets; the last length is never read
  {
    size_t bytes = 0;
    GOSH_TRY_HIP(rocprim::exclusive_scan(nullptr, bytes, length, xadj_out, int64_t(0), static_cast<size_t>(n_coarse) + 1,
                                         rocprim::plus<int64_t>(), nullptr),
                 "offset scan (size query)");
    char *temp = nullptr;
    if (int rc = buf.alloc(&temp, bytes, "scan workspace")) return rc;
    GOSH_TRY_HIP(rocprim::exclusive_scan(temp, bytes, length, xadj_out, int64_t(0), static_cast<size_t>(n_coarse) + 1,
                                         rocprim::plus<int64_t>(), nullptr),
                 "offset scan");
  }
  hipLaunchKernelGGL(coarse_shape_kernel, dim3(std::min(blocks_for(n_coarse, 2048), 256)), dim3(256), 0, nullptr, length,
                     xadj_out, n_coarse, classes);
  if (int rc = gosh::check_launch("coarse_shape_kernel")) return rc;
  Classes shape{};
  GOSH_TRY_HIP(hipMemcpy(&shape, classes, sizeof(shape), hipMemcpyDeviceToHost), "read coarse size");
  coarse.nnz = shape.entries;
  coarse.top_degree = shape.longest;
  if (int rc = persistent(&coarse.adj, static_cast<size_t>(coarse.nnz), "coarse adjacency")) return rc;
  WT *mult_out = nullptr;
  if (int rc = persistent(&mult_out, static_cast<size_t>(coarse.nnz), "coarse multiplicities")) return rc;
  coarse.mult = mult_out;
  coarse.mult_is64 = sizeof(WT) == 8;
  if (denses > 0)
    hipLaunchKernelGGL((dense_strips_kernel<WT, true>), dim3(static_cast<unsigned>(dense_jobs)), dim3(1024), 0, nullptr,
                       dense_list, dense_strips, table, in_dense_strip, length, xadj_out, coarse.adj, mult_out);
  for (const Ranked &r : ranked)
    if (r.count > 0)
      hipLaunchKernelGGL((write_pieces_kernel<WT, WEIGHTED>), dim3(blocks_for(r.count * pieces, 1)), dim3(1024), 0,
                         nullptr, segment, r.list, r.count, pieces, static_cast<int64_t>(c.columns), entry, held,
                         weight, r.in_strip, xadj_out, coarse.adj, mult_out);
  if (coarse.nnz > 0) {
    const int64_t tiles = (coarse.nnz + kGatherTile - 1) / kGatherTile;
    int32_t *tile_row = nullptr;
    if (int rc = buf.alloc(&tile_row, static_cast<size_t>(tiles) + 1, "tile rows")) return rc;
    hipLaunchKernelGGL(coarse_tiles_kernel, dim3(blocks_for(n_coarse, 256)), dim3(256), 0, nullptr, xadj_out, n_coarse,
                       coarse.nnz, tile_row);
    hipLaunchKernelGGL(copy_merged_kernel<WT>, dim3(blocks_for(coarse.nnz, kGatherTile)), dim3(256), 0, nullptr, segment,
                       bitmap_from(c.columns), radix_merged ? radix_above(c.columns, ways) : INT64_MAX, tile_row,
                       coarse.nnz, entry, pack, weight, xadj_out, coarse.adj, mult_out);
  }
  if (int rc = gosh::check_launch("coarse rows")) return rc;
  GOSH_TRY_HIP(hipDeviceSynchronize(), "coarse CSR");
  return GOSH_OK;
}

template <typename WT, bool WEIGHTED>
int quotient_by_offsets(gosh::DeviceCoarsener *dc, const gosh::DeviceLevel &fine, int64_t n_coarse,
                        gosh::DeviceLevel &coarse, int64_t *xadj_out) {
  return fine.xadj_is64 ? quotient<int64_t, WT, WEIGHTED>(dc, fine, n_coarse, coarse, xadj_out)
                        : quotient<int32_t, WT, WEIGHTED>(dc, fine, n_coarse, coarse, xadj_out);
}

// Sums of multiplicities are kept in 32 bits unless a graph has more entries than those hold.
constexpr int64_t kWideSumsFrom = int64_t{1} << 32;

}  // namespace

namespace gosh {

int device_rebuild(DeviceCoarsener *dc, const DeviceLevel &fine, int64_t n_coarse, DeviceLevel &coarse) {
  if (dc == nullptr || !fine.present() || fine.map == nullptr)
    return fail(GOSH_EINVAL, "device level or its map is missing");
  device_level_free(coarse);
  coarse.device = fine.device;
  coarse.n = n_coarse;
  coarse.weight = fine.weight;
  coarse.xadj_is64 = 1;
  const bool weighted = fine.mult != nullptr;
  const int64_t wide_from = seam(kSeamWideSums) ? seam(kSeamWideSums) : kWideSumsFrom;
  const bool wide = weighted ? fine.mult_is64 : fine.weight >= wide_from;
  int64_t *xadj_out = nullptr;
  if (int rc = persistent(&xadj_out, static_cast<size_t>(n_coarse) + 1, "coarse offsets")) return rc;
  coarse.xadj = xadj_out;
  if (fine.nnz == 0) {
    coarse.nnz = 0;
    GOSH_TRY_HIP(hipMemset(xadj_out, 0, (static_cast<size_t>(n_coarse) + 1) * 8), "clear coarse offsets");
    if (int rc = persistent(&coarse.adj, 0, "coarse adjacency")) return rc;
    coarse.mult_is64 = wide;
    return persistent(reinterpret_cast<uint64_t **>(&coarse.mult), 0, "coarse multiplicities");
  }
  if (!wide)
    return weighted ? quotient_by_offsets<uint32_t, true>(dc, fine, n_coarse, coarse, xadj_out)
                    : quotient_by_offsets<uint32_t, false>(dc, fine, n_coarse, coarse, xadj_out);
  return weighted ? quotient_by_offsets<unsigned long long, true>(dc, fine, n_coarse, coarse, xadj_out)
                  : quotient_by_offsets<unsigned long long, false>(dc, fine, n_coarse, coarse, xadj_out);
}

}  // namespace gosh
