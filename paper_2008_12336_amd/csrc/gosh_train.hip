// Device side of libgosh for graphs that fit the device: sampler, epoch kernel
// (Alg. 3 with the update of Alg. 1), initialisation and projection.  gfx950 only:
// 64-lane wavefronts, coalesced row accesses, cross-lane reductions with DPP.
//
// Work layout of the epoch kernel (the generic kernel lives in gosh_device.h).  A
// "lane group" of LPG lanes (a power of two covering d/4) owns one source vertex, so a
// wavefront carries 64/LPG sources (two at d = 128, eight at d = 32).  The source row
// stays in registers for its 1 + k_neg updates and is written back once; sample rows
// are fetched four at a time before the first dot product so that their HBM latencies
// overlap.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <mutex>

#include "gosh_common.h"
#include "gosh_device.h"

namespace {

using gosh::philox_draw;
using gosh::scale_draw;
using gosh::Float4;

struct SamplerArgs {
  const void *xadj;
  const int32_t *adj;
  int64_t nnz;
  uint32_t n;
  uint32_t key0, key1;
  uint32_t epoch, level;
};

// Number of entries of the row [begin, end) that may be read.  The kernels stay inside
// their operands whatever the graph arrays hold: a row that the offsets place outside adj
// counts as empty, and an entry that names no vertex is no sample.
template <typename OffT>
__device__ __forceinline__ uint32_t row_entries(OffT begin, OffT end, int64_t nnz) {
  const bool inside = begin >= 0 && begin <= end && static_cast<int64_t>(end) <= nnz;
  return inside ? static_cast<uint32_t>(end - begin) : 0u;
}

// Sample j of source src: j = 0 positive (uniform neighbour, -1 if none), j >= 1
// negative (uniform vertex).
template <typename OffT>
__device__ __forceinline__ int32_t draw_sample(const SamplerArgs &a, uint32_t src, uint32_t j) {
  const uint64_t r = philox_draw(src, j, a.epoch, a.level, a.key0, a.key1);
  if (j != 0) return static_cast<int32_t>(scale_draw(r, a.n));
  const OffT *xadj = static_cast<const OffT *>(a.xadj);
  const OffT begin = xadj[src];
  const uint32_t deg = row_entries(begin, xadj[src + 1], a.nnz);
  if (deg == 0) return -1;
  const int32_t neighbour = a.adj[begin + static_cast<OffT>(scale_draw(r, deg))];
  return static_cast<uint32_t>(neighbour) < a.n ? neighbour : -1;
}

template <typename OffT>
__global__ __launch_bounds__(256) void sample_epoch_kernel(SamplerArgs a, int32_t k_neg,
                                                           int32_t *__restrict__ out) {
  const int64_t total = static_cast<int64_t>(a.n) * (k_neg + 1);
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < total; i += gridDim.x * 256LL) {
    const uint32_t src = static_cast<uint32_t>(i / (k_neg + 1));
    const uint32_t j = static_cast<uint32_t>(i % (k_neg + 1));
    out[i] = draw_sample<OffT>(a, src, j);
  }
}

// Work description of one epoch of Alg. 3 for the generic kernel: every vertex is a
// source, sample t is draw t of that source, rows live in one matrix.
template <typename OffT>
struct EpochWork {
  static constexpr bool kLongTurns = false;  // a source takes one round of samples
  SamplerArgs s;
  float *M;
  int32_t d;
  bool rows_at_lines() const { return gosh::rows_at_lines(M, d); }
  __device__ __forceinline__ int64_t count() const { return s.n; }
  __device__ __forceinline__ int32_t source_id(int64_t i) const { return static_cast<int32_t>(i); }
  __device__ __forceinline__ float *source_row(int64_t i) const { return M + i * d; }
  // What sampling needs from memory knowing the source alone: where its neighbour list is.
  struct Pre {
    OffT begin;
    uint32_t deg;
  };
  __device__ __forceinline__ Pre stage1(int64_t i, bool) const {  // i is a valid source also when unwanted
    const OffT *xadj = static_cast<const OffT *>(s.xadj);
    const OffT begin = xadj[i];
    return Pre{begin, row_entries(begin, xadj[i + 1], s.nnz)};
  }
  // Sample t of a source is draw t; the positive reads the neighbour list.  Written
  // without branches around the read: lanes that do not want a positive read the
  // first offset again instead of a neighbour entry.
  // The draw itself is arithmetic only; the kernel skips it where no group of the wavefront wants it.
  __device__ __forceinline__ uint64_t draw(int64_t, int32_t src, int32_t t) const {
    return philox_draw(static_cast<uint32_t>(src), static_cast<uint32_t>(t), s.epoch, s.level, s.key0, s.key1);
  }
  __device__ __forceinline__ int32_t stage2(int64_t, int32_t, int32_t, bool want, bool positive, const Pre &pre,
                                            uint64_t r) const {
    const bool read_adj = want && positive && pre.deg != 0;
    const int32_t *entry = read_adj ? s.adj + (pre.begin + static_cast<OffT>(scale_draw(r, pre.deg)))
                                    : reinterpret_cast<const int32_t *>(s.xadj);
    const int32_t neighbour = *entry;
    const int32_t uniform = static_cast<int32_t>(scale_draw(r, s.n));
    const bool is_vertex = static_cast<uint32_t>(neighbour) < s.n;
    const int32_t id = positive ? (read_adj && is_vertex ? neighbour : -1) : uniform;
    return want ? id : -1;
  }
  __device__ __forceinline__ float *sample_row(int64_t, int32_t v) const {
    return M + static_cast<int64_t>(v) * d;
  }
  __device__ __forceinline__ int32_t source_slot(int64_t i) const { return static_cast<int32_t>(i); }
  __device__ __forceinline__ int32_t sample_slot(int64_t, int32_t v) const { return v; }
};

template <typename OffT>
__global__ __launch_bounds__(256) void mark_hot_kernel(const OffT *__restrict__ xadj, int64_t n,
                                                       int64_t min_degree,
                                                       unsigned long long *__restrict__ bits) {
  // one vertex per lane, one 64-bit word of the bitmap per wavefront
  const int64_t words = (n + 63) / 64;
  const int64_t wave0 = (blockIdx.x * 256LL + threadIdx.x) >> 6;
  const int64_t nwaves = (gridDim.x * 256LL) >> 6;
  const int lane = threadIdx.x & 63;
  for (int64_t w = wave0; w < words; w += nwaves) {
    const int64_t v = w * 64 + lane;
    bool hot = false;
    if (v < n) hot = static_cast<int64_t>(xadj[v + 1]) - static_cast<int64_t>(xadj[v]) >= min_degree;
    const unsigned long long mask = __ballot(hot);
    if (lane == 0) bits[w] = mask;
  }
}

// Counts the positive samples of an epoch by the row they name (see most_draws), and clears the
// counts of the launch before.  Bound by the chain of reads of a draw: 6 us for 67,000 vertices.
template <typename OffT>
__global__ __launch_bounds__(256) void count_positives_kernel(SamplerArgs a, uint32_t *__restrict__ draws,
                                                              uint32_t *__restrict__ stale, int64_t stale_rows) {
  for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < stale_rows; i += gridDim.x * 256LL) stale[i] = 0;
  for (int64_t first = blockIdx.x * 256LL; first < a.n; first += gridDim.x * 256LL) {
    const int64_t src = first + threadIdx.x;
    const int32_t v = src < a.n ? draw_sample<OffT>(a, static_cast<uint32_t>(src), 0) : -1;
    gosh::count_draws(v == src ? -1 : v, draws);
  }
}

// ---------------------------------------------------------------------------------
// The projection below walks a row-major matrix in tiles of whole rows, at most kTileUnits
// 128-bit units: inside a tile a unit's row comes from one 24-bit product instead of a 64-bit
// division per unit, and consecutive lanes still write consecutive addresses whatever d is.
constexpr int kTileUnits = 2048, kTileRows = 256, kTileBlocks = 1 << 16;

// unit / d4 for unit < kTileUnits, magic = ceil(2^20 / d4), since unit * (magic * d4 - 2^20) < kTileUnits * d4 < 2^20.
__device__ __forceinline__ uint32_t row_of(uint32_t unit, uint32_t magic) { return (unit * magic) >> 20; }
uint32_t row_magic(int32_t d4) {
  static_assert(static_cast<int64_t>(kTileUnits) * (GOSH_MAX_DIM / 4) < (1 << 20), "row_of");
  return static_cast<uint32_t>(((1 << 20) + d4 - 1) / d4);
}

struct RowTiles {
  int32_t d4;     // units per row
  int32_t rows;   // rows per tile
  uint32_t magic;
};
RowTiles row_tiles(int32_t d4) { return RowTiles{d4, std::min(kTileRows, kTileUnits / d4), row_magic(d4)}; }

// A Philox round in four instructions instead of the eight the compiler makes of the same
// expressions: both words of a product from one multiply-add, three-way xors.  For the kernel
// below, which is bound by them; the training kernels wait for memory and gain nothing.
__device__ __forceinline__ uint2 mul_wide(uint32_t constant, uint32_t x) {  // {low word, high word}
  uint64_t p;
  asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(p) : "v"(x), "s"(constant) : "vcc");
  return uint2{static_cast<uint32_t>(p), static_cast<uint32_t>(p >> 32)};
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// M points at row `first_row` of the matrix being initialised.
//
// Entry = (24 random bits / 2^24 - 1/2) / d, one fp32 rounding of the exact value.  The random
// bits of a unit come from Philox(row, unit in the row, 0xFFFFFFFF, level); three of the twenty
// products of its rounds depend on the row alone, one on the column alone and one on neither,
// and are taken once per row of a tile and once per column (`by_row`, `by_col`).  The quotient
// k / (d 2^24), k = bits - 2^23, is a product with the rounded reciprocal and one correction,
// which is the rounded quotient (checked for every k and d) without a division.
//
// Bound by the write stream, whose rate depends on how much is being written at a time: a workgroup writes
// TILE units that begin at a multiple of as many, wherever in a row that is, and ends.  A matrix of more than
// kStreamInit bytes, which no cache holds, is written 4 KB to a wavefront, others 16 KB to a workgroup.  Calls one after
// another on one matrix, us, with tiles of whole rows up to 32 KB / 16 KB / 4 KB (both of any rows):
//   d = 128: 260 MB 41.2 / 41.5 / 42.5   300 MB 48 / 50 / 50   400 MB 80 / 75 / 66   1 GB 194 / 183 / 162
//            2.1 GB 382 / 353 / 323 (6.5 TB/s; 6.4 where other matrices were written in between)
//   d = 8:   260 MB 59 / 44 / 45         300 MB 61 / 53 / 53   400 MB 76 / 70 / 70   1 GB 170 / 170 / 168
//            2.1 GB 334 / 337 / 336
// Below, 4 KB lose: 64 MB 12.5 / 14.5 in the kernel, 1 MB the same.  Its arithmetic alone takes 248 us for 2.1 GB.
// The tables of a wavefront take less than 5 KB of LDS, for 32 to fit a CU: 335 us with 5.2 KB.
constexpr int64_t kStreamInit = int64_t{320} << 20;
template <int THREADS, int TILE, int SHORTEST>  // rows of SHORTEST units at least
__global__ __launch_bounds__(THREADS) void init_embedding_kernel(float4 *__restrict__ M, int64_t units_total,
                                                                 int64_t first_row, uint32_t d4, uint32_t magic,
                                                                 uint64_t magic64, float d_scaled, float rcp_scaled,
                                                                 uint32_t key0, uint32_t key1, uint32_t level) {
  using namespace gosh;
  static_assert(TILE + GOSH_MAX_DIM / 4 <= kTileUnits, "row_of");
  __shared__ uint4 by_row[TILE / SHORTEST + 2];
  __shared__ uint2 by_col[GOSH_MAX_DIM / 4];
  // round 0 multiplies the constant third counter word, round 1 (lo_const) uses it
  constexpr uint32_t kWord = 0xFFFFFFFFu;
  const uint32_t hi_const = mul_hi32(kPhiloxMulB, kWord), lo_const = kPhiloxMulB * kWord;
  for (uint32_t c = threadIdx.x; c < d4; c += THREADS) {
    const uint32_t x = hi_const ^ c ^ key0;  // state word 0 after round 0
    by_col[c] = uint2{mul_hi32(kPhiloxMulA, x) ^ (key1 + kPhiloxWeylB), kPhiloxMulA * x};
  }
  const int64_t tiles = (units_total + TILE - 1) / TILE;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const uint64_t u0 = static_cast<uint64_t>(tile) * TILE;
    // u0 / d4: magic64 = ceil(2^64 / d4) is exact for u0 * d4 < 2^64
    const uint64_t row0 = d4 == 1 ? u0 : __umul64hi(u0, magic64);
    const uint32_t c0 = static_cast<uint32_t>(u0 - row0 * d4);
    const uint32_t units = static_cast<uint32_t>(std::min<int64_t>(TILE, units_total - static_cast<int64_t>(u0)));
    const uint32_t rows = row_of(c0 + units - 1, magic) + 1;
    __syncthreads();  // by_col is there; the previous tile's by_row has been used
    for (uint32_t q = threadIdx.x; q < rows; q += THREADS) {
      const uint32_t v = static_cast<uint32_t>(first_row + static_cast<int64_t>(row0) + q);
      const uint32_t lo0 = kPhiloxMulA * v;                                   // state word 3 after round 0
      const uint32_t x2 = mul_hi32(kPhiloxMulA, v) ^ level ^ key1;            // word 2 after round 0
      const uint32_t x0 = mul_hi32(kPhiloxMulB, x2) ^ lo_const ^ (key0 + kPhiloxWeylA);  // word 0 after round 1
      by_row[q] = uint4{lo0, (kPhiloxMulB * x2) ^ (key0 + 2 * kPhiloxWeylA),
                        mul_hi32(kPhiloxMulA, x0) ^ (key1 + 2 * kPhiloxWeylB), kPhiloxMulA * x0};
    }
    __syncthreads();
    float4 *const out = M + u0;
    for (uint32_t i = threadIdx.x; i < units; i += THREADS) {
      const uint32_t j = c0 + i, row = row_of(j, magic);
      const uint4 r = by_row[row];
      const uint2 c = by_col[j - row * d4];
      const uint32_t x2 = c.x ^ r.x;  // word 2 after round 1
      const uint2 b2 = mul_wide(kPhiloxMulB, x2);
      uint32_t w[4] = {b2.y ^ r.y, b2.x, r.z ^ c.y, r.w};  // after round 2
#pragma unroll
      for (uint32_t round = 3; round < 10; ++round) {
        const uint2 a = mul_wide(kPhiloxMulA, w[0]), b = mul_wide(kPhiloxMulB, w[2]);
        w[0] = xor3(b.y, w[1], key0 + round * kPhiloxWeylA);
        w[1] = b.x;
        w[2] = xor3(a.y, w[3], key1 + round * kPhiloxWeylB);
        w[3] = a.x;
      }
      float o[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float k = static_cast<float>(static_cast<int32_t>(w[q] >> 8) - (1 << 23));
        const float quotient = k * rcp_scaled;
        o[q] = fmaf(fmaf(-quotient, d_scaled, k), rcp_scaled, quotient);
      }
      out[i] = float4{o[0], o[1], o[2], o[3]};
    }
  }
}

// A map entry that names no coarse vertex gives a row of zeros.  Four units of a thread are
// requested together (map entries, then rows).  Bound by the row gather beside the write stream:
// 0.6 M rows onto 4.2 M at d = 128 take 665 us, 6.4 TB/s of rows.  The stores to a matrix that the memory-side
// cache does not hold are non-temporal (STREAM): the check of the matrix that follows a projection runs into
// fewer write-backs.  A smaller one stays there for the epochs that follow.  Projection and check / projection
// and epoch at d = 128, us, streamed and plain: 64 MB 59, 57 / 205, 157;  96 MB 75, 72 / 297, 225;  128 MB 89, 91 /
// 433, 435;  224 MB 134, 136 / 553, 550;  400 MB 207, 216 / 846, 865.  (The projection by itself gains nothing:
// 64 MB 22.3 streamed, 23.1 plain; 120 MB 39.3, 40.3.)
constexpr int64_t kStreamBytes = int64_t{128} << 20;
template <bool STREAM>
__global__ __launch_bounds__(256) void project_kernel(const Float4 *__restrict__ coarse,
                                                      const int32_t *__restrict__ map,
                                                      Float4 *__restrict__ fine, int64_t n_fine,
                                                      RowTiles t, uint32_t n_coarse) {
  constexpr int kUnits = 4;
  const int64_t tiles = (n_fine + t.rows - 1) / t.rows;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t lo = tile * t.rows;
    const uint32_t units = static_cast<uint32_t>(std::min<int64_t>(t.rows, n_fine - lo)) * t.d4;
    const int32_t *const map_rows = map + lo;
    Float4 *const out = fine + lo * t.d4;
    for (uint32_t i0 = threadIdx.x; i0 < units; i0 += 256 * kUnits) {
      uint32_t row[kUnits], c[kUnits];
      Float4 x[kUnits];
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        row[q] = row_of(std::min(i0 + q * 256, units - 1), t.magic);
        c[q] = static_cast<uint32_t>(map_rows[row[q]]);
      }
#pragma unroll
      for (int q = 0; q < kUnits; ++q) {
        const uint32_t column = std::min(i0 + q * 256, units - 1) - row[q] * t.d4;
        x[q] = coarse[static_cast<int64_t>(c[q] < n_coarse ? c[q] : 0) * t.d4 + column];
      }
#pragma unroll
      for (int q = 0; q < kUnits; ++q)
        if (i0 + q * 256 < units) {
          const Float4 y = c[q] < n_coarse ? x[q] : Float4{0.f, 0.f, 0.f, 0.f};
          if constexpr (STREAM) __builtin_nontemporal_store(y, out + i0 + q * 256);
          else out[i0 + q * 256] = y;
        }
    }
  }
}

// Row probe: the row traffic of the training kernels without their arithmetic.  A lane group
// of `lpg` lanes (a power of two covering d/4, at most 64) moves one row with 128-bit
// accesses, so a wavefront carries 64/lpg rows at a time, like the training kernels.
//   kProbeReadWrite  a random row is read and written back with `nothing` (zero) added
//   kProbeRead       a random row is read (a store that never happens keeps the loads alive)
//   kProbeWrite      a random row is overwritten with `nothing`
//   kProbeEpochMix   what one source of an epoch with three negatives moves: row i (sources
//                    are consecutive) and four random rows are read, all five requested
//                    before the first is used, then written back with `nothing` added
// Draw q of access i is Philox(counter = (i_lo, i_hi, 0xFFFFFFFE, q), key = seed).
enum ProbeMode : int32_t { kProbeReadWrite = 0, kProbeRead = 1, kProbeWrite = 2, kProbeEpochMix = 3 };

template <int MODE>
__global__ __launch_bounds__(256) void row_probe_kernel(float4 *__restrict__ M, uint64_t n, int32_t d4,
                                                        int32_t lpg, uint64_t accesses, uint32_t key0,
                                                        uint32_t key1, float nothing) {
  constexpr int kRows = MODE == kProbeEpochMix ? 5 : 1;
  const int lane = threadIdx.x & 63, gl = lane & (lpg - 1), gpw = 64 / lpg;
  const uint64_t wave = (blockIdx.x * 256ull + threadIdx.x) >> 6, waves = (gridDim.x * 256ull) >> 6;
  float sink = 0.f;
  for (uint64_t base = wave * gpw; base < accesses; base += waves * gpw) {
    const uint64_t i = base + lane / lpg;
    if (i >= accesses) continue;
    uint64_t row[kRows];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const uint64_t draw = philox_draw(static_cast<uint32_t>(i), static_cast<uint32_t>(i >> 32), 0xFFFFFFFEu,
                                        static_cast<uint32_t>(q), key0, key1);
      row[q] = (MODE == kProbeEpochMix && q == 0) ? i % n : scale_draw(draw, static_cast<uint32_t>(n));
    }
    float4 v[kRows][2];
#pragma unroll
    for (int q = 0; q < kRows; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = gl + u * lpg;
        v[q][u] = float4{0.f, 0.f, 0.f, 0.f};
        if (MODE != kProbeWrite && c < d4) v[q][u] = M[row[q] * d4 + c];
      }
#pragma unroll
    for (int q = 0; q < kRows; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = gl + u * lpg;
        if (MODE == kProbeRead) {
          sink += v[q][u].x;
        } else if (c < d4) {
          float4 x = v[q][u];
          x.x += nothing;
          M[row[q] * d4 + c] = x;
        }
      }
  }
  if (MODE == kProbeRead && sink == 1.2345e-30f) M[0].x = sink;  // practically never: keeps the loads
}

// Largest finite |x| and the number of non-finite entries of `total4` float4s, accumulated
// into *out (which the caller has cleared).  The bits of a non-negative finite float order
// like the float, so the maximum is taken on them.
// Bound by the read stream.  All workgroups update the same two words and such atomics take
// about 6 ns each one after another, so there are few workgroups, each reduces its own entries
// first, and it adds its maximum only if that is above what it reads there.  The tiles are
// taken from the end of the matrix: what was written last is still in the memory-side cache.
// The loads are non-temporal (2.1 GB: 364 -> 325 us).  2.1 GB took 554 us with one atomic per
// wavefront of 8,192 workgroups.  A workgroup takes four tiles where that leaves 256 of them, and more in large
// matrices: beyond two on a CU the atomics of all, which come at once, cost more than the further loads in flight
// bring.  us of a whole gosh_matrix_check of matrices read before, with 2,048 workgroups / a quarter of the tiles, up to
// 2,048 / the same up to 512: 64 MB 60 / 40 / 40, 128 MB 65 / 54 / 48, 200 MB 64 / 68 / 57, 256 MB 75 / 75 / 65,
// 400 MB 90 / 91 / 86, 2 GB 325 / 325 / 321.
constexpr int kCheckTile = 2048;  // float4s per workgroup and turn
constexpr int kCheckBlocks = 512;
__global__ __launch_bounds__(256) void matrix_check_kernel(const Float4 *__restrict__ M, int64_t total4,
                                                           gosh::CheckResult *__restrict__ out) {
  constexpr int kUnits = kCheckTile / 256;
  gosh::EntryCheck check;
  const int64_t tiles = (total4 + kCheckTile - 1) / kCheckTile;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t first = (tiles - 1 - t) * kCheckTile + threadIdx.x;
    if (first - threadIdx.x + kCheckTile <= total4) {
      Float4 x[kUnits];
#pragma unroll
      for (int q = 0; q < kUnits; ++q) x[q] = __builtin_nontemporal_load(M + first + q * 256);
#pragma unroll
      for (int q = 0; q < kUnits; ++q) check.look(x[q]);
    } else {
      for (int64_t i = first; i < total4; i += 256) check.look(__builtin_nontemporal_load(M + i));
    }
  }
  check.reduce_wave();
  __shared__ uint32_t tops[4], bads[4];
  if ((threadIdx.x & 63) == 0) {
    tops[threadIdx.x >> 6] = check.top;
    bads[threadIdx.x >> 6] = check.bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    check.top = max(max(tops[0], tops[1]), max(tops[2], tops[3]));
    check.bad = bads[0] + bads[1] + bads[2] + bads[3];
    check.add_to(out);
  }
}

__global__ void clear_checks_kernel(gosh::CheckResult *out, int count) {
  for (int i = threadIdx.x; i < count; i += 64) out[i] = gosh::CheckResult{0, 0, 0};
}

int grid_for(int64_t items, int per_block, int max_blocks) {
  int64_t b = (items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > max_blocks) b = max_blocks;
  return static_cast<int>(b);
}

SamplerArgs sampler_args(const gosh_csr *g, uint64_t seed, uint32_t epoch, uint32_t level) {
  SamplerArgs s;
  s.xadj = g->xadj;
  s.adj = g->adj;
  s.nnz = g->nnz;
  s.n = static_cast<uint32_t>(g->n);
  s.key0 = static_cast<uint32_t>(seed);
  s.key1 = static_cast<uint32_t>(seed >> 32);
  s.epoch = epoch;
  s.level = level;
  return s;
}

// Whether a call on this stream is being recorded.  Such calls, and gosh_train_epoch_static, take
// no locks: the words may be replaced by larger ones later, which a recorded launch would not see.
bool capturing(hipStream_t st) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// bits_override: the hot-row bitmap to use instead of the library's grown-on-demand scratch
// (at least (n + 63) / 64 * 8 bytes), or null.
template <typename OffT>
int launch_epoch(const gosh_csr *g, float *M, int32_t d, int32_t k_neg, float lr, uint64_t seed,
                 uint32_t epoch, uint32_t level, uint32_t flags, void *bits_override, hipStream_t st) {
  const bool seq = (flags & GOSH_FLAG_SEQUENTIAL) != 0;
  // the write paths of the concurrent kernel: in concurrent mode, and in the sequential walk
  // that is asked to use them
  const bool concurrent_paths = !seq || (flags & GOSH_FLAG_CONCURRENT_LAYOUT) != 0;
  const gosh_tuning tune = gosh::tuning();
  const int64_t n = g->n;
  EpochWork<OffT> w;
  w.s = sampler_args(g, seed, epoch, level);
  w.M = M;
  w.d = d;
  gosh::SgdArgs a{};
  a.d = d;
  a.k_neg = k_neg;
  a.samples = k_neg + 1;
  a.lr = lr;
  a.hot = gosh::HotSet{nullptr, gosh::kHotNone};
  gosh::LockSet lock;
  const int64_t max_waves = tune.max_waves;
  if (concurrent_paths) {
    // Sources in flight C, and the hot-row rule.  A vertex is hot if its expected
    // positive hits per epoch, deg/avg_deg, give more than eps = 1/64 concurrent holders:
    // deg * C / nnz > eps.  On graphs so small that even the k+1 uniform touches of
    // every row overlap ((k+1)*C/n > 1/4, i.e. fewer than 16 rounds at k = 3) all rows
    // are hot.  Both constants come from link-prediction AUCROC against the sequential
    // reference on R-MAT graphs of 2^12..2^20 vertices: with them the concurrent kernel
    // stays within 0.001..0.005 of the reference, without them it drops by up to 0.4.
    const int gpw = gosh::SgdLauncher<EpochWork<OffT>>::groups_per_wave(d);
    int64_t waves = std::min<int64_t>((n + gpw - 1) / gpw, max_waves);
    const int64_t in_flight = std::min<int64_t>(waves, gosh::resident_waves()) * gpw;
    const int64_t capacity = std::min<int64_t>(max_waves, gosh::resident_waves()) * gpw;
    int mode = gosh::kHotBitmap;
    // Locks stand in for the adds of an all-hot launch and for nothing else: with more vertices the
    // degree rule leaves most writes of a skewed graph to plain stores, which are cheaper (k = 3,
    // d = 128, us, stores and adds by degree against locks: R-MAT of 300,000 vertices 246 / 307, of
    // 500,000 445 / 626; power law 437 / 309 and 507 / 655; only uniform graphs gain throughout).
    if (tune.hot_min_degree == 0 && (k_neg + 1) * in_flight * tune.hot_all_inv_eps > n)
      mode = bits_override == nullptr && tune.plain_rows == 0 && gosh::worth_locking(n, k_neg + 1, capacity, d) && !capturing(st)
                 ? gosh::kHotLocked
                 : gosh::kHotAll;
    if (flags & GOSH_FLAG_PLAIN_STORES) mode = gosh::kHotNone;
    if (flags & GOSH_FLAG_ATOMIC_ADDS) mode = gosh::kHotAll;
    if (mode == gosh::kHotLocked) {
      gosh::LockWords words{};
      const int rc = gosh::lock_scratch(n, st, &words);
      if (rc == GOSH_ENOMEM) {
        mode = gosh::kHotAll;  // which needs no memory
      } else {
        if (rc != GOSH_OK) return rc;
        hipLaunchKernelGGL(count_positives_kernel<OffT>, dim3(grid_for(n, 256, 1 << 16)), dim3(256), 0, st, w.s,
                           words.draws, words.stale, words.stale_rows);
        if (int rc2 = gosh::check_launch("count_positives_kernel")) return rc2;
        lock = gosh::LockSet{words.locks, words.draws, gosh::most_draws(n, k_neg + 2, in_flight), gosh::lock_tries()};
      }
    }
    if (mode == gosh::kHotBitmap) {
      const int64_t min_degree =
          tune.hot_min_degree > 0 ? tune.hot_min_degree : g->nnz / (tune.hot_inv_eps * in_flight) + 1;
      void *bits = bits_override;
      if (bits == nullptr)
        if (int rc = gosh::hot_scratch(static_cast<size_t>((n + 63) / 64) * 8, &bits)) return rc;
      const int blocks = static_cast<int>(std::min<int64_t>(((n + 63) / 64 + 3) / 4, 1 << 16));
      hipLaunchKernelGGL(mark_hot_kernel<OffT>, dim3(blocks), dim3(256), 0, st,
                         static_cast<const OffT *>(g->xadj), n, min_degree,
                         static_cast<unsigned long long *>(bits));
      if (int rc = gosh::check_launch("mark_hot_kernel")) return rc;
      a.hot.bits = static_cast<const uint32_t *>(bits);
    }
    a.hot.mode = mode;
  }
  gosh::seam(gosh::kSeamHotMode) = a.hot.mode;
  if (a.hot.bits == nullptr) {
    // the kernel reads word 0 of the bitmap unconditionally (one with locks does not, but a call under
    // capture after it will, and cannot allocate)
    void *bits = bits_override;
    if (bits == nullptr)
      if (int rc = gosh::hot_scratch(8, &bits)) return rc;
    a.hot.bits = static_cast<const uint32_t *>(bits);
  }
  const bool plain_rows = tune.plain_rows != 0 || (seq && !concurrent_paths);
  gosh::SgdLauncher<EpochWork<OffT>>::launch(w, a, lock, n, seq, plain_rows, max_waves, st);
  return gosh::check_launch("sgd_kernel (epoch)");
}

// Hot-row bitmap of gosh_train_epoch_static: one bit per vertex, in the code object itself.
// Host code must not use this name as an address (on the host it is a stand-in, not device
// memory): static_bitmap() asks the runtime for the array's address on the current device.
static __device__ __align__(256) unsigned long long scratch[GOSH_STATIC_MAX_N / 64];

int static_bitmap(void **out) {
  constexpr int kMaxDevices = 64;
  static void *address[kMaxDevices] = {};  // every device holds its own copy of the array
  static std::mutex mutex;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return gosh::fail(GOSH_EHIP, "cannot identify the current device");
  std::lock_guard<std::mutex> lock(mutex);
  if (address[dev] == nullptr) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return gosh::fail(GOSH_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    }
    address[dev] = p;
  }
  *out = address[dev];
  return GOSH_OK;
}

int check_epoch_args(const gosh_csr *g_dev, float *M_dev, int32_t d, int32_t k_neg, float lr_epoch,
                     uint32_t flags) {
  if (int rc = gosh::check_csr(g_dev)) return rc;
  if (int rc = gosh::check_matrix(M_dev, d, "M")) return rc;
  if (k_neg < 0 || k_neg > GOSH_MAX_NEG)
    return gosh::fail(GOSH_EINVAL, "k_neg = %d: must be in [0, %d]", k_neg, GOSH_MAX_NEG);
  if (flags & ~(GOSH_FLAG_SEQUENTIAL | GOSH_FLAG_PLAIN_STORES | GOSH_FLAG_ATOMIC_ADDS | GOSH_FLAG_CONCURRENT_LAYOUT))
    return gosh::fail(GOSH_EINVAL, "unknown flags 0x%x", flags);
  if ((flags & GOSH_FLAG_PLAIN_STORES) && (flags & GOSH_FLAG_ATOMIC_ADDS))
    return gosh::fail(GOSH_EINVAL, "flags ask for plain stores and atomic adds at once");
  if (!(lr_epoch == lr_epoch)) return gosh::fail(GOSH_EINVAL, "lr is NaN");
  if (int rc = gosh::check_device_csr(g_dev)) return rc;
  return gosh::check_device_span(M_dev, static_cast<size_t>(g_dev->n) * d * 4, "M");
}

}  // namespace

namespace gosh {

int matrix_check_clear(CheckResult *results_dev, hipStream_t st, int count) {
  hipLaunchKernelGGL(clear_checks_kernel, dim3(1), dim3(64), 0, st, results_dev, count);
  return check_launch("clear_checks_kernel");
}

int matrix_check_add(const float *rows_dev, int64_t floats, CheckResult *result_dev, hipStream_t st) {
  const int64_t total4 = floats / 4;
  if (total4 <= 0) return GOSH_OK;
  const int64_t tiles = (total4 + kCheckTile - 1) / kCheckTile;
  const int64_t blocks = std::min<int64_t>(std::max(std::min<int64_t>(tiles, 256), tiles / 4), kCheckBlocks);
  hipLaunchKernelGGL(matrix_check_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st,
                     reinterpret_cast<const Float4 *>(rows_dev), total4, result_dev);
  return check_launch("matrix_check_kernel");
}

int matrix_check_read(const CheckResult *result_dev, float *max_abs, int64_t *nonfinite, hipStream_t st) {
  CheckResult host{};
  GOSH_TRY_HIP(hipMemcpyAsync(&host, result_dev, sizeof(host), hipMemcpyDeviceToHost, st), "read matrix check");
  GOSH_TRY_HIP(hipStreamSynchronize(st), "matrix check");
  if (max_abs) {
    float f;
    static_assert(sizeof(f) == sizeof(host.max_bits), "fp32");
    __builtin_memcpy(&f, &host.max_bits, 4);
    *max_abs = f;
  }
  if (nonfinite) *nonfinite = static_cast<int64_t>(host.nonfinite);
  return GOSH_OK;
}

int row_probe(float *M_dev, int64_t n, int32_t d, int64_t accesses, uint64_t seed, int32_t mode, hipStream_t st) {
  if (accesses <= 0) return GOSH_OK;
  const int32_t d4 = d / 4;
  int32_t lpg = 1;
  while (lpg < d4 && lpg < 64) lpg *= 2;
  const int64_t per_block = 4 * (64 / lpg);  // four wavefronts per block
  const int blocks = grid_for(accesses, static_cast<int>(per_block), 1 << 18);
  float4 *M4 = reinterpret_cast<float4 *>(M_dev);
  const uint64_t un = static_cast<uint64_t>(n), ua = static_cast<uint64_t>(accesses);
  const uint32_t k0 = static_cast<uint32_t>(seed), k1 = static_cast<uint32_t>(seed >> 32);
  switch (mode) {
    case kProbeReadWrite:
      hipLaunchKernelGGL(row_probe_kernel<kProbeReadWrite>, dim3(blocks), dim3(256), 0, st, M4, un, d4, lpg, ua, k0, k1, 0.0f);
      break;
    case kProbeRead:
      hipLaunchKernelGGL(row_probe_kernel<kProbeRead>, dim3(blocks), dim3(256), 0, st, M4, un, d4, lpg, ua, k0, k1, 0.0f);
      break;
    case kProbeWrite:
      hipLaunchKernelGGL(row_probe_kernel<kProbeWrite>, dim3(blocks), dim3(256), 0, st, M4, un, d4, lpg, ua, k0, k1, 0.0f);
      break;
    case kProbeEpochMix:
      hipLaunchKernelGGL(row_probe_kernel<kProbeEpochMix>, dim3(blocks), dim3(256), 0, st, M4, un, d4, lpg, ua, k0, k1, 0.0f);
      break;
    default:
      return fail(GOSH_EINVAL, "probe mode %d: must be 0 (read-write), 1 (read), 2 (write) or 3 (epoch mix)", mode);
  }
  return check_launch("row_probe_kernel");
}

int init_rows(float *rows_dev, int64_t first_row, int64_t count, int32_t d, uint64_t seed,
              uint32_t level, hipStream_t st) {
  const uint32_t d4 = static_cast<uint32_t>(d / 4);
  const float d_scaled = static_cast<float>(d) * 16777216.0f;  // exact; its reciprocal is rounded once
  const uint64_t magic64 = d4 == 1 ? 0 : ~uint64_t{0} / d4 + 1;
  auto run = [&](auto kernel, int threads, int tile) {
    const int most = (1 << 30) / threads;  // a grid counts its threads in 32 bits
    hipLaunchKernelGGL(kernel, dim3(grid_for(count * d4, tile, most)), dim3(threads), 0, st,
                       reinterpret_cast<float4 *>(rows_dev), count * d4, first_row, d4, row_magic(d / 4), magic64, d_scaled,
                       1.0f / d_scaled, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32), level);
  };
  if (count * d * 4 > kStreamInit && d4 >= 2) run(init_embedding_kernel<64, 256, 2>, 64, 256);
  else run(init_embedding_kernel<256, 1024, 1>, 256, 1024);
  return check_launch("init_embedding_kernel");
}

}  // namespace gosh

extern "C" {

int gosh_init_embedding(float *M_dev, int64_t n, int32_t d, uint64_t seed, uint32_t level,
                        void *hip_stream) {
  if (int rc = gosh::check_matrix(M_dev, d, "M")) return rc;
  if (n < 1 || n >= 2147483647LL) return gosh::fail(GOSH_EINVAL, "n = %lld out of range", (long long)n);
  if (int rc = gosh::check_device_span(M_dev, static_cast<size_t>(n) * d * 4, "M")) return rc;
  return gosh::init_rows(M_dev, 0, n, d, seed, level, gosh::as_stream(hip_stream));
}

int gosh_sample_epoch(const gosh_csr *g_dev, int32_t k_neg, uint64_t seed, uint32_t epoch,
                      uint32_t level, int32_t *out_dev, void *hip_stream) {
  if (int rc = gosh::check_csr(g_dev)) return rc;
  if (k_neg < 0 || k_neg > GOSH_MAX_NEG)
    return gosh::fail(GOSH_EINVAL, "k_neg = %d: must be in [0, %d]", k_neg, GOSH_MAX_NEG);
  if (out_dev == nullptr) return gosh::fail(GOSH_EINVAL, "out is null");
  if (int rc = gosh::check_device_csr(g_dev)) return rc;
  if (int rc = gosh::check_device_span(out_dev, static_cast<size_t>(g_dev->n) * (k_neg + 1) * 4, "out")) return rc;
  const SamplerArgs s = sampler_args(g_dev, seed, epoch, level);
  const int blocks = grid_for(g_dev->n * (k_neg + 1), 256, 1 << 16);
  if (g_dev->xadj_is64)
    hipLaunchKernelGGL(sample_epoch_kernel<int64_t>, dim3(blocks), dim3(256), 0,
                       gosh::as_stream(hip_stream), s, k_neg, out_dev);
  else
    hipLaunchKernelGGL(sample_epoch_kernel<int32_t>, dim3(blocks), dim3(256), 0,
                       gosh::as_stream(hip_stream), s, k_neg, out_dev);
  return gosh::check_launch("sample_epoch_kernel");
}

int gosh_train_epoch(const gosh_csr *g_dev, float *M_dev, int32_t d, int32_t k_neg, float lr_epoch,
                     uint64_t seed, uint32_t epoch, uint32_t level, uint32_t flags,
                     void *hip_stream) {
  if (int rc = check_epoch_args(g_dev, M_dev, d, k_neg, lr_epoch, flags)) return rc;
  hipStream_t st = gosh::as_stream(hip_stream);
  if (g_dev->xadj_is64)
    return launch_epoch<int64_t>(g_dev, M_dev, d, k_neg, lr_epoch, seed, epoch, level, flags, nullptr, st);
  return launch_epoch<int32_t>(g_dev, M_dev, d, k_neg, lr_epoch, seed, epoch, level, flags, nullptr, st);
}

int gosh_train_epoch_static(const gosh_csr *g_dev, float *M_dev, int32_t d, int32_t k_neg, float lr_epoch,
                            uint64_t seed, uint32_t epoch, uint32_t level, uint32_t flags,
                            void *hip_stream) {
  if (g_dev != nullptr && g_dev->n > GOSH_STATIC_MAX_N)
    return gosh::fail(GOSH_EINVAL, "n = %lld: gosh_train_epoch_static takes at most %lld vertices (use gosh_train_epoch)",
                      (long long)g_dev->n, (long long)GOSH_STATIC_MAX_N);
  if (int rc = check_epoch_args(g_dev, M_dev, d, k_neg, lr_epoch, flags)) return rc;
  void *bits = nullptr;
  if (int rc = static_bitmap(&bits)) return rc;
  hipStream_t st = gosh::as_stream(hip_stream);
  if (g_dev->xadj_is64)
    return launch_epoch<int64_t>(g_dev, M_dev, d, k_neg, lr_epoch, seed, epoch, level, flags, bits, st);
  return launch_epoch<int32_t>(g_dev, M_dev, d, k_neg, lr_epoch, seed, epoch, level, flags, bits, st);
}

int gosh_matrix_check(const float *M_dev, int64_t n, int32_t d, float *max_abs, int64_t *nonfinite,
                      void *hip_stream) {
  if (int rc = gosh::check_matrix(M_dev, d, "M")) return rc;
  if (n < 1 || n >= 2147483647LL) return gosh::fail(GOSH_EINVAL, "n = %lld out of range", (long long)n);
  if (int rc = gosh::check_device_span(M_dev, static_cast<size_t>(n) * d * 4, "M")) return rc;
  hipStream_t st = gosh::as_stream(hip_stream);
  gosh::CheckResult *result = nullptr;
  if (int rc = gosh::check_scratch(&result)) return rc;
  if (int rc = gosh::matrix_check_clear(result, st)) return rc;
  if (int rc = gosh::matrix_check_add(M_dev, n * d, result, st)) return rc;
  return gosh::matrix_check_read(result, max_abs, nonfinite, st);
}

int gosh_row_probe(float *M_dev, int64_t n, int32_t d, int64_t accesses, uint64_t seed, int32_t mode,
                   void *hip_stream) {
  if (int rc = gosh::check_matrix(M_dev, d, "M")) return rc;
  if (n < 1 || n >= 2147483647LL) return gosh::fail(GOSH_EINVAL, "n = %lld out of range", (long long)n);
  if (accesses < 0) return gosh::fail(GOSH_EINVAL, "accesses = %lld is negative", (long long)accesses);
  if (mode < 0 || mode > 3)
    return gosh::fail(GOSH_EINVAL, "probe mode %d: must be 0 (read-write), 1 (read), 2 (write) or 3 (epoch mix)", mode);
  if (int rc = gosh::check_device_span(M_dev, static_cast<size_t>(n) * d * 4, "M")) return rc;
  return gosh::row_probe(M_dev, n, d, accesses, seed, mode, gosh::as_stream(hip_stream));
}

int gosh_project(const float *M_coarse_dev, int64_t n_coarse, const int32_t *map_dev, int64_t n_fine,
                 int32_t d, float *M_fine_dev, void *hip_stream) {
  if (int rc = gosh::check_matrix(M_coarse_dev, d, "M_coarse")) return rc;
  if (int rc = gosh::check_matrix(M_fine_dev, d, "M_fine")) return rc;
  if (map_dev == nullptr) return gosh::fail(GOSH_EINVAL, "map is null");
  if (n_coarse < 1 || n_fine < 1)
    return gosh::fail(GOSH_EINVAL, "need n_coarse (%lld) >= 1 and n_fine (%lld) >= 1",
                      (long long)n_coarse, (long long)n_fine);
  if (int rc = gosh::check_device_span(M_coarse_dev, static_cast<size_t>(n_coarse) * d * 4, "M_coarse")) return rc;
  if (int rc = gosh::check_device_span(M_fine_dev, static_cast<size_t>(n_fine) * d * 4, "M_fine")) return rc;
  if (int rc = gosh::check_device_span(map_dev, static_cast<size_t>(n_fine) * 4, "map")) return rc;
  const RowTiles t = row_tiles(d / 4);
  const bool stream = n_fine * d * 4 > kStreamBytes;
  hipLaunchKernelGGL(stream ? project_kernel<true> : project_kernel<false>,
                     dim3(grid_for(n_fine, t.rows, kTileBlocks)), dim3(256), 0,
                     gosh::as_stream(hip_stream), reinterpret_cast<const Float4 *>(M_coarse_dev),
                     map_dev, reinterpret_cast<Float4 *>(M_fine_dev), n_fine, t,
                     static_cast<uint32_t>(std::min<int64_t>(n_coarse, 2147483647LL)));
  return gosh::check_launch("project_kernel");
}

}  // extern "C"
