// Device-side building blocks of libgosh shared by the epoch kernel (Alg. 3) and the
// part-pair kernel (Alg. 5): the counter-based generator, the cross-lane reduction,
// the row access policies and the generic lock-free SGD kernel.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

namespace gosh {

// ---------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  philox_draw returns the first two output words as
// one 64-bit draw.  Usable on host and device.
// ---------------------------------------------------------------------------------
__host__ __device__ __forceinline__ uint32_t mul_hi32(uint32_t a, uint32_t b) {
  return static_cast<uint32_t>((static_cast<uint64_t>(a) * b) >> 32);
}

constexpr uint32_t kPhiloxMulA = 0xD2511F53u, kPhiloxMulB = 0xCD9E8D57u;
constexpr uint32_t kPhiloxWeylA = 0x9E3779B9u, kPhiloxWeylB = 0xBB67AE85u;

__host__ __device__ __forceinline__ uint64_t philox_draw(uint32_t c0, uint32_t c1, uint32_t c2,
                                                         uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hiA = mul_hi32(kPhiloxMulA, c0), loA = kPhiloxMulA * c0;
    const uint32_t hiB = mul_hi32(kPhiloxMulB, c2), loB = kPhiloxMulB * c2;
    c0 = hiB ^ c1 ^ k0;
    c1 = loB;
    c2 = hiA ^ c3 ^ k1;
    c3 = loA;
    k0 += kPhiloxWeylA;
    k1 += kPhiloxWeylB;
  }
  return static_cast<uint64_t>(c0) | (static_cast<uint64_t>(c1) << 32);
}

// floor(r * bound / 2^64) for bound < 2^32.
__host__ __device__ __forceinline__ uint32_t scale_draw(uint64_t r, uint32_t bound) {
  const uint32_t lo = static_cast<uint32_t>(r), hi = static_cast<uint32_t>(r >> 32);
  const uint64_t t = static_cast<uint64_t>(hi) * bound + mul_hi32(lo, bound);
  return static_cast<uint32_t>(t >> 32);
}

// ---------------------------------------------------------------------------------
// Sum over the LPG lanes of a group; every lane of the group gets the total.
// Steps inside a 16-lane row use DPP (no LDS traffic); 32 and 64 lanes finish with
// swizzle / bpermute.
// ---------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

template <int LPG>
__device__ __forceinline__ float group_sum(float x) {
  if (LPG >= 2) x += dpp_move<0xB1>(x);    // quad_perm [1,0,3,2]
  if (LPG >= 4) x += dpp_move<0x4E>(x);    // quad_perm [2,3,0,1]
  if (LPG >= 8) x += dpp_move<0x141>(x);   // row_half_mirror (quads already uniform)
  if (LPG >= 16) x += dpp_move<0x140>(x);  // row_mirror (halves already uniform)
  if (LPG >= 32) x += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x401F));  // lane ^ 16
  if (LPG >= 64) x += __shfl_xor(x, 32, 64);
  return x;
}

// ---------------------------------------------------------------------------------
// Row access policies.  A row is moved in "units" of F floats per lane.
//
// The chip's eight XCDs each have their own L2, and plain stores sit in the writer's
// L2 until they are evicted or the kernel ends: with plain accesses a row updated on
// one XCD is read stale on the others and the last write-back wins.  Lock-free SGD
// needs the rows to be coherent across the whole device, so the concurrent kernels
// move rows with agent-scope (device-scope) accesses, which are served behind the
// per-XCD L2s.  Every sample row is touched once per turn, so no L2 reuse is lost.
//   RowAgent32: 32-bit relaxed atomic loads and stores at agent scope, lanes interleaved
//     over the row (lane g owns floats g, g+LPG, ...) so that every access instruction
//     of a group covers one whole 128-byte line.  Measured on a 2^24-vertex graph this
//     is as fast as wider per-lane accesses, and it makes the atomic adds used for hot
//     rows (below) dense: one line per instruction instead of half-filled lines, which
//     the memory-side atomic units process at half the rate.
//   RowPlain128: ordinary 128-bit accesses (coherent only inside one XCD); used by the
//     sequential-order mode, which runs on a single wavefront.
// ---------------------------------------------------------------------------------
template <int F>
struct Unit {
  float v[F];
};
// Four floats live in one 128-bit register tuple: an explicit 128-bit load (RowAgent128)
// then delivers straight into the unit, with no instruction in between that could touch
// registers whose data has not arrived yet.
typedef float Float4 __attribute__((ext_vector_type(4)));
template <>
struct Unit<4> {
  Float4 v;
};

__device__ __forceinline__ void atomic_step(float *p, float x) {
  // Built with -munsafe-fp-atomics: the matrix is ordinary coarse-grained device
  // memory, where the hardware fp32 add is available.
  __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Policies whose loads the compiler issues itself need no explicit wait.
struct TrackedLoads {
  static constexpr bool kWaveAtomics = false;  // a hot row is added to by the lanes that own it
  static constexpr bool kAligned = false;      // lane g's first column is g, wherever the row starts
  static __device__ __forceinline__ void wait_all() {}
  template <int F>
  static __device__ __forceinline__ void settle(Unit<F> &) {}
};

struct RowPlain128 : TrackedLoads {
  static constexpr int F = 4;
  static __device__ __forceinline__ Unit<4> load(const float *p) {
    return Unit<4>{*reinterpret_cast<const Float4 *>(p)};
  }
  static __device__ __forceinline__ void store(float *p, const Unit<4> &u) {
    *reinterpret_cast<Float4 *>(p) = u.v;
  }
};

// RowAgent128: 128-bit accesses at agent scope, four consecutive floats per lane, for
// d <= 64, where a row is at most two lines: rows that short move 12-23 % faster in 128-bit
// pieces on d/4 lanes than in 64-bit pieces on d/2 lanes (5.9 against 4.8 TB/s at d = 32),
// plain or device-scope alike.  The compiler offers device-scope accesses only as atomics of
// at most 64 bits, so the two instructions are written out (global_load_dwordx4 / global_store_dwordx4 with the sc1
// bit, which is what an agent-scope access is on this chip).  The compiler does not count
// these loads in its waits: settle() waits for all outstanding memory operations and ties
// every loaded unit to that wait, and must be called for a unit before its first use.
struct RowAgent128 {
  static constexpr int F = 4;
  static constexpr bool kWaveAtomics = true;  // a hot row is added to by the whole wavefront, see add_rows_as_a_wave
  static constexpr bool kAligned = false;
  static __device__ __forceinline__ Unit<4> load(const float *p) {
    Unit<4> u;
    asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(u.v) : "v"(p) : "memory");
    return u;
  }
  static __device__ __forceinline__ void store(float *p, const Unit<4> &u) {
    // A store of more than 64 bits still reads its data registers for two wait states after
    // it issues; the compiler pads its own stores and cannot see into this one.
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(u.v) : "memory");
  }
  static __device__ __forceinline__ void wait_all() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
  static __device__ __forceinline__ void settle(Unit<4> &u) { asm volatile("" : "+v"(u.v)); }
};

struct RowAgent32 : TrackedLoads {
  static constexpr int F = 1;
  static __device__ __forceinline__ Unit<1> load(const float *p) {
    return Unit<1>{{__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)}};
  }
  static __device__ __forceinline__ void store(float *p, const Unit<1> &u) {
    __hip_atomic_store(p, u.v[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// RowAgentLine: RowAgent32 for rows that do not start at line borders (d no multiple of 32, or
// such a matrix).  With lane g at column g every access instruction of such a row straddles one
// line more than it covers, and the memory system charges per instruction and 64-byte block
// touched, for atomic adds above all (20.5 G blocks/s).  Here a lane's columns follow from the
// address of the row: slot g + i * LPG lies that far behind the line border below the row's
// start, and the slots before the start take the columns that are left over at the end.  An
// element of the matrix keeps its lane, but two rows have theirs at different ones, so the source row
// is held in LDS by column while its samples are worked at.
struct RowAgentLine : RowAgent32 {
  static constexpr bool kAligned = true;
};

// ---------------------------------------------------------------------------------
// Hot rows.  A lock-free update is a read-modify-write of a row; when two wavefronts
// hold the same row at once, one of the two writes is lost (Sec. 3.1 of the paper
// accepts such races, and reports that too many of them hurt the embedding).  With
// C sources in flight out of n, a row that is touched h times per epoch has about
// h*C/n concurrent holders.  Rows for which that is not small -- every row of a
// small graph, the high-degree vertices of a large one, which are drawn as positive
// samples in proportion to their degree -- are "hot": their updates are applied as
// atomic adds of the step (M[v] += g*M[src], and M[src] += its accumulated change),
// which cannot be lost.  Cold rows are written back with plain stores, which cost
// half as much on this memory system.
// ---------------------------------------------------------------------------------
//
// Locked rows.  fp32 atomic adds run at 20.5 G 64-byte blocks per second on the whole chip, and
// a launch in which every row is hot is bound by that.  A row can also be written without losing
// an update by taking a lock first: one 32-bit exchange instead of an atomic add per block, then
// the row is read, changed and written back like a cold one (7.0 G rows of 512 bytes per second where
// the memory-side cache holds them, 5.0 G where it does not, read included, against 2.55 G as adds
// alone).  In kHotLocked mode every row is written that way, except hubs, whose holders would queue up:
// their rows take atomic adds, always, so that a row is only ever written one way in a launch (but see
// kMaxTries).
enum HotMode : int32_t { kHotNone = 0, kHotBitmap = 1, kHotAll = 2, kHotLocked = 3 };

struct HotSet {
  const uint32_t *bits;  // one bit per vertex when mode is kHotBitmap (hot); in the other modes still
                         // a readable device word (the kernel reads word 0 blindly)
  int32_t mode;
};

// What a launch in kHotLocked mode needs besides.  A word each per row: a lock, 0 before and after
// the launch, and how often the row is drawn (see most_draws); a hub is a row of which that is above
// `most`.  An argument of its own: the other kernels start a little sooner without it.
struct LockSet {
  uint32_t *locks = nullptr;
  const uint32_t *draws = nullptr;
  uint32_t most = 0;
  int32_t max_tries = 0;  // of a lock
  int32_t waves_per_cu = 0;  // wavefronts of the launch that a CU may hold (0: kLockedWaves alone decides)
};

// Whether a launch in which every row is hot takes locks.  `capacity` sources run at a time (C when
// the device is full), so a launch is sources / capacity rounds.  Adds cost time per block of a
// row, a lock costs about as much as one round trip however long the row is: what it saves grows
// with what the rows in flight have together (131,072 blocks are a full chip at d = 64, 128 and
// 256), and what it costs on top -- the counting, the longer chain of one source -- must spread
// over some rounds and samples.  Rows that start inside a block share lines with their neighbours:
// they count by their columns, and barely pay where half of a lane group is idle.  With few negatives
// many of the rows drawn are positives, of which R-MAT graphs have few, and such launches must be
// larger.  The edge is where a kernel of chunks of four samples broke even, and the tests hold it there
// vertex for vertex; sgd_locked_walk breaks even earlier where rows straddle lines or leave lanes idle, so
// launches of such rows below the edge forgo up to a fifth, and R-MAT graphs with one negative gain
// nothing just above it.  Time with locks over time with adds, power law / R-MAT with m = 10 n, by
// rounds, and the rule's edge:
//   d = 128, k = 9   1.5: 0.65 / 0.71                (1.3)     k = 3   2: 0.70 / 0.79        (1.8)
//            k = 1   3: 0.69 / 0.86                  (2.7)     d = 192, k = 3  4: 0.66 / 0.69  (3.2)
//   d = 80,  k = 3   6: 0.81 / 0.80                  (4.6)     d = 384, k = 9  1: 0.65 / 0.70  (0.8)
//   d = 64,  k = 3   2: 0.77 / 0.96                  (1.8)     k = 1   3: 0.76 / 1.05, 4: 0.75 / 1.03  (3.6)
//   d = 52,  k = 3   1.8: 0.84 / 1.05, 2.5: 0.77 / 0.87  (2.2)  k = 1  3: 0.83 / 1.05, 4: 0.78 / 1.02  (4.4)
//   d = 100, k = 9   2.5: 0.70 / 0.76 (2.3)    k = 3   2.5: 0.80 / 0.91, 3: 0.77 / 0.85      (3.3)
//            k = 1   4: 0.83 / 0.97, 6: 0.78 / 0.87  (6.7)
//   d = 76,  k = 9   3.6: 0.79 / 0.80, 6: 0.72 / 0.72 (4.6)    k = 2   6: 0.89 / 0.89        (8.8)
//   d = 68,  k = 9   4: 0.85 / 0.87, 8: 0.75 / 0.75 (7.4)      k = 3   6: 0.90 / 0.87, 12: 0.82 / 0.82 (10.6)
//   d = 132, k = 9   4: 0.84 / 0.84, 8: 0.75 / 0.76 (7.4)      k = 3   6: 0.88 / 0.92, 12: 0.83 / 0.82 (10.6)
//   d = 260, k = 9   1.5: 0.91 / 0.91, 2.5: 0.83 / 0.83 (2.1)  k = 3   2: 0.94 / 0.98, 3: 0.88 / 0.91  (3.0)
//   d = 36,  k = 3   4: 0.85 / 0.97, 6: 0.78 / 0.85  (6.0), three blocks, which adds do in one instruction
inline bool worth_locking(int64_t sources, int64_t samples, int64_t capacity, int32_t d) {
  const int64_t blocks = (d + 15) / 16;
  if (blocks < 3) return false;
  const bool aligned = d % 16 == 0;
  double full = static_cast<double>(d * capacity) / (131072.0 * 16);
  if (d > 256 && !aligned) full *= 0.8;  // fewer wavefronts: more registers per row
  const double saved = blocks == 3 ? 0.3
                       : aligned   ? std::min(full, full * full)
                       : d <= 64   ? full
                       : full < 0.58 ? 0.17
                                     : std::min(full, full * full * std::sqrt(full));
  const double per_sample = 1.0 / static_cast<double>(samples);
  const double rounds = std::max(0.9 + 3.6 * per_sample, aligned && d > 64 ? 0.0 : 7.2 * per_sample);
  return static_cast<double>(sources) * saved >= static_cast<double>(capacity) * rounds;
}

// Hubs.  Whoever holds a row keeps the others waiting for about as long as a source takes for one
// sample, so rows that are drawn too often as positive samples hold up the whole launch.  How
// often a row is drawn is counted, draw by draw, before the launch: a degree does not tell (many
// edges may lead to a vertex that has few of its own, and a vertex whose neighbours have no others
// is drawn by each of them; with a degree rule a graph of 67,000 vertices, a fifth of whose edges
// lead to twenty without out-edges, took 29 ms per epoch, 0.15 as adds and 0.15 like this).  A row
// is a hub if its draws would keep it locked for more than 1 / kHubShare of the launch, C sources
// at a time, each with `per_source` row updates in a row:
//   draws > max(2, sources * per_source / (kHubShare * C))
// or if more than kMostAtOnce of 64 consecutive sources draw it, which start at the same time.
// Shares of 2 / 8 / 16 on 200,000 x 128, us: stars of ten leaves in a row 504 / 374 / 375, R-MAT
// 231 / 228 / 226, power law 230 / 226 / 226; at 67,000 with a bound of 1 instead of 2 every fourth
// row is a hub.  Counting takes 7 us of 79 at 67,000 x 128.
constexpr int64_t kHubShare = 8;
constexpr uint32_t kMostAtOnce = 2;
constexpr uint32_t kDrawnAtOnce = 0x80000000u;  // flag in a word of draws

inline uint32_t most_draws(int64_t sources, int64_t per_source, int64_t in_flight) {
  const int64_t most = sources * per_source / (kHubShare * std::max<int64_t>(in_flight, 1));
  return static_cast<uint32_t>(std::min<int64_t>(std::max<int64_t>(most, 2), 0x7FFFFFFF));
}

// One draw per lane (at = -1: none) added to the words of `draws`; all lanes of the wavefront are
// present.  Equal draws of a wavefront are one atomic, since thousands of atomics on one word take
// some 6 ns each one after another; only the first few rows met are gathered like that, which
// is enough to meet one that many lanes draw.
__device__ __forceinline__ void count_draws(int32_t at, uint32_t *draws) {
  constexpr int kGathered = 8;
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(at >= 0);
  uint32_t mine = at >= 0 ? 1 : 0;  // draws that this lane adds
#pragma unroll 1
  for (int i = 0; i < kGathered && todo != 0; ++i) {
    const int leader = __builtin_amdgcn_readfirstlane(__builtin_ctzll(todo));
    const unsigned long long same = __ballot(at == __builtin_amdgcn_readlane(at, leader));
    if ((same >> lane) & 1) mine = lane == leader ? static_cast<uint32_t>(__popcll(same)) : 0;
    todo &= ~same;
  }
  if (mine > kMostAtOnce) atomicOr(draws + at, kDrawnAtOnce);
  else if (mine != 0) atomicAdd(draws + at, mine);
}

// Largest finite |entry| (the bits of a non-negative finite float order like the float) and the number of
// non-finite entries that a lane, then its wavefront, has looked at.
struct EntryCheck {
  uint32_t top = 0, bad = 0;
  __device__ __forceinline__ void look(const Float4 &x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t mag = __float_as_uint(x[c]) & 0x7FFFFFFFu;
      const bool finite = mag < 0x7F800000u;
      top = finite ? max(top, mag) : top;
      bad += finite ? 0u : 1u;
    }
  }
  __device__ __forceinline__ void reduce_wave() {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      top = max(top, static_cast<uint32_t>(__shfl_xor(static_cast<int>(top), off, 64)));
      bad += static_cast<uint32_t>(__shfl_xor(static_cast<int>(bad), off, 64));
    }
  }
  template <class Result>
  __device__ __forceinline__ void add_to(Result *out) const {
    // the word only grows: a stale value can only cost an atomic that was not needed
    if (top > __hip_atomic_load(&out->max_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&out->max_bits, top);
    if (bad) atomicAdd(&out->nonfinite, static_cast<unsigned long long>(bad));
  }
};

struct SgdArgs {
  HotSet hot;
  int32_t d;
  int32_t k_neg;    // sample t of a source is a positive iff t % (k_neg + 1) == 0
  int32_t samples;  // samples per source: k_neg + 1 per round
  float lr;
  int64_t sources_per_block;  // consecutive sources that one workgroup walks (a multiple of
                              // the sources that its wavefronts take per turn)
};

constexpr int kChunk = 4;  // sample rows in flight per source
// Tries of a lock before an update is added without it, and may be lost to the holder's store like
// any update of the lock-free scheme.  Every holder lets go after its own memory accesses and waits
// for no other lock meanwhile, and a row that many want is a hub, so this is not reached; it bounds
// the kernel's time whatever the lock words hold.
constexpr int32_t kMaxTries = 1 << 14;
inline int32_t lock_tries() { return seam(kSeamLockTries) ? static_cast<int32_t>(seam(kSeamLockTries)) : kMaxTries; }

// Atomic adds of whole rows with 128-bit units, by the whole wavefront.  A memory-side fp32 atomic
// costs one operation per instruction and line it touches, full or sparse.  A lane group of d/4
// lanes that adds its own four floats per lane needs four instructions per row, each touching every
// line of the row; here the rows to be added (one per lane group that asks, `mine`) are laid out
// side by side in LDS, 4 * LPG floats each, and lane l of the wavefront adds float l of every 64:
// 16 / LPG rows per instruction, each line touched once, and at most four instructions however many
// groups a wavefront has.  Needs d <= 64 and every lane of the wavefront present (no divergent branch
// around the call); `mine` and `row` are uniform inside a lane group.
//
// One row per instruction, its floats fetched from the lanes that hold them, made a wavefront's rows a
// serial chain.  us of epochs with k = 3, before / now (65,536 sources: the adds themselves bound it):
//   1,024 sources:  d = 8 24.8 / 6.4   d = 16 12.1 / 6.0   d = 32 9.4 / 5.9   d = 64 7.0 / 6.0
//   65,536 sources: d = 8 29.4 / 20.0  d = 16 26.1 / 24.1  d = 32 42.1 / 39.8
//   4.2 M sources, a mix of stores and adds: d = 32 1,124 / 1,100
template <int LPG>
struct RowsOfWave {
  Float4 step[64];
  float *row[64 / LPG];
};
template <int LPG>
__device__ __forceinline__ void add_rows_as_a_wave(bool mine, float *row, const Unit<4> &step, int32_t d, int lane,
                                                   RowsOfWave<LPG> &rows) {
  static_assert(LPG <= 16, "a row is at most 64 floats");
  const unsigned long long todo = __ballot(mine);
  if (todo == 0) return;  // the same for the whole wavefront
  rows.step[lane] = step.v;
  if ((lane & (LPG - 1)) == 0) rows.row[lane / LPG] = row;
  // a wavefront's LDS accesses take effect in program order; the compiler must keep it
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const float *const floats = reinterpret_cast<const float *>(rows.step);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (((todo >> (16 * r)) & 0xFFFFu) == 0) continue;  // no owner of these 64 floats adds
    const int owner = 16 * r + (lane >> 2), column = (64 * r + lane) & (4 * LPG - 1);
    const float x = floats[64 * r + lane];
    float *const target = rows.row[owner / LPG];
    if (((todo >> owner) & 1) != 0 && column < d) atomic_step(target + column, x);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Position of a chunk of kChunk samples in the work of one lane group: source index, first
// sample of the chunk, and the index of the next positive sample at or after it.  All lane
// groups of a wavefront are at the same (t0, np); only idx differs.
struct ChunkPos {
  int64_t idx;
  int32_t t0, np;
  // The chunk that follows: the next kChunk samples of the same source, or the first chunk of
  // the group's next source.
  __device__ __forceinline__ ChunkPos next(int32_t samples, int32_t per_round, int64_t stride) const {
    const int32_t end = t0 + kChunk;
    int32_t p = np;
#pragma unroll
    for (int q = 0; q < kChunk; ++q) p = p < end ? p + per_round : p;
    const bool wrap = end >= samples;
    return ChunkPos{wrap ? idx + stride : idx, wrap ? 0 : end, wrap ? 0 : p};
  }
  // Which of the chunk's samples are positives.
  __device__ __forceinline__ void positives(int32_t per_round, bool (&is_pos)[kChunk]) const {
    int32_t p = np;
#pragma unroll
    for (int q = 0; q < kChunk; ++q) {
      is_pos[q] = (t0 + q == p);
      p = is_pos[q] ? p + per_round : p;
    }
  }
};

// The lock-free SGD kernel.  Every source applies `samples` updates of Alg. 1 in order:
//   g = lr * (b - sigmoid(M[src] . M[v]));  M[src] += g*M[v];  M[v] += g*M[src]
// with the source row held in registers for its whole turn.
//   W (work description, passed by value) provides
//     int64_t count()                         number of sources
//     int32_t source_id(int64_t i)            vertex id of source i (random counter, self test)
//     float  *source_row(int64_t i)
//     Pre     stage1(int64_t i, bool want)    what sampling for source i needs from memory and
//                                             can be asked for knowing i alone (row offsets)
//     uint64_t draw(int64_t i, int32_t id, int32_t t)
//                                             the random draw of sample t: arithmetic only
//     int32_t stage2(int64_t i, int32_t id, int32_t t, bool want, bool positive, Pre, uint64_t r)
//                                             vertex id of sample t from its draw r (-1 = none,
//                                             or !want)
//     float  *sample_row(int64_t i, int32_t v)
//     int32_t source_slot(int64_t i), sample_slot(int64_t i, int32_t v)
//                                             place of a row among the words of HotSet
//     bool    rows_at_lines()                 (host) every row starts at a line border, or near enough
//     Both stages must be free of branches around their memory reads (read a safe address
//     when !want).
//   Sample t of a source is a positive iff t % (k_neg + 1) == 0.
//   P: row access policy; LPG lanes per source, UPL units per lane (LPG*UPL*P::F >= d).
//   SEQ: a single lane group walks all sources in ascending index (the sequential-order
//   result), with whatever policy, geometry and hot-row mode it is instantiated and called
//   with: all accesses to the matrix then come from one wavefront in program order, and the
//   memory system keeps the accesses of a wavefront to one address in that order, so stores
//   and atomic adds alike take effect in the order of Alg. 3.  Otherwise every workgroup
//   walks a block of consecutive sources, its lane groups working side by side.
//
// Sampling is independent of the matrix (the draws are counter-based), so it runs ahead of
// the updates as a three-stage pipeline over chunks of kChunk samples: while the rows of
// chunk c are in flight, the neighbour-list entry (or pool entry) of chunk c+1 is requested
// with offsets that were requested one chunk earlier, and the offsets of chunk c+2 are
// requested.  A lane group thus waits for one memory round trip per chunk -- its rows --
// instead of three in a row (offsets, then neighbour, then rows); for rows of a few hundred
// bytes or less that chain, not bandwidth, is what bounds the kernel.
//
// The body is written without branches around memory reads: a sample that does not
// exist, or a column beyond d, reads a harmless valid address and is masked afterwards
// (its step is forced to zero, its store is skipped).  All reads of a chunk are therefore
// issued back to back and waited for once, which is what keeps their latencies overlapped;
// with predicated reads the compiler splits the code into blocks and waits in each.
template <class P, int LPG, int UPL, class W, bool SEQ>
__device__ __forceinline__ void sgd_walk(const W &w, const SgdArgs &a) {
  constexpr int kGroupsPerWave = 64 / LPG;
  constexpr int kPasses = (kChunk + LPG - 1) / LPG;  // sampler passes per chunk (lane q takes sample q)
  constexpr int F = P::F;
  using U = Unit<F>;
  using Pre = typename W::Pre;
  const int lane = threadIdx.x & 63;
  const int gl = lane & (LPG - 1);
  // The sequential walk is done by the first lane group of the first wavefront; the other
  // groups of that wavefront tag along without a source (the wavefront-wide atomic adds want
  // all 64 lanes present).
  if (SEQ && (threadIdx.x >= 64 || blockIdx.x != 0)) return;
  const bool group_on = !SEQ || lane < LPG;

  // A workgroup walks a block of consecutive sources: in each turn its wavefronts take one load
  // of kGroupsPerWave sources each, next to each other.  Workgroups start in the order of their
  // index, so the sources of an epoch are taken up in ascending order in time however many of
  // them one wavefront walks, and neighbouring sources (whose neighbour lists share cache
  // lines) are handled on one compute unit at one time.  `n` is the end of the block.
  const int64_t waves_per_block = SEQ ? 1 : blockDim.x / 64;
  const int64_t block_lo = SEQ ? 0 : blockIdx.x * a.sources_per_block;
  const int64_t first_of_wave = block_lo + (SEQ ? 0 : (threadIdx.x >> 6) * kGroupsPerWave);
  const int64_t n = SEQ ? w.count() : std::min<int64_t>(w.count(), block_lo + a.sources_per_block);
  const int64_t stride = SEQ ? 1 : waves_per_block * kGroupsPerWave;
  const int64_t first = first_of_wave + (SEQ ? 0 : lane / LPG);
  const int32_t d = a.d;
  const int32_t per_round = a.k_neg + 1;
  const bool use_bitmap = a.hot.mode == kHotBitmap;
  const bool all_hot = a.hot.mode == kHotAll;
  const uint32_t *const bits = a.hot.bits;  // always a readable word, also without a bitmap

  // Lane gl owns floats [(gl + i*LPG)*F, +F) of a row, i < UPL: consecutive lanes touch
  // consecutive addresses, so each access instruction covers whole cache lines.  Columns
  // beyond d are read from the last unit of the row instead and masked.
  // With P::kAligned the lane's columns depend on the address of the row (see RowAgentLine).
  constexpr int kSlots = LPG * UPL;
  static_assert(!P::kAligned || (F == 1 && (kSlots & (kSlots - 1)) == 0), "slots wrap around by masking");
  auto column = [&](const float *row, int i) -> int32_t {
    if constexpr (P::kAligned) {
      const int32_t behind_line = static_cast<int32_t>(reinterpret_cast<uintptr_t>(row) >> 2) & 31;
      return (gl + i * LPG - behind_line) & (kSlots - 1);
    } else {
      return (gl + i * LPG) * F;
    }
  };
  auto readable = [&](int32_t c) { return c < d ? c : d - F; };
  // the source row by column; the entries past d stay zero
  __shared__ float held_rows[P::kAligned ? 256 / LPG * kSlots : 1];
  float *const held = held_rows + (P::kAligned ? threadIdx.x / LPG * kSlots : 0);
  auto held_in_order = [] {  // the wavefront's LDS accesses take effect in program order; keep that order
    if constexpr (P::kAligned) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };

  __shared__ RowsOfWave<P::kWaveAtomics ? LPG : 16> all_rows[P::kWaveAtomics ? 4 : 1];
  auto &rows_of_wave = all_rows[P::kWaveAtomics ? threadIdx.x >> 6 : 0];

  // Stage 2 for the chunk at `pos`: lane q of the group evaluates sample pos.t0 + q (in
  // several passes if the group has fewer than kChunk lanes).
  auto draw_ids = [&](const ChunkPos &pos, const Pre &pre, int32_t (&mine)[kPasses]) {
    const bool live = group_on && pos.idx < n;
    const bool any_live = __ballot(live) != 0;  // the same for the whole wavefront: a jump, not a mask
    const int64_t i = live ? pos.idx : 0;
    const int32_t id = w.source_id(i);
    bool is_pos[kChunk];
    pos.positives(per_round, is_pos);
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int32_t t = pos.t0 + p * LPG + gl;
      const bool want = live && p * LPG + gl < kChunk && t < a.samples;
      bool mine_pos = false;
#pragma unroll
      for (int q = 0; q < LPG && p * LPG + q < kChunk; ++q) mine_pos = (gl == q) ? is_pos[p * LPG + q] : mine_pos;
      // Past a wavefront's last chunk nobody wants the draw: only the arithmetic is skipped,
      // the reads of stage 2 stay unconditional.
      uint64_t r = 0;
      if (any_live) r = w.draw(i, id, want ? t : 0);
      mine[p] = w.stage2(i, id, want ? t : 0, want, mine_pos, pre, r);
    }
  };
  auto offsets_for = [&](const ChunkPos &pos) {
    const bool live = group_on && pos.idx < n;
    return w.stage1(live ? pos.idx : 0, live);
  };

  // Pipeline prologue: the ids of the group's first chunk and the offsets of its second.
  int32_t mine[kPasses];
  Pre pre_next;
  {
    const ChunkPos c0{first, 0, 0};
    draw_ids(c0, offsets_for(c0), mine);
    pre_next = offsets_for(c0.next(a.samples, per_round, stride));
  }

  // The loop bound is uniform over the wave.  A group without a source (past the end, or
  // tagging along in the sequential walk) goes through the motions on source 0 -- it reads,
  // computes and writes nothing -- so that no lane ever leaves the wavefront's control flow.
  for (int64_t base = first_of_wave; base < n; base += stride) {
    const int64_t idx_raw = first + (base - first_of_wave);
    const bool live = group_on && idx_raw < n;
    const int64_t idx = live ? idx_raw : 0;
    const int32_t src = w.source_id(idx);
    float *const src_row = w.source_row(idx);
    // The source row is requested here and first touched after the rows of the first chunk
    // have been requested too (`fresh`): nothing may read a unit before P::settle.
    U s[UPL], s_before[UPL];
#pragma unroll
    for (int i = 0; i < UPL; ++i) s[i] = P::load(src_row + readable(column(src_row, i)));
    const uint32_t src_word = bits[use_bitmap ? (src >> 5) : 0];
    bool fresh = true;

    ChunkPos cur{idx_raw, 0, 0};
    for (int32_t t0 = 0; t0 < a.samples; t0 += kChunk) {
      bool is_pos[kChunk];
      cur.positives(per_round, is_pos);
      // The ids of this chunk were drawn one chunk ago; spread them over the group.
      int32_t v[kChunk];
#pragma unroll
      for (int p = 0; p < kPasses; ++p)
#pragma unroll
        for (int q = 0; q < LPG && p * LPG + q < kChunk; ++q) v[p * LPG + q] = __shfl(mine[p], q, LPG);

      // Request every row of the chunk (a missing sample reads the source row instead).
      U r[kChunk][UPL];
      uint32_t word[kChunk];
      bool valid[kChunk];
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        valid[q] = live && v[q] >= 0 && v[q] != src;  // a sample that hits the source applies no update
        const float *row = valid[q] ? w.sample_row(idx, v[q]) : src_row;
#pragma unroll
        for (int i = 0; i < UPL; ++i) r[q][i] = P::load(row + readable(column(row, i)));
        word[q] = bits[(use_bitmap && valid[q]) ? (v[q] >> 5) : 0];
      }
      // While they are in flight: the ids of the next chunk (its offsets arrived a chunk
      // ago) and the offsets of the chunk after it.
      const ChunkPos ahead1 = cur.next(a.samples, per_round, stride);
      draw_ids(ahead1, pre_next, mine);
      pre_next = offsets_for(ahead1.next(a.samples, per_round, stride));
      cur = ahead1;  // (its idx is this source's again unless this was the last chunk)

      // Everything this chunk needs has been asked for: from here on the rows may be used.
      P::wait_all();
#pragma unroll
      for (int i = 0; i < UPL; ++i) {
        P::settle(s[i]);
#pragma unroll
        for (int c = 0; c < F; ++c) {
          s[i].v[c] = column(src_row, i) < d ? s[i].v[c] : 0.f;
          s_before[i].v[c] = fresh ? s[i].v[c] : s_before[i].v[c];
        }
        if constexpr (P::kAligned)
          if (fresh) held[column(src_row, i)] = s[i].v[0];
      }
      held_in_order();
      fresh = false;
#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        const float *const row = valid[q] ? w.sample_row(idx, v[q]) : src_row;
#pragma unroll
        for (int i = 0; i < UPL; ++i) {
          P::settle(r[q][i]);
#pragma unroll
          for (int c = 0; c < F; ++c) r[q][i].v[c] = column(row, i) < d ? r[q][i].v[c] : 0.f;
        }
      }

#pragma unroll
      for (int q = 0; q < kChunk; ++q) {
        float *const row = valid[q] ? w.sample_row(idx, v[q]) : src_row;
        if constexpr (P::kAligned) {
#pragma unroll
          for (int i = 0; i < UPL; ++i) s[i].v[0] = held[column(row, i)];
        }
        float partial = 0.f;
#pragma unroll
        for (int i = 0; i < UPL; ++i)
#pragma unroll
          for (int c = 0; c < F; ++c) partial = fmaf(s[i].v[c], r[q][i].v[c], partial);
        const float x = group_sum<LPG>(partial);
        const float label = is_pos[q] ? 1.f : 0.f;
        // a missing sample takes a zero step: both rows stay exactly as they are
        const float g = valid[q] ? a.lr * (label - 1.f / (1.f + expf(-x))) : 0.f;
#pragma unroll
        for (int i = 0; i < UPL; ++i)
#pragma unroll
          for (int c = 0; c < F; ++c) {
            s[i].v[c] = fmaf(g, r[q][i].v[c], s[i].v[c]);
            r[q][i].v[c] = fmaf(g, s[i].v[c], r[q][i].v[c]);
          }
        if constexpr (P::kAligned) {
#pragma unroll
          for (int i = 0; i < UPL; ++i) held[column(row, i)] = s[i].v[0];
          held_in_order();
        }
        {
          const bool hot = valid[q] && (all_hot || ((word[q] >> (v[q] & 31)) & 1u));
          if (valid[q] && !hot) {  // uniform over the group; only writes inside
#pragma unroll
            for (int i = 0; i < UPL; ++i)
              if (column(row, i) < d) P::store(row + column(row, i), r[q][i]);
          }
          if constexpr (P::kWaveAtomics) {
            static_assert(!P::kWaveAtomics || (UPL == 1 && F == 4), "one 128-bit unit per lane");
            U step;
#pragma unroll
            for (int c = 0; c < F; ++c) step.v[c] = g * s[0].v[c];
            add_rows_as_a_wave<LPG>(hot, row, step, d, lane, rows_of_wave);
          } else if (hot) {
#pragma unroll
            for (int i = 0; i < UPL; ++i)
#pragma unroll
              for (int c = 0; c < F; ++c)
                if (column(row, i) < d) atomic_step(row + column(row, i) + c, g * s[i].v[c]);
          }
        }
        // A later sample of the same chunk that names the same vertex must see this
        // update: forward the registers instead of the stale prefetched copy.
#pragma unroll
        for (int z = q + 1; z < kChunk; ++z) {
          const bool same = valid[q] && v[z] == v[q];
#pragma unroll
          for (int i = 0; i < UPL; ++i)
#pragma unroll
            for (int c = 0; c < F; ++c) r[z][i].v[c] = same ? r[q][i].v[c] : r[z][i].v[c];
        }
      }
    }
    if constexpr (P::kAligned) {
#pragma unroll
      for (int i = 0; i < UPL; ++i) s[i].v[0] = held[column(src_row, i)];
      held_in_order();
    }
    const bool src_hot = live && (all_hot || ((src_word >> (src & 31)) & 1u));
    if (live && !src_hot) {
#pragma unroll
      for (int i = 0; i < UPL; ++i)
        if (column(src_row, i) < d) P::store(src_row + column(src_row, i), s[i]);
    }
    if constexpr (P::kWaveAtomics) {
      U step;
#pragma unroll
      for (int c = 0; c < F; ++c) step.v[c] = s[0].v[c] - s_before[0].v[c];
      add_rows_as_a_wave<LPG>(src_hot, src_row, step, d, lane, rows_of_wave);
    } else if (src_hot) {
#pragma unroll
      for (int i = 0; i < UPL; ++i)
#pragma unroll
        for (int c = 0; c < F; ++c)
          if (column(src_row, i) < d) atomic_step(src_row + column(src_row, i) + c, s[i].v[c] - s_before[i].v[c]);
    }
  }
}

// Workgroups of sgd_locked_kernel: one wavefront, which makes room for the next when it ends and not
// when three others end too; long rows, of which few fit a CU, stay at four.
template <int UPL>
constexpr int kLockedThreads = UPL > 4 ? 256 : 64;
// Wavefronts per SIMD, no fewer (the registers allow them without scratch) and no more.  More sources in
// flight are faster, but a source then works on a copy of its row that is further behind, and the result
// lies further from the sequential order of Alg. 3: these counts keep it where chunks of four samples in
// workgroups of four had it.  Sources of a visit hold their rows for B rounds.  Relative distance from
// the sequential result, and us: with chunks of four / up to seven wavefronts per SIMD / these counts
//   epoch 67,000 x 128, k = 3       2.66e-4 / 2.87e-4 / 2.67e-4      101 /     80 /     83
//   epoch 262,144 x 64, k = 3       1.98e-4 / 2.14e-4 / 1.98e-4      178 /    158 /    164
//   epoch 333,337 x 100, k = 9      2.92e-4 / 3.11e-4 / 2.89e-4    1,003 /    828 /    860
//   epoch 60,000 x 260, k = 9       3.70e-4 / 4.18e-4 / 3.65e-4      492 /    355 /    424
//   visits, in place 2 M x 128      8.77e-5 / 1.02e-4 / 8.65e-5   47,400 / 40,900 / 42,800
//   visits, in place 262,147 x 100  5.85e-5 / 6.91e-5 / 5.85e-5    3,510 /  2,620 /  2,960
//   visits, in place 400,001 x 64   1.60e-4 / 1.79e-4 / 1.53e-4    4,880 /  4,320 /  4,700
//   visits, in place 100,001 x 512  6.09e-5 / 8.18e-5 / 5.40e-5    3,150 /  3,060 /  3,150
//   visits, in place 300,001 x 128  3.11e-5 / 4.00e-5 / 3.38e-5    2,220 /  1,930 /  1,970  (R-MAT)
template <class P, int UPL, class W>
constexpr int kLockedWaves = UPL > 4 ? (P::kAligned || W::kLongTurns ? 3 : 4)
                                     : (P::kAligned ? 5 : 6) - (W::kLongTurns ? 1 : 0);

// Waits for all outstanding accesses to memory, and lets the compiler know that it has.
__device__ __forceinline__ void wait_memory() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), nothing else
  asm volatile("" ::: "memory");
}

// The same epoch or visit with every row written under a lock (see kHotLocked); template arguments as
// in sgd_walk.  The samples of a source are taken one after another, each group at its own pace, in
// chunks of at most LPG whose ids lie one to a lane: a chunk's ids are drawn while the chunk before it
// runs, one round of Philox for up to LPG samples.  A row takes two round trips: the exchange of its
// lock (never waited for; behind it the stores of the row before have arrived, and that row's lock is
// given back), then the read of the row.  A group holds one lock while it tries another but never waits
// for one, so no two can wait for each other.
//
// What bounds it is the latency of those round trips (70 to 80 % of a wavefront's time), so the layout is
// made for few registers: the source row as it was read lies in LDS, ids and hub flags are a register
// each and not one per sample, places are 32-bit.  With chunks of four samples as in sgd_walk 67,000 x
// 128, k = 3 took 93.5 us, now 78.5 with the counting of the draws; 333,337 x 100, k = 9 1,045, now 969 (750
// on one matrix that stays in the memory-side cache); the pair scheme in place on 4 x 500,000 rows at d = 128 47.4 ms,
// now 43.0 (3.9 G rows/s; visits of 2 x 58,000 rows, which the memory-side cache holds, 5.2 G).
// The source row is read with the first sample's, where that can be: read earlier it is older (67,000 x
// 128 with seven wavefronts per SIMD: distance from the sequential epoch 2.96e-4, so 2.88e-4, for the same
// time).
// What lost: the lock of the next row asked for while a row is read (one round trip per row, but then a
// lock is held while another is not to be had: 67,000 x 128 98 -> 1,200 us, visits 1.5 to 2.5 times
// as long); versions in the lock words, which let a row be read beside its lock (140 us: a load from a
// line that others write words of costs more than the round trip, also where the versions lie apart);
// eight wavefronts per SIMD by spilling (878 -> 945 us at 333,337 x 100).
template <class P, int LPG, int UPL, class W, bool SEQ>
__device__ __forceinline__ void sgd_locked_walk(const W &w, const SgdArgs &a, const LockSet &lock) {
  constexpr int kGroupsPerWave = 64 / LPG;
  constexpr int F = P::F;
  using U = Unit<F>;
  // Whether the source row is read with the first sample's row or, where loads are written out, before
  // it with the lock: the wait for them must follow in the code too.
  constexpr bool kLate = !P::kWaveAtomics;
  using Pre = typename W::Pre;
  using Mask = std::conditional_t<(LPG > 32), uint64_t, uint32_t>;  // a bit per lane of the group
  const int lane = threadIdx.x & 63;
  const int gl = lane & (LPG - 1);
  if (SEQ && (threadIdx.x >= 64 || blockIdx.x != 0)) return;
  const bool group_on = !SEQ || lane < LPG;

  // A workgroup walks a block of consecutive sources, as in sgd_walk.  (Rotations gain 3 % when the turns
  // of a workgroup lie the grid's width apart, but that takes the sources of both parts of a visit up
  // side by side instead of one part's after the other's.)  Sources fit 31 bits, as vertices do, and so
  // does what follows the last ones.
  constexpr uint32_t kWaves = SEQ ? 1 : kLockedThreads<UPL> / 64;
  const uint32_t per_block = static_cast<uint32_t>(a.sources_per_block);
  const uint32_t block_lo = SEQ ? 0 : blockIdx.x * per_block;
  const uint32_t count = static_cast<uint32_t>(w.count());
  const uint32_t n = SEQ ? count : std::min(count, block_lo + per_block);
  const uint32_t first_of_wave = block_lo + (SEQ ? 0 : threadIdx.x / 64 * kGroupsPerWave);
  const uint32_t stride = SEQ ? 1 : kWaves * kGroupsPerWave;
  const uint32_t first = first_of_wave + (SEQ ? 0 : lane / LPG);
  const int32_t d = a.d;
  const int32_t per_round = a.k_neg + 1;

  constexpr int kSlots = LPG * UPL;
  static_assert(!P::kAligned || (F == 1 && (kSlots & (kSlots - 1)) == 0), "slots wrap around by masking");
  auto column = [&](const float *row, int i) -> int32_t {
    if constexpr (P::kAligned) {
      const int32_t behind_line = static_cast<int32_t>(reinterpret_cast<uintptr_t>(row) >> 2) & 31;
      return (gl + i * LPG - behind_line) & (kSlots - 1);
    } else {
      return (gl + i * LPG) * F;
    }
  };
  auto readable = [&](int32_t c) { return c < d ? c : d - F; };
  // the source row by column; the entries past d stay zero
  __shared__ float held_rows[P::kAligned ? kLockedThreads<UPL> / LPG * kSlots : 1];
  float *const held = held_rows + (P::kAligned ? threadIdx.x / LPG * kSlots : 0);
  auto held_in_order = [] {  // the wavefront's LDS accesses take effect in program order; keep that order
    if constexpr (P::kAligned) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  // the source row as it was read, later its change; every lane uses its own entries only
  __shared__ float kept_rows[kLockedThreads<UPL> * UPL * F];
  auto kept = [&](int i, int c) -> float & { return kept_rows[(i * F + c) * kLockedThreads<UPL> + threadIdx.x]; };

  __shared__ RowsOfWave<P::kWaveAtomics ? LPG : 16> all_rows[P::kWaveAtomics ? kLockedThreads<UPL> / 64 : 1];
  auto &rows_of_wave = all_rows[P::kWaveAtomics ? threadIdx.x >> 6 : 0];

  auto in_group = [&](bool x) -> Mask {
    return static_cast<Mask>(__ballot(x) >> (lane & ~(LPG - 1))) & static_cast<Mask>(~uint64_t{0} >> (64 - LPG));
  };
  auto first_of = [](Mask m) -> int { return LPG > 32 ? __builtin_ctzll(m) : __builtin_ctz(static_cast<uint32_t>(m)); };

  const bool whole = d == kSlots * F;
  auto store_row = [&](float *row, const U (&u)[UPL]) {
    if (!P::kAligned && whole) {
#pragma unroll
      for (int i = 0; i < UPL; ++i) P::store(row + (gl + i * LPG) * F, u[i]);
    } else {
#pragma unroll
      for (int i = 0; i < UPL; ++i)
        if (column(row, i) < d) P::store(row + column(row, i), u[i]);
    }
  };

  // Lane gl draws sample t0 + gl of source idx (-1 = none).
  auto draw_ids = [&](uint32_t idx, int32_t t0, const Pre &pre) -> int32_t {
    const bool live = group_on && idx < n;
    const bool any_live = __ballot(live) != 0;  // the same for the whole wavefront: a jump, not a mask
    const uint32_t i = live ? idx : 0;
    const int32_t id = w.source_id(i);
    const bool want = live && t0 + gl < a.samples;
    const int32_t t = want ? t0 + gl : 0;
    uint64_t r = 0;
    if (any_live) r = w.draw(i, id, t);
    const int32_t v = w.stage2(i, id, t, want, t % per_round == 0, pre, r);
    return v == id ? -1 : v;  // a sample that hits the source applies no update
  };
  auto offsets_for = [&](uint32_t idx) {
    const bool live = group_on && idx < n;
    return w.stage1(live ? idx : 0, live);
  };

  // The lock to let go (slot, -1 none) behind the next wait.
  int32_t held_slot = -1;
  auto wait_and_release = [&]() {
    P::wait_all();
    wait_memory();
    if (held_slot >= 0 && gl == 0)
      __hip_atomic_store(lock.locks + held_slot, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    held_slot = -1;
  };
  // One try at a lock: what its word was (0 = the lock was free and is now held).
  auto try_lock = [&](bool ask, int32_t slot) -> uint32_t {
    uint32_t old = 1;
    if (ask && gl == 0) old = __hip_atomic_exchange(lock.locks + slot, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return old;
  };

  // Pipeline prologue: the ids of the group's first chunk, the offsets of its second.
  int32_t mine = draw_ids(first, 0, offsets_for(first));
  const bool one_chunk = a.samples <= LPG;
  Pre pre_next = offsets_for(one_chunk ? first + stride : first);
  const uint32_t first_idx = group_on && first < n ? first : 0;
  uint32_t draws = lock.draws[mine >= 0 ? w.sample_slot(first_idx, mine) : 0];  // of the lane's sample

  for (uint32_t base = first_of_wave; base < n; base += stride) {
    const uint32_t idx_raw = first + (base - first_of_wave);
    const bool live = group_on && idx_raw < n;
    const uint32_t idx = live ? idx_raw : 0;
    float *const src_row = w.source_row(idx);
    const int32_t src_slot = w.source_slot(idx);
    const uint32_t src_draws = lock.draws[src_slot];
    U s[UPL];
    auto read_source = [&] {
#pragma unroll
      for (int i = 0; i < UPL; ++i) s[i] = P::load(src_row + readable(column(src_row, i)));
    };
    auto keep_source = [&] {  // behind a wait
#pragma unroll
      for (int i = 0; i < UPL; ++i) {
        P::settle(s[i]);
        const bool inside = column(src_row, i) < d;
#pragma unroll
        for (int c = 0; c < F; ++c) {
          s[i].v[c] = inside ? s[i].v[c] : 0.f;
          kept(i, c) = s[i].v[c];
        }
        if constexpr (P::kAligned) held[column(src_row, i)] = s[i].v[0];
      }
      held_in_order();
    };
    for (int32_t t0 = 0; t0 < a.samples; t0 += LPG) {
      const bool last = t0 + LPG >= a.samples;
      const uint32_t idx_ahead = last ? idx_raw + stride : idx_raw;
      const int32_t t0_ahead = last ? 0 : t0 + LPG;
      Mask todo = in_group(mine >= 0);  // samples of the chunk that this group has not applied yet
      const Mask hubs = in_group(draws > lock.most);
      const Mask positives = in_group((t0 + gl) % per_round == 0);
      int32_t mine_ahead = -1;
      int32_t id = __shfl(mine, todo ? first_of(todo) : 0, LPG);
      for (int32_t tries = 0;; ++tries) {
        const bool want = todo != 0;
        if (tries > 0 && __ballot(want) == 0) break;  // the same for the whole wavefront
        const int q = want ? first_of(todo) : 0;
        const bool hub = want && ((hubs >> q) & 1u) != 0;
        const int32_t slot = want ? w.sample_slot(idx, id) : 0;
        const uint32_t word = try_lock(want && !hub, slot);
        const bool fresh = t0 == 0 && tries == 0;  // the source row has not been read yet
        if (fresh && !kLate) read_source();
        if (tries == 0) {
          mine_ahead = draw_ids(idx_ahead, t0_ahead, pre_next);
          pre_next = offsets_for(t0_ahead + LPG >= a.samples ? idx_ahead + stride : idx_ahead);
        }
        wait_and_release();
        if (fresh && !kLate) keep_source();
        const bool locked = __shfl(word, 0, LPG) == 0;
        const bool add = want && (hub || (!locked && tries >= lock.max_tries));
        const bool apply = locked || add;
        float *const row = apply ? w.sample_row(idx, id) : src_row;
        U r[UPL];
        if (apply)
#pragma unroll
          for (int i = 0; i < UPL; ++i) r[i] = P::load(row + readable(column(row, i)));
        if (fresh && kLate) read_source();
        if (tries == 0)
          draws = lock.draws[mine_ahead >= 0 ? w.sample_slot(group_on && idx_ahead < n ? idx_ahead : 0, mine_ahead) : 0];
        P::wait_all();
        if (fresh && kLate) keep_source();

        float partial = 0.f;
#pragma unroll
        for (int i = 0; i < UPL; ++i) {
          P::settle(r[i]);
          if constexpr (P::kAligned) s[i].v[0] = held[column(row, i)];
#pragma unroll
          for (int c = 0; c < F; ++c) {
            r[i].v[c] = apply && column(row, i) < d ? r[i].v[c] : 0.f;  // no step leaves the source as it is, infinities too
            partial = fmaf(s[i].v[c], r[i].v[c], partial);
          }
        }
        const float x = group_sum<LPG>(partial);
        const float label = ((positives >> q) & 1u) ? 1.f : 0.f;
        const float g = apply ? a.lr * (label - 1.f / (1.f + expf(-x))) : 0.f;
#pragma unroll
        for (int i = 0; i < UPL; ++i)
#pragma unroll
          for (int c = 0; c < F; ++c) {
            s[i].v[c] = fmaf(g, r[i].v[c], s[i].v[c]);
            r[i].v[c] = fmaf(g, s[i].v[c], r[i].v[c]);
          }
        if constexpr (P::kAligned) {
#pragma unroll
          for (int i = 0; i < UPL; ++i) held[column(row, i)] = s[i].v[0];
          held_in_order();
        }
        if (locked) {  // uniform over the group; only writes inside
          store_row(row, r);
          held_slot = slot;
        }
        if constexpr (P::kWaveAtomics) {
          U step;
#pragma unroll
          for (int c = 0; c < F; ++c) step.v[c] = g * s[0].v[c];
          add_rows_as_a_wave<LPG>(add, row, step, d, lane, rows_of_wave);
        } else if (add) {
#pragma unroll
          for (int i = 0; i < UPL; ++i)
#pragma unroll
            for (int c = 0; c < F; ++c)
              if (column(row, i) < d) atomic_step(row + column(row, i) + c, g * s[i].v[c]);
        }
        if (apply) {
          todo &= todo - 1;
          id = __shfl(mine, todo ? first_of(todo) : 0, LPG);
        }
      }
      mine = mine_ahead;
    }

    // The source's change, added to its row as it is now.
    if constexpr (P::kAligned) {
#pragma unroll
      for (int i = 0; i < UPL; ++i) s[i].v[0] = held[column(src_row, i)];
      held_in_order();
    }
#pragma unroll
    for (int i = 0; i < UPL; ++i)
#pragma unroll
      for (int c = 0; c < F; ++c) kept(i, c) = s[i].v[c] - kept(i, c);
    const bool hub = src_draws > lock.most;
    bool add = live;
    bool todo_src = live && !hub;
    for (int32_t tries = 0;; ++tries) {
      if (tries > 0 && __ballot(todo_src) == 0) break;  // the same for the whole wavefront
      const uint32_t word = try_lock(todo_src, src_slot);
      wait_and_release();
      const bool locked = __shfl(word, 0, LPG) == 0;
      U now[UPL];
      if (locked)
#pragma unroll
        for (int i = 0; i < UPL; ++i) now[i] = P::load(src_row + readable(column(src_row, i)));
      P::wait_all();
#pragma unroll
      for (int i = 0; i < UPL; ++i) {
        P::settle(now[i]);
#pragma unroll
        for (int c = 0; c < F; ++c) now[i].v[c] += kept(i, c);
      }
      if (locked) {
        store_row(src_row, now);
        held_slot = src_slot;
      }
      todo_src = todo_src && !locked && tries < lock.max_tries;
      add = add && !locked;
    }
    if constexpr (P::kWaveAtomics) {
      U step;
#pragma unroll
      for (int c = 0; c < F; ++c) step.v[c] = kept(0, c);
      add_rows_as_a_wave<LPG>(add, src_row, step, d, lane, rows_of_wave);
    } else if (add) {
#pragma unroll
      for (int i = 0; i < UPL; ++i)
#pragma unroll
        for (int c = 0; c < F; ++c)
          if (column(src_row, i) < d) atomic_step(src_row + column(src_row, i) + c, kept(i, c));
    }
  }
  wait_and_release();
}

template <class P, int LPG, int UPL, class W, bool SEQ>
__global__ __launch_bounds__(256) void sgd_kernel(W w, SgdArgs a) {
  sgd_walk<P, LPG, UPL, W, SEQ>(w, a);
}
template <class P, int LPG, int UPL, class W, bool SEQ>
__global__ __launch_bounds__(kLockedThreads<UPL>)
    __attribute__((amdgpu_waves_per_eu((kLockedWaves<P, UPL, W>), (kLockedWaves<P, UPL, W>)))) void
    sgd_locked_kernel(W w, SgdArgs a, LockSet lock) {
  sgd_locked_walk<P, LPG, UPL, W, SEQ>(w, a, lock);
}

// Whether the access instructions of lanes at columns 0, 1, 2, ... touch no more 64-byte blocks
// than they cover in every row of a matrix.
inline bool rows_at_lines(const float *M, int32_t d) { return reinterpret_cast<uintptr_t>(M) % 64 == 0 && d % 16 == 0; }

// Launches sgd_kernel for a given dimension.  Geometry:
//   plain_rows             plain 128-bit units, LPG = pow2ceil(d/4) lanes (<= 64): the layout
//                          of the sequential-order debug mode
//   otherwise, d <= 64     128-bit agent-scope units, LPG = pow2ceil(d/4) lanes, one unit per
//                          lane (4..64 sources per wavefront); hot rows are added to by the
//                          whole wavefront
//   otherwise, d  > 64     32-bit agent-scope units interleaved over LPG = pow2ceil(d/4)
//                          lanes (<= 64), four or eight units per lane; their columns from the
//                          address of the row where rows do not start at line borders
// Each of them runs concurrently (seq = false) or as one lane group (seq = true).
// `a.sources_per_block` is filled in here from `count`.
template <class W>
struct SgdLauncher {
  // LDS of a locked workgroup beyond what it uses, so that no more than `waves` wavefronts fit a CU.
  template <class P, int LPG, int UPL>
  static unsigned lds_for(int waves) {
    if (waves == 0) return 0;
    constexpr int kThreads = kLockedThreads<UPL>;
    constexpr unsigned kOwn = 4 * kThreads * UPL * P::F + (P::kAligned ? 4 * kThreads * UPL : 4) +
                              (P::kWaveAtomics ? kThreads / 64 * sizeof(RowsOfWave<(LPG <= 16 ? LPG : 16)>) : 0);
    constexpr unsigned kPerCu = 160 * 1024, kGranule = 1280;
    const unsigned share = kPerCu / std::max(waves / (kThreads / 64), 1) / kGranule * kGranule;
    return share > kOwn ? share - kOwn : 0;
  }

  template <class P, int LPG, int UPL>
  static void run(const W &w, SgdArgs a, const LockSet &lock, int64_t count, bool seq, int64_t max_waves,
                  hipStream_t st) {
    const bool locked = a.hot.mode == kHotLocked && !std::is_same_v<P, RowPlain128>;
    const int waves_per_block = locked ? kLockedThreads<UPL> / 64 : 4;
    constexpr int kGroupsPerWave = 64 / LPG;
    const int64_t per_turn = waves_per_block * kGroupsPerWave;  // sources a workgroup takes per turn
    const int64_t turns = std::max<int64_t>((count + per_turn - 1) / per_turn, 1);
    const int64_t max_blocks = std::max<int64_t>(max_waves / waves_per_block, 1);
    const int64_t per_block = (turns + max_blocks - 1) / max_blocks;  // turns of one workgroup
    const int64_t blocks64 = (turns + per_block - 1) / per_block;
    a.sources_per_block = per_block * per_turn;
    const int blocks = static_cast<int>(blocks64);
    if constexpr (!std::is_same_v<P, RowPlain128>) {
      if (locked && seq) hipLaunchKernelGGL((sgd_locked_kernel<P, LPG, UPL, W, true>), dim3(1), dim3(64), 0, st, w, a, lock);
      else if (locked)
        hipLaunchKernelGGL((sgd_locked_kernel<P, LPG, UPL, W, false>), dim3(blocks), dim3(kLockedThreads<UPL>),
                           (lds_for<P, LPG, UPL>(lock.waves_per_cu)), st, w, a, lock);
      if (locked) return;
    }
    if (seq) hipLaunchKernelGGL((sgd_kernel<P, LPG, UPL, W, true>), dim3(1), dim3(64), 0, st, w, a);
    else hipLaunchKernelGGL((sgd_kernel<P, LPG, UPL, W, false>), dim3(blocks), dim3(256), 0, st, w, a);
  }

  static int pow2_lanes(int units) {
    int lanes = 1;
    while (lanes < units && lanes < 64) lanes *= 2;
    return lanes;
  }

  // Lane groups per wavefront in concurrent mode (to size the launch and the hot-row rule).
  static int groups_per_wave(int32_t d) { return 64 / pow2_lanes(d / 4); }

  static void launch(const W &w, const SgdArgs &a, const LockSet &lock, int64_t count, bool seq, bool plain_rows,
                     int64_t max_waves, hipStream_t st) {
    const int d = a.d;
    if (plain_rows) {
      if (d > 256) return run<RowPlain128, 64, 2>(w, a, lock, count, seq, max_waves, st);
      switch (pow2_lanes(d / 4)) {
        case 64: return run<RowPlain128, 64, 1>(w, a, lock, count, seq, max_waves, st);
        case 32: return run<RowPlain128, 32, 1>(w, a, lock, count, seq, max_waves, st);
        case 16: return run<RowPlain128, 16, 1>(w, a, lock, count, seq, max_waves, st);
        case 8: return run<RowPlain128, 8, 1>(w, a, lock, count, seq, max_waves, st);
        case 4: return run<RowPlain128, 4, 1>(w, a, lock, count, seq, max_waves, st);
        case 2: return run<RowPlain128, 2, 1>(w, a, lock, count, seq, max_waves, st);
        default: return run<RowPlain128, 1, 1>(w, a, lock, count, seq, max_waves, st);
      }
    }
    if (d <= 64) {
      switch (pow2_lanes(d / 4)) {
        case 16: return run<RowAgent128, 16, 1>(w, a, lock, count, seq, max_waves, st);
        case 8: return run<RowAgent128, 8, 1>(w, a, lock, count, seq, max_waves, st);
        case 4: return run<RowAgent128, 4, 1>(w, a, lock, count, seq, max_waves, st);
        case 2: return run<RowAgent128, 2, 1>(w, a, lock, count, seq, max_waves, st);
        default: return run<RowAgent128, 1, 1>(w, a, lock, count, seq, max_waves, st);
      }
    }
    // Rows that straddle lines.  Measured before and after on 2^20 vertices (a mix of stores and
    // atomic adds) and 2^17 (all atomic adds), k = 3, us: d = 68 1,076 / 215 -> 967 / 170; d = 100
    // 1,456 / 304 -> 1,179 / 231; 124 1,620 / 356 -> 1,282 / 278; 132 1,417 / 348 -> 1,497 / 317;
    // 200 1,742 / 473 -> 1,710 / 429; 300 2,792 / 733 -> 2,718 / 644; 444 4,132 / 1,066 ->
    // 4,018 / 923.  At 132 half the lanes idle and the longer code costs more than the blocks
    // saved, unless every write is an atomic add.
    if (!w.rows_at_lines() && (d <= 128 || d > 192 || a.hot.mode >= kHotAll)) {
      if (d > 256) return run<RowAgentLine, 64, 8>(w, a, lock, count, seq, max_waves, st);
      if (d > 128) return run<RowAgentLine, 64, 4>(w, a, lock, count, seq, max_waves, st);
      return run<RowAgentLine, 32, 4>(w, a, lock, count, seq, max_waves, st);
    }
    if (d > 256) return run<RowAgent32, 64, 8>(w, a, lock, count, seq, max_waves, st);
    if (d > 128) return run<RowAgent32, 64, 4>(w, a, lock, count, seq, max_waves, st);
    return run<RowAgent32, 32, 4>(w, a, lock, count, seq, max_waves, st);
  }
};

}  // namespace gosh
