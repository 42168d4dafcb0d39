// MultiEdgeCollapse (Alg. 4 of the paper) on the device: the degree order and the marking
// sweep, with the results of the sequential algorithm.
//
// Order: a stable radix sort of the vertex ids by descending degree.
//
// Marking: in the sequential sweep a vertex becomes a hub iff none of the neighbours that
// precede it in the order and may take it (one of the two degrees is at most the mean
// degree) is itself a hub.  That recurrence is resolved out of order: a vertex above the
// mean degree is always a hub, a low-degree vertex with such a neighbour never is, and
// the remaining low-degree vertices are decided in rounds (hub once every preceding
// neighbour is decided and none is a hub, taken as soon as one is).  A decision is final
// and equals the sequential one, so stale reads can only delay it.  Hubs are numbered by
// a scan over the order; every other vertex joins its first hub in the order.
//
// Sort and scan are rocPRIM device primitives; the kernels around them are here.  The rebuild
// is in gosh_quotient.hip.  Everything runs on the null stream and the calls block.
#include <hip/hip_runtime.h>
#include <omp.h>

#include <algorithm>
#include <chrono>
#include <cstring>

#include <rocprim/rocprim.hpp>

#include "gosh_coarsen_internal.h"
#include "gosh_common.h"
#include "gosh_device_pool.h"
#include "gosh_quotient.h"

namespace {

using gosh::blocks_for;
using gosh::persistent;
using gosh::raise_by_block;

constexpr uint32_t kHighBit = 0x80000000u;   // set in rk[v] when deg(v) is above the mean
constexpr uint32_t kRankMask = 0x7FFFFFFFu;  // rk[v] & kRankMask = position of v in the order
enum : int32_t { kUndecided = 0, kHub = 1, kTaken = 2 };

__device__ inline int64_t first_wave() { return (blockIdx.x * 256LL + threadIdx.x) >> 6; }
__device__ inline int64_t wave_count() { return (gridDim.x * 256LL) >> 6; }

__device__ inline int32_t load_status(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_status(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// key = largest degree - degree: ascending keys are descending degrees; stable => ties by id.
template <typename OffT>
__global__ __launch_bounds__(256) void degree_keys_kernel(const OffT *__restrict__ xadj, int64_t n, uint32_t top,
                                                          uint32_t *__restrict__ keys) {
  for (int64_t v = blockIdx.x * 256LL + threadIdx.x; v < n; v += gridDim.x * 256LL)
    keys[v] = top - static_cast<uint32_t>(xadj[v + 1] - xadj[v]);
}

// rk[order[t]] = t, with the high bit set when the degree exceeds the mean degree
// (deg * n > nnz, exact in 64-bit integers).
__global__ __launch_bounds__(256) void rank_kernel(const uint32_t *__restrict__ sorted_keys,
                                                   const int32_t *__restrict__ order, int64_t n,
                                                   int64_t nnz, uint32_t top, uint32_t *__restrict__ rk) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL) {
    const int64_t deg = static_cast<int64_t>(top - sorted_keys[t]);
    rk[order[t]] = static_cast<uint32_t>(t) | (deg * n > nnz ? kHighBit : 0u);
  }
}

// Lanes per vertex of classify_kernel and join_kernel.  Both look at the entries of vertices of at most
// mean degree, after a chain of dependent reads (rank, offsets, entry, rank or status), and are bound by
// that chain: with a wavefront per vertex most lanes have no entry and few vertices are in flight.  Fewer
// lanes pay until the vertices no longer fill the device.  us with 64 / 16 / 8 / 4 lanes, both kernels, before
// the first stopped at a neighbour that decides and the second read ahead:
//   4.2 M vertices, R-MAT, mean degree 30: 1,430 / 868 / 774 / 724    its next level, mean above 100: 421 / 152 / 109 / 84
//   2.1 M, power law: 2,200 / 1,720 / 1,465 / 1,160                   1 M, uniform: 440 / 344 / 294 / 238
//   the last one's next levels, each about a tenth: 288 / 192 / 177 / 196, 82 / 59 / 68 / 98, 24 / 50 / 80 / 140
inline int lanes_per_vertex(int64_t n, int64_t nnz) {
  int lanes = n >= (int64_t{1} << 20) ? 4 : n >= (int64_t{1} << 16) ? 8 : n >= (int64_t{1} << 13) ? 16 : 64;
  while (lanes < 64 && lanes * 64 * n < nnz) lanes *= 2;  // at most 64 entries of a mean row to a lane
  return lanes;
}

// First classification, LANES lanes per vertex: needs no knowledge of other decisions.  Most vertices have
// a neighbour above the mean degree among their first few and need not look at the others.  What is left
// undecided is gathered in LDS, a wavefront's by itself, and takes its places in the list a hundred
// vertices at a time: one atomic per wavefront and turn, on one word, took 6 ns each and bound the kernel.
// 67 M entries of 4.2 M vertices (power law) 1,186 us, now 242; 128 M (R-MAT) 440, now 170.
constexpr int kHeldVertices = 128;
template <typename OffT, int LANES>
__global__ __launch_bounds__(256) void classify_kernel(const OffT *__restrict__ xadj,
                                                       const int32_t *__restrict__ adj,
                                                       const uint32_t *__restrict__ rk, int64_t n,
                                                       int32_t *__restrict__ status,
                                                       int32_t *__restrict__ pending,
                                                       unsigned long long *__restrict__ pending_count) {
  constexpr int kPerWave = 64 / LANES;
  __shared__ int32_t held[4][kHeldVertices];
  const int lane = threadIdx.x & 63, gl = lane & (LANES - 1), group = lane & ~(LANES - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t of_group = ~uint64_t{0} >> (64 - LANES) << group;
  int count = 0;  // vertices held, the same for the whole wavefront
  auto list_held = [&] {
    if (count == 0) return;
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(pending_count, static_cast<unsigned long long>(count));
    at = __shfl(at, 0, 64);
    for (int i = lane; i < count; i += 64) pending[at + i] = held[wave][i];
    count = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  for (int64_t base = first_wave() * kPerWave; base < n; base += wave_count() * kPerWave) {
    const int64_t v = base + lane / LANES;
    const uint32_t r = v < n ? rk[v] : kHighBit;
    bool open = !(r & kHighBit), taken = false, predecessor = false;  // the first two the same for a group
    int64_t e = 0, end = 0;
    if (open) {
      e = static_cast<int64_t>(xadj[v]) + gl;
      end = static_cast<int64_t>(xadj[v + 1]);
    }
    while (__ballot(open && e < end) != 0) {
      bool high = false;
      if (open && e < end) {
        const uint32_t ru = rk[adj[e]];
        high = (ru & kHighBit) != 0;
        predecessor |= (ru & kRankMask) < r;
      }
      if ((__ballot(high) & of_group) != 0) {
        taken = true;
        open = false;
      }
      e += LANES;
    }
    const bool undecided = !taken && (__ballot(predecessor) & of_group) != 0;
    if (gl == 0 && v < n) status[v] = taken ? kTaken : undecided ? kUndecided : kHub;
    const bool lists = gl == 0 && v < n && undecided;
    const uint64_t listed = __ballot(lists);
    if (listed != 0) {
      if (lists) held[wave][count + __popcll(listed & ((uint64_t{1} << lane) - 1))] = static_cast<int32_t>(v);
      count += __popcll(listed);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (count > kHeldVertices - kPerWave) list_held();
    }
  }
  list_held();
}

// One round over the undecided vertices, one wavefront per vertex.
template <typename OffT>
__global__ __launch_bounds__(256) void round_kernel(const OffT *__restrict__ xadj,
                                                    const int32_t *__restrict__ adj,
                                                    const uint32_t *__restrict__ rk,
                                                    int32_t *status,  // shared with other waves
                                                    const int32_t *__restrict__ pending, int64_t count,
                                                    int32_t *__restrict__ still,
                                                    unsigned long long *__restrict__ still_count) {
  const int lane = threadIdx.x & 63;
  for (int64_t i = first_wave(); i < count; i += wave_count()) {
    const int32_t v = pending[i];
    const uint32_t r = rk[v];  // low degree: no high bit
    bool taken = false, blocked = false;
    const int64_t begin = static_cast<int64_t>(xadj[v]), end = static_cast<int64_t>(xadj[v + 1]);
    for (int64_t e = begin + lane; e < end; e += 64) {
      const int32_t u = adj[e];
      if ((rk[u] & kRankMask) < r) {
        const int32_t su = load_status(status + u);
        taken |= su == kHub;
        blocked |= su == kUndecided;
      }
    }
    const bool any_taken = __ballot(taken) != 0, any_blocked = __ballot(blocked) != 0;
    if (lane == 0) {
      if (any_taken) store_status(status + v, kTaken);
      else if (!any_blocked) store_status(status + v, kHub);
      else still[atomicAdd(still_count, 1ull)] = v;
    }
  }
}

__global__ __launch_bounds__(256) void hub_flags_kernel(const int32_t *__restrict__ status,
                                                        const int32_t *__restrict__ order, int64_t n,
                                                        int32_t *__restrict__ flags) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL)
    flags[t] = status[order[t]] == kHub ? 1 : 0;
}

// Cluster ids are the hubs' positions among the hubs in the order.
__global__ __launch_bounds__(256) void number_hubs_kernel(const int32_t *__restrict__ flags,
                                                          const int32_t *__restrict__ index,
                                                          const int32_t *__restrict__ order, int64_t n,
                                                          int32_t *__restrict__ map,
                                                          unsigned long long *__restrict__ hubs) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL) {
    if (flags[t]) map[order[t]] = index[t];
    if (t == n - 1) *hubs = static_cast<unsigned long long>(index[t] + flags[t]);
  }
}

// Every taken vertex joins its first hub in the order, LANES lanes per vertex, four entries of a lane
// requested together.  A neighbour above the mean degree is a hub without asking.  (Graphs as above 519 us,
// now 336; 276, now 169.)  The hubs' own entries of map (read here) were written by the launch before this
// one; this launch writes only entries of taken vertices.
template <typename OffT, int LANES>
__global__ __launch_bounds__(256) void join_kernel(const OffT *__restrict__ xadj,
                                                   const int32_t *__restrict__ adj,
                                                   const uint32_t *__restrict__ rk,
                                                   const int32_t *__restrict__ status,
                                                   const int32_t *__restrict__ order, int64_t n,
                                                   int32_t *map) {
  constexpr int kPerWave = 64 / LANES, kAhead = 4;
  const int lane = threadIdx.x & 63, gl = lane & (LANES - 1);
  for (int64_t base = first_wave() * kPerWave; base < n; base += wave_count() * kPerWave) {
    const int64_t v = base + lane / LANES;
    uint32_t best = kRankMask;
    if (v < n && status[v] == kTaken) {
      const uint32_t r = rk[v];
      const int64_t begin = static_cast<int64_t>(xadj[v]), end = static_cast<int64_t>(xadj[v + 1]);
      for (int64_t e = begin + gl; e < end; e += kAhead * LANES) {
        int32_t u[kAhead];
        uint32_t ru[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) u[q] = adj[std::min(e + q * LANES, end - 1)];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) ru[q] = rk[u[q]];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
          const uint32_t t = ru[q] & kRankMask;
          if (t < r && t < best && ((ru[q] & kHighBit) != 0 || status[u[q]] == kHub)) best = t;
        }
      }
    }
    for (int offset = LANES / 2; offset > 0; offset >>= 1) best = min(best, __shfl_xor(best, offset, 64));
    // a taken vertex has a hub before it, so best is a valid position; the guard keeps a
    // broken invariant from turning into a wild read
    if (gl == 0 && best < static_cast<uint32_t>(n)) map[v] = map[order[best]];
  }
}

// Shape checks before any kernel follows the offsets or the neighbour ids: whether the offsets run
// from 0 to nnz without decreasing, and (second kernel) whether every neighbour id is inside [0, n).
// found->top becomes the largest degree met, for the order.
struct Found {
  uint32_t top;
  int32_t bad_offsets, bad_neighbour;
};

template <typename OffT>
__global__ __launch_bounds__(256) void check_offsets_kernel(const OffT *__restrict__ xadj, int64_t n,
                                                            int64_t nnz, Found *__restrict__ found) {
  uint32_t top = 0;
  for (int64_t v = blockIdx.x * 256LL + threadIdx.x; v < n; v += gridDim.x * 256LL) {
    const int64_t lo = static_cast<int64_t>(xadj[v]), hi = static_cast<int64_t>(xadj[v + 1]);
    if (lo > hi || lo < 0 || hi > nnz || (v == 0 && lo != 0) || (v == n - 1 && hi != nnz)) found->bad_offsets = 1;
    top = max(top, static_cast<uint32_t>(hi - lo));
  }
  __shared__ unsigned int block_top;
  if (threadIdx.x == 0) block_top = 0;
  __syncthreads();
  raise_by_block(&found->top, top, &block_top);
}

// Eight entries of a thread requested together: 128 M take 75 us, 152 one by one.  Offsets that are wrong say
// nothing of how many entries there are: then none is read.
__global__ __launch_bounds__(256) void check_neighbours_kernel(const int32_t *__restrict__ adj, int64_t nnz,
                                                               int64_t n, Found *__restrict__ found) {
  constexpr int kAhead = 8;
  if (found->bad_offsets) return;  // written by the launch before this one
  bool bad = false;
  for (int64_t first = blockIdx.x * (256LL * kAhead) + threadIdx.x; first < nnz; first += gridDim.x * (256LL * kAhead)) {
    int32_t u[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) u[q] = __builtin_nontemporal_load(adj + std::min(first + q * 256, nnz - 1));
#pragma unroll
    for (int q = 0; q < kAhead; ++q) bad |= u[q] < 0 || u[q] >= n;
  }
  if (bad) found->bad_neighbour = 1;
}

double ms_since(std::chrono::steady_clock::time_point t0) {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

}  // namespace

namespace gosh {

DeviceCoarsener *device_coarsener_new(int threads) {
  DeviceCoarsener *dc = new DeviceCoarsener();
  dc->threads = std::max(threads, 1);
  return dc;
}

void device_coarsener_free(DeviceCoarsener *dc) { delete dc; }

void device_coarsener_trim(DeviceCoarsener *dc) {
  if (dc) dc->pool.trim();
}

void device_blocks_trim() { block_trim(); }

void device_level_free(DeviceLevel &level) {
  void *const blocks[4] = {level.borrowed_graph ? nullptr : level.xadj, level.borrowed_graph ? nullptr : level.adj,
                           level.mult, level.map};
  block_give(blocks, 4);
  level = DeviceLevel();
}

void device_level_drop_map(DeviceLevel &level) {
  void *const map = level.map;
  block_give(&map, 1);
  level.map = nullptr;
}

int device_level_upload(DeviceCoarsener *dc, const gosh_csr &host, DeviceLevel &out) {
  device_level_free(out);
  GOSH_TRY_HIP(hipGetDevice(&out.device), "hipGetDevice");
  out.n = host.n;
  out.nnz = out.weight = host.nnz;
  out.xadj_is64 = host.xadj_is64 ? 1 : 0;
  const size_t off_bytes = static_cast<size_t>(host.n + 1) * (host.xadj_is64 ? 8 : 4);
  char *offsets = nullptr;
  if (int rc = persistent(&offsets, off_bytes, "offsets")) return rc;
  out.xadj = offsets;
  if (int rc = persistent(&out.adj, static_cast<size_t>(host.nnz), "adjacency")) return rc;
  if (int rc = device_upload(dc, out.xadj, host.xadj, off_bytes)) return rc;
  if (int rc = device_upload(dc, out.adj, host.adj, static_cast<size_t>(host.nnz) * 4)) return rc;
  return device_level_check(out);
}

int device_level_borrow(const gosh_csr &on_device, DeviceLevel &out) {
  device_level_free(out);
  GOSH_TRY_HIP(hipGetDevice(&out.device), "hipGetDevice");
  out.n = on_device.n;
  out.nnz = out.weight = on_device.nnz;
  out.xadj_is64 = on_device.xadj_is64 ? 1 : 0;
  out.xadj = const_cast<void *>(on_device.xadj);
  out.adj = const_cast<int32_t *>(on_device.adj);
  out.borrowed_graph = true;
  return device_level_check(out);
}

bool is_device_pointer(const void *p) {
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
    (void)hipGetLastError();  // plain pageable memory is unknown to the runtime
    return false;
  }
  return attr.type == hipMemoryTypeDevice;
}

// The kernels follow offsets and neighbour ids without further checks: verify them once.
int device_level_check(DeviceLevel &out) {
  Found *found_dev = nullptr;
  if (int rc = persistent(&found_dev, 1, "check flags")) return rc;
  struct FlagGuard {
    void *block;
    ~FlagGuard() { block_give(&block, 1); }
  } guard{found_dev};
  GOSH_TRY_HIP(hipMemset(found_dev, 0, sizeof(Found)), "clear check flags");
  const int off_blocks = std::min(blocks_for(out.n, 1024), 512);  // whose maxima are atomics on one word
  if (out.xadj_is64)
    hipLaunchKernelGGL(check_offsets_kernel<int64_t>, dim3(off_blocks), dim3(256), 0, nullptr,
                       static_cast<const int64_t *>(out.xadj), out.n, out.nnz, found_dev);
  else
    hipLaunchKernelGGL(check_offsets_kernel<int32_t>, dim3(off_blocks), dim3(256), 0, nullptr,
                       static_cast<const int32_t *>(out.xadj), out.n, out.nnz, found_dev);
  if (out.nnz > 0)
    hipLaunchKernelGGL(check_neighbours_kernel, dim3(blocks_for(out.nnz, 2048)), dim3(256), 0, nullptr, out.adj, out.nnz,
                       out.n, found_dev);
  if (int rc = gosh::check_launch("check_offsets_kernel")) return rc;
  Found found{};
  GOSH_TRY_HIP(hipMemcpy(&found, found_dev, sizeof(found), hipMemcpyDeviceToHost), "read check flags");
  if (found.bad_offsets) return gosh::fail(GOSH_EINVAL, "xadj does not run from 0 to nnz without decreasing");
  if (found.bad_neighbour) return gosh::fail(GOSH_EINVAL, "a neighbour id is outside [0, n)");
  out.top_degree = found.top;
  return GOSH_OK;
}

int device_level_set_map(DeviceLevel &level, const int32_t *map_host) {
  if (level.map == nullptr)
    if (int rc = persistent(&level.map, static_cast<size_t>(level.n), "map")) return rc;
  GOSH_TRY_HIP(hipMemcpy(level.map, map_host, static_cast<size_t>(level.n) * 4, hipMemcpyHostToDevice), "copy map");
  return GOSH_OK;
}

namespace {

// Ascending, so that `from` may be the second half of `to`.
void widen_words(char *to, const char *from, size_t count) {
  for (size_t i = 0; i < count; ++i) {
    uint32_t word;
    memcpy(&word, from + 4 * i, 4);
    const int64_t wide = static_cast<int64_t>(word);
    memcpy(to + 8 * i, &wide, 8);
  }
}

// Copies between pageable host memory and the device through two pinned slots, so that the
// DMA of one piece overlaps the host-side copy of the next, which all threads share (on a
// download that also spreads the page faults of a fresh destination over the threads).
// The runtime's own copy of pageable memory moves 12 GB/s and shares nothing.
struct StagedCopy {
  const int threads;
  char *slots;
  hipEvent_t done[2] = {nullptr, nullptr};  // the DMA that last used slot i
  explicit StagedCopy(const DeviceCoarsener *dc) : threads(dc->threads), slots(staging_take()) {}
  ~StagedCopy() {
    (void)hipStreamSynchronize(nullptr);  // after a failed call a copy may still be using a slot
    for (int i = 0; i < 2; ++i)
      if (done[i]) (void)hipEventDestroy(done[i]);
    staging_give(slots);
  }
  bool available() const { return slots != nullptr; }
  int open() {
    for (int i = 0; i < 2; ++i)
      GOSH_TRY_HIP(hipEventCreateWithFlags(&done[i], hipEventDisableTiming), "create copy event");
    return GOSH_OK;
  }
  char *slot(size_t c) const { return slots + (c & 1) * kStagingBytes; }
  // `to` gets the 32-bit words of `from` as 64-bit ones where `widen` is set.
  void host_copy(char *to, const char *from, size_t bytes, bool widen = false) const {
    const int64_t len = static_cast<int64_t>(bytes);
    const int64_t grain = int64_t(1) << 18;
    const int64_t grains = (len + grain - 1) / grain;
#pragma omp parallel for num_threads(threads) schedule(static)
    for (int64_t g = 0; g < grains; ++g) {
      const size_t part = static_cast<size_t>(std::min(grain, len - g * grain));
      if (widen) widen_words(to + 2 * g * grain, from + g * grain, part / 4);
      else memcpy(to + g * grain, from + g * grain, part);
    }
  }
};

// Pieces of a copy: eight, but none shorter than a megabyte or longer than a slot.
constexpr size_t kStagedFrom = size_t(4) << 20;  // below, one call of the runtime is as fast
size_t piece_bytes_of(size_t bytes) {
  const size_t eighth = ((bytes + 7) / 8 + 4095) / 4096 * 4096;
  return std::min(std::max(eighth, size_t(1) << 20), kStagingBytes);
}

bool is_pinned_host(const void *p) {
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
    (void)hipGetLastError();  // plain pageable memory is unknown to the runtime
    return false;
  }
  return attr.type == hipMemoryTypeHost;
}

}  // namespace

namespace {

// Through the staging, if there is any and it pays: *done says so.
int staged_download(DeviceCoarsener *dc, char *dst, const char *src_dev, size_t bytes, bool widen, bool *done) {
  *done = false;
  if (dc == nullptr || bytes < kStagedFrom) return GOSH_OK;
  StagedCopy q(dc);
  if (!q.available()) return GOSH_OK;
  if (int rc = q.open()) return rc;
  const size_t piece = piece_bytes_of(bytes), pieces = (bytes + piece - 1) / piece;
  auto len = [&](size_t c) { return std::min(piece, bytes - c * piece); };
  auto start = [&](size_t c) -> hipError_t {
    hipError_t e = hipMemcpyAsync(q.slot(c), src_dev + c * piece, len(c), hipMemcpyDeviceToHost, nullptr);
    return e != hipSuccess ? e : hipEventRecord(q.done[c & 1], nullptr);
  };
  GOSH_TRY_HIP(start(0), "start download");
  for (size_t c = 0; c < pieces; ++c) {
    // slot (c + 1) & 1 was emptied in the previous iteration
    if (c + 1 < pieces) GOSH_TRY_HIP(start(c + 1), "start download");
    GOSH_TRY_HIP(hipEventSynchronize(q.done[c & 1]), "wait for download");
    q.host_copy(dst + c * piece * (widen ? 2 : 1), q.slot(c), len(c), widen);
  }
  *done = true;
  return GOSH_OK;
}

}  // namespace

int device_download(DeviceCoarsener *dc, void *dst, const void *src_dev, size_t bytes) {
  if (bytes == 0) return GOSH_OK;
  bool done = false;
  if (int rc = staged_download(dc, static_cast<char *>(dst), static_cast<const char *>(src_dev), bytes, false, &done))
    return rc;
  if (!done) GOSH_TRY_HIP(hipMemcpy(dst, src_dev, bytes, hipMemcpyDeviceToHost), "download");
  return GOSH_OK;
}

int device_download_widened(DeviceCoarsener *dc, int64_t *dst, const void *src_dev, size_t count) {
  if (count == 0) return GOSH_OK;
  char *const to = reinterpret_cast<char *>(dst);
  bool done = false;
  if (int rc = staged_download(dc, to, static_cast<const char *>(src_dev), count * 4, true, &done)) return rc;
  if (done) return GOSH_OK;
  GOSH_TRY_HIP(hipMemcpy(to + count * 4, src_dev, count * 4, hipMemcpyDeviceToHost), "download");
  widen_words(to, to + count * 4, count);
  return GOSH_OK;
}

int device_upload(DeviceCoarsener *dc, void *dst_dev, const void *src, size_t bytes) {
  if (bytes == 0) return GOSH_OK;
  if (dc == nullptr || bytes < kStagedFrom || is_pinned_host(src)) {
    GOSH_TRY_HIP(hipMemcpy(dst_dev, src, bytes, hipMemcpyHostToDevice), "upload");
    return GOSH_OK;
  }
  StagedCopy q(dc);
  if (!q.available()) {
    GOSH_TRY_HIP(hipMemcpy(dst_dev, src, bytes, hipMemcpyHostToDevice), "upload");
    return GOSH_OK;
  }
  if (int rc = q.open()) return rc;
  const size_t piece = piece_bytes_of(bytes), pieces = (bytes + piece - 1) / piece;
  for (size_t c = 0; c < pieces; ++c) {
    const size_t len = std::min(piece, bytes - c * piece);
    // the DMA of piece c - 2 must have drained this slot
    if (c >= 2) GOSH_TRY_HIP(hipEventSynchronize(q.done[c & 1]), "wait for upload");
    q.host_copy(q.slot(c), static_cast<const char *>(src) + c * piece, len);
    GOSH_TRY_HIP(hipMemcpyAsync(static_cast<char *>(dst_dev) + c * piece, q.slot(c), len, hipMemcpyHostToDevice, nullptr),
                 "upload piece");
    GOSH_TRY_HIP(hipEventRecord(q.done[c & 1], nullptr), "record upload");
  }
  GOSH_TRY_HIP(hipStreamSynchronize(nullptr), "finish upload");
  return GOSH_OK;
}

namespace {

template <typename OffT>
int mark_impl(DeviceCoarsener *dc, DeviceLevel &fine, int64_t *n_coarse, bool *done, double *order_ms) {
  const int64_t n = fine.n, nnz = fine.nnz;
  const OffT *xadj = static_cast<const OffT *>(fine.xadj);
  const int32_t *adj = fine.adj;
  *done = false;
  Buffers buf(dc->pool);
  const auto t_order = std::chrono::steady_clock::now();

  // degree order
  uint32_t *keys = nullptr, *keys_sorted = nullptr, *rk = nullptr;
  int32_t *order = nullptr;
  if (int rc = buf.alloc(&keys, static_cast<size_t>(n), "degree keys")) return rc;
  if (int rc = buf.alloc(&keys_sorted, static_cast<size_t>(n), "sorted degree keys")) return rc;
  if (int rc = buf.alloc(&order, static_cast<size_t>(n), "order")) return rc;
  if (int rc = buf.alloc(&rk, static_cast<size_t>(n), "ranks")) return rc;
  const int flat_blocks = blocks_for(n, 256);
  hipLaunchKernelGGL(degree_keys_kernel<OffT>, dim3(flat_blocks), dim3(256), 0, nullptr, xadj, n, fine.top_degree, keys);
  if (int rc = gosh::check_launch("degree_keys_kernel")) return rc;
  {
    // a pass per eight bits: no more of them than the largest degree has
    unsigned bits = 1;
    while (bits < 32 && (fine.top_degree >> bits) != 0) ++bits;
    const rocprim::counting_iterator<int32_t> ids(0);
    size_t temp_bytes = 0;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs<SortConfig>(nullptr, temp_bytes, keys, keys_sorted, ids, order,
                                         static_cast<size_t>(n), 0u, bits, nullptr),
               "degree sort (size query)");
    char *temp = nullptr;
    if (int rc = buf.alloc(&temp, temp_bytes, "sort workspace")) return rc;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs<SortConfig>(temp, temp_bytes, keys, keys_sorted, ids, order,
                                         static_cast<size_t>(n), 0u, bits, nullptr),
               "degree sort");
    buf.release(temp);  // what takes it up again is on the same stream
  }
  hipLaunchKernelGGL(rank_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, keys_sorted, order, n, nnz, fine.top_degree,
                     rk);
  if (int rc = gosh::check_launch("rank_kernel")) return rc;
  GOSH_TRY_HIP(hipDeviceSynchronize(), "ranks");
  buf.release(keys);
  buf.release(keys_sorted);
  *order_ms = ms_since(t_order);

  // first classification
  int32_t *status = nullptr, *pending = nullptr, *still = nullptr;
  unsigned long long *counters = nullptr;  // sizes of the two pending lists
  if (int rc = buf.alloc(&status, static_cast<size_t>(n), "status")) return rc;
  if (int rc = buf.alloc(&pending, static_cast<size_t>(n), "pending list")) return rc;
  if (int rc = buf.alloc(&still, static_cast<size_t>(n), "pending list")) return rc;
  if (int rc = buf.alloc(&counters, 2, "pending counters")) return rc;
  GOSH_TRY_HIP(hipMemset(counters, 0, 16), "clear counters");
  const int lanes = lanes_per_vertex(n, nnz);
  const auto classify = lanes == 4    ? classify_kernel<OffT, 4>
                        : lanes == 8  ? classify_kernel<OffT, 8>
                        : lanes == 16 ? classify_kernel<OffT, 16>
                        : lanes == 32 ? classify_kernel<OffT, 32>
                                      : classify_kernel<OffT, 64>;
  const auto join = lanes == 4    ? join_kernel<OffT, 4>
                    : lanes == 8  ? join_kernel<OffT, 8>
                    : lanes == 16 ? join_kernel<OffT, 16>
                    : lanes == 32 ? join_kernel<OffT, 32>
                                  : join_kernel<OffT, 64>;
  const int group_blocks = blocks_for(n, 256 / lanes);
  // a wavefront walks enough vertices for its turns at the list to be few, where there are that many
  hipLaunchKernelGGL(classify, dim3(std::min(group_blocks, 2048)), dim3(256), 0, nullptr, xadj, adj, rk, n, status,
                     pending, counters);
  if (int rc = gosh::check_launch("classify_kernel")) return rc;
  unsigned long long count = 0;
  GOSH_TRY_HIP(hipMemcpy(&count, counters, 8, hipMemcpyDeviceToHost), "read pending count");

  // rounds: each decides at least the first pending vertex of the order, usually most
  const int kMaxRounds = 256;
  int which = 0;  // counters[which] is the size of `pending`
  for (int round = 0; count > 0; ++round) {
    if (round == kMaxRounds) return GOSH_OK;  // *done stays false
    GOSH_TRY_HIP(hipMemset(counters + (which ^ 1), 0, 8), "clear counter");
    hipLaunchKernelGGL(round_kernel<OffT>, dim3(blocks_for(static_cast<int64_t>(count), 4)), dim3(256), 0, nullptr,
                       xadj, adj, rk, status, pending, static_cast<int64_t>(count), still, counters + (which ^ 1));
    if (int rc = gosh::check_launch("round_kernel")) return rc;
    unsigned long long left = 0;
    GOSH_TRY_HIP(hipMemcpy(&left, counters + (which ^ 1), 8, hipMemcpyDeviceToHost), "read pending count");
    // a long chain: a few vertices per round would take forever
    if (round >= 16 && left > 4096 && left * 100 > count * 99) return GOSH_OK;
    std::swap(pending, still);
    which ^= 1;
    count = left;
  }
  buf.release(pending);
  buf.release(still);

  // number the hubs in the order
  int32_t *flags = nullptr, *index = nullptr;
  if (int rc = buf.alloc(&flags, static_cast<size_t>(n), "hub flags")) return rc;
  if (int rc = buf.alloc(&index, static_cast<size_t>(n), "hub numbers")) return rc;
  hipLaunchKernelGGL(hub_flags_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, status, order, n, flags);
  if (int rc = gosh::check_launch("hub_flags_kernel")) return rc;
  {
    size_t temp_bytes = 0;
    GOSH_TRY_HIP(rocprim::exclusive_scan(nullptr, temp_bytes, flags, index, int32_t(0), static_cast<size_t>(n),
                                       rocprim::plus<int32_t>(), nullptr),
               "hub scan (size query)");
    char *temp = nullptr;
    if (int rc = buf.alloc(&temp, temp_bytes, "scan workspace")) return rc;
    GOSH_TRY_HIP(rocprim::exclusive_scan(temp, temp_bytes, flags, index, int32_t(0), static_cast<size_t>(n),
                                       rocprim::plus<int32_t>(), nullptr),
               "hub scan");
    buf.release(temp);
  }
  if (fine.map == nullptr)
    if (int rc = persistent(&fine.map, static_cast<size_t>(n), "map")) return rc;
  hipLaunchKernelGGL(number_hubs_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, flags, index, order, n, fine.map,
                     counters);
  if (int rc = gosh::check_launch("number_hubs_kernel")) return rc;
  hipLaunchKernelGGL(join, dim3(group_blocks), dim3(256), 0, nullptr, xadj, adj, rk, status, order, n, fine.map);
  if (int rc = gosh::check_launch("join_kernel")) return rc;
  GOSH_TRY_HIP(hipMemcpy(&count, counters, 8, hipMemcpyDeviceToHost), "read hub count");  // and waits for the marking
  *n_coarse = static_cast<int64_t>(count);
  *done = true;
  return GOSH_OK;
}

}  // namespace

int device_mark(DeviceCoarsener *dc, DeviceLevel &fine, int64_t *n_coarse, bool *done, double *order_ms) {
  if (dc == nullptr || !fine.present() || fine.n < 1) return gosh::fail(GOSH_EINVAL, "device level is missing");
  return fine.xadj_is64 ? mark_impl<int64_t>(dc, fine, n_coarse, done, order_ms)
                        : mark_impl<int32_t>(dc, fine, n_coarse, done, order_ms);
}

}  // namespace gosh
