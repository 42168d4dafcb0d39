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

namespace {

using gosh::blocks_for;
using gosh::persistent;

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

// key = 2^31 - 1 - degree: ascending keys are descending degrees; stable => ties by id.
template <typename OffT>
__global__ __launch_bounds__(256) void degree_keys_kernel(const OffT *__restrict__ xadj, int64_t n,
                                                          uint32_t *__restrict__ keys,
                                                          int32_t *__restrict__ ids) {
  for (int64_t v = blockIdx.x * 256LL + threadIdx.x; v < n; v += gridDim.x * 256LL) {
    keys[v] = kRankMask - static_cast<uint32_t>(xadj[v + 1] - xadj[v]);
    ids[v] = static_cast<int32_t>(v);
  }
}

// rk[order[t]] = t, with the high bit set when the degree exceeds the mean degree
// (deg * n > nnz, exact in 64-bit integers).
__global__ __launch_bounds__(256) void rank_kernel(const uint32_t *__restrict__ sorted_keys,
                                                   const int32_t *__restrict__ order, int64_t n,
                                                   int64_t nnz, uint32_t *__restrict__ rk) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL) {
    const int64_t deg = static_cast<int64_t>(kRankMask - sorted_keys[t]);
    rk[order[t]] = static_cast<uint32_t>(t) | (deg * n > nnz ? kHighBit : 0u);
  }
}

// Lanes per vertex of classify_kernel and join_kernel.  Both look at the entries of vertices of at most
// mean degree, after a chain of dependent reads (rank, offsets, entry, rank or status), and are bound by
// that chain: with a wavefront per vertex most lanes have no entry and few vertices are in flight.  Fewer
// lanes pay until the vertices no longer fill the device.  us with 64 / 16 / 8 / 4 lanes, both kernels:
//   4.2 M vertices, R-MAT, mean degree 30: 1,430 / 868 / 774 / 724    its next level, mean above 100: 421 / 152 / 109 / 84
//   2.1 M, power law: 2,200 / 1,720 / 1,465 / 1,160                   1 M, uniform: 440 / 344 / 294 / 238
//   the last one's next levels, each about a tenth: 288 / 192 / 177 / 196, 82 / 59 / 68 / 98, 24 / 50 / 80 / 140
inline int lanes_per_vertex(int64_t n, int64_t nnz) {
  int lanes = n >= (int64_t{1} << 20) ? 4 : n >= (int64_t{1} << 16) ? 8 : n >= (int64_t{1} << 13) ? 16 : 64;
  while (lanes < 64 && lanes * 64 * n < nnz) lanes *= 2;  // at most 64 entries of a mean row to a lane
  return lanes;
}

// First classification, LANES lanes per vertex: needs no knowledge of other decisions.
template <typename OffT, int LANES>
__global__ __launch_bounds__(256) void classify_kernel(const OffT *__restrict__ xadj,
                                                       const int32_t *__restrict__ adj,
                                                       const uint32_t *__restrict__ rk, int64_t n,
                                                       int32_t *__restrict__ status,
                                                       int32_t *__restrict__ pending,
                                                       unsigned long long *__restrict__ pending_count) {
  constexpr int kPerWave = 64 / LANES;
  const int lane = threadIdx.x & 63, gl = lane & (LANES - 1), group = lane & ~(LANES - 1);
  for (int64_t base = first_wave() * kPerWave; base < n; base += wave_count() * kPerWave) {
    const int64_t v = base + lane / LANES;
    const uint32_t r = v < n ? rk[v] : kHighBit;
    bool high_neighbour = false, predecessor = false;
    if (!(r & kHighBit)) {
      const int64_t begin = static_cast<int64_t>(xadj[v]), end = static_cast<int64_t>(xadj[v + 1]);
      for (int64_t e = begin + gl; e < end; e += LANES) {
        const uint32_t ru = rk[adj[e]];
        high_neighbour |= (ru & kHighBit) != 0;
        predecessor |= (ru & kRankMask) < r;
      }
    }
    const uint64_t of_group = ~uint64_t{0} >> (64 - LANES) << group;
    const bool taken = (__ballot(high_neighbour) & of_group) != 0;
    const bool undecided = !taken && (__ballot(predecessor) & of_group) != 0;
    if (gl == 0 && v < n) status[v] = taken ? kTaken : undecided ? kUndecided : kHub;
    // one atomic per wavefront: thousands on one word follow one another
    const bool lists = gl == 0 && v < n && undecided;
    const uint64_t listed = __ballot(lists);
    if (listed != 0) {
      const int leader = __builtin_ctzll(listed);
      unsigned long long at = 0;
      if (lane == leader) at = atomicAdd(pending_count, static_cast<unsigned long long>(__popcll(listed)));
      at = __shfl(at, leader, 64) + __popcll(listed & ((uint64_t{1} << lane) - 1));
      if (lists) pending[at] = static_cast<int32_t>(v);
    }
  }
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
                                                          int32_t *__restrict__ map) {
  for (int64_t t = blockIdx.x * 256LL + threadIdx.x; t < n; t += gridDim.x * 256LL)
    if (flags[t]) map[order[t]] = index[t];
}

// Every taken vertex joins its first hub in the order, LANES lanes per vertex.  The
// hubs' own entries of map (read here) were written by the launch before this one; this
// launch writes only entries of taken vertices.
template <typename OffT, int LANES>
__global__ __launch_bounds__(256) void join_kernel(const OffT *__restrict__ xadj,
                                                   const int32_t *__restrict__ adj,
                                                   const uint32_t *__restrict__ rk,
                                                   const int32_t *__restrict__ status,
                                                   const int32_t *__restrict__ order, int64_t n,
                                                   int32_t *map) {
  constexpr int kPerWave = 64 / LANES;
  const int lane = threadIdx.x & 63, gl = lane & (LANES - 1);
  for (int64_t base = first_wave() * kPerWave; base < n; base += wave_count() * kPerWave) {
    const int64_t v = base + lane / LANES;
    uint32_t best = kRankMask;
    if (v < n && status[v] == kTaken) {
      const uint32_t r = rk[v];
      const int64_t begin = static_cast<int64_t>(xadj[v]), end = static_cast<int64_t>(xadj[v + 1]);
      for (int64_t e = begin + gl; e < end; e += LANES) {
        const int32_t u = adj[e];
        const uint32_t ru = rk[u] & kRankMask;
        if (ru < r && ru < best && status[u] == kHub) best = ru;
      }
    }
    for (int offset = LANES / 2; offset > 0; offset >>= 1) best = min(best, __shfl_xor(best, offset, 64));
    // a taken vertex has a hub before it, so best is a valid position; the guard keeps a
    // broken invariant from turning into a wild read
    if (gl == 0 && best < static_cast<uint32_t>(n)) map[v] = map[order[best]];
  }
}

// Shape checks before any kernel follows the offsets or the neighbour ids: *bad becomes
// nonzero if the offsets do not run from 0 to nnz without decreasing, or (second kernel)
// if a neighbour id is outside [0, n).
template <typename OffT>
__global__ __launch_bounds__(256) void check_offsets_kernel(const OffT *__restrict__ xadj, int64_t n,
                                                            int64_t nnz, int32_t *__restrict__ bad) {
  for (int64_t v = blockIdx.x * 256LL + threadIdx.x; v < n; v += gridDim.x * 256LL) {
    const int64_t lo = static_cast<int64_t>(xadj[v]), hi = static_cast<int64_t>(xadj[v + 1]);
    if (lo > hi || lo < 0 || hi > nnz || (v == 0 && lo != 0) || (v == n - 1 && hi != nnz)) *bad = 1;
  }
}

__global__ __launch_bounds__(256) void check_neighbours_kernel(const int32_t *__restrict__ adj, int64_t nnz,
                                                               int64_t n, int32_t *__restrict__ bad) {
  for (int64_t e = blockIdx.x * 256LL + threadIdx.x; e < nnz; e += gridDim.x * 256LL)
    if (adj[e] < 0 || adj[e] >= n) *bad = 1;
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
int device_level_check(const DeviceLevel &out) {
  const gosh_csr host{out.n, out.nnz, out.xadj, out.adj, out.xadj_is64};
  int32_t *bad_dev = nullptr;
  if (int rc = persistent(&bad_dev, 1, "check flag")) return rc;
  struct FlagGuard {
    int32_t *p;
    ~FlagGuard() {
      void *const block = p;
      block_give(&block, 1);
    }
  } guard{bad_dev};
  int32_t bad = 0;
  GOSH_TRY_HIP(hipMemset(bad_dev, 0, 4), "clear check flag");
  const int off_blocks = blocks_for(host.n, 256);
  if (host.xadj_is64)
    hipLaunchKernelGGL(check_offsets_kernel<int64_t>, dim3(off_blocks), dim3(256), 0, nullptr,
                       static_cast<const int64_t *>(out.xadj), out.n, out.nnz, bad_dev);
  else
    hipLaunchKernelGGL(check_offsets_kernel<int32_t>, dim3(off_blocks), dim3(256), 0, nullptr,
                       static_cast<const int32_t *>(out.xadj), out.n, out.nnz, bad_dev);
  if (int rc = gosh::check_launch("check_offsets_kernel")) return rc;
  GOSH_TRY_HIP(hipMemcpy(&bad, bad_dev, 4, hipMemcpyDeviceToHost), "read check flag");
  if (bad) return gosh::fail(GOSH_EINVAL, "xadj does not run from 0 to nnz without decreasing");
  if (host.nnz > 0) {
    hipLaunchKernelGGL(check_neighbours_kernel, dim3(blocks_for(host.nnz, 256)), dim3(256), 0, nullptr, out.adj,
                       out.nnz, out.n, bad_dev);
    if (int rc = gosh::check_launch("check_neighbours_kernel")) return rc;
    GOSH_TRY_HIP(hipMemcpy(&bad, bad_dev, 4, hipMemcpyDeviceToHost), "read check flag");
    if (bad) return gosh::fail(GOSH_EINVAL, "a neighbour id is outside [0, n)");
  }
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
  int32_t *ids = nullptr, *order = nullptr;
  if (int rc = buf.alloc(&keys, static_cast<size_t>(n), "degree keys")) return rc;
  if (int rc = buf.alloc(&keys_sorted, static_cast<size_t>(n), "sorted degree keys")) return rc;
  if (int rc = buf.alloc(&ids, static_cast<size_t>(n), "vertex ids")) return rc;
  if (int rc = buf.alloc(&order, static_cast<size_t>(n), "order")) return rc;
  if (int rc = buf.alloc(&rk, static_cast<size_t>(n), "ranks")) return rc;
  const int flat_blocks = blocks_for(n, 256);
  hipLaunchKernelGGL(degree_keys_kernel<OffT>, dim3(flat_blocks), dim3(256), 0, nullptr, xadj, n, keys, ids);
  if (int rc = gosh::check_launch("degree_keys_kernel")) return rc;
  {
    size_t temp_bytes = 0;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs(nullptr, temp_bytes, keys, keys_sorted, ids, order,
                                         static_cast<size_t>(n), 0u, 31u, nullptr),
               "degree sort (size query)");
    char *temp = nullptr;
    if (int rc = buf.alloc(&temp, temp_bytes, "sort workspace")) return rc;
    GOSH_TRY_HIP(rocprim::radix_sort_pairs(temp, temp_bytes, keys, keys_sorted, ids, order,
                                         static_cast<size_t>(n), 0u, 31u, nullptr),
               "degree sort");
    GOSH_TRY_HIP(hipDeviceSynchronize(), "degree sort");
    buf.release(temp);
  }
  hipLaunchKernelGGL(rank_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, keys_sorted, order, n, nnz, rk);
  if (int rc = gosh::check_launch("rank_kernel")) return rc;
  GOSH_TRY_HIP(hipDeviceSynchronize(), "ranks");
  buf.release(keys);
  buf.release(keys_sorted);
  buf.release(ids);
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
  hipLaunchKernelGGL(classify, dim3(group_blocks), dim3(256), 0, nullptr, xadj, adj, rk, n, status, pending, counters);
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
    GOSH_TRY_HIP(hipDeviceSynchronize(), "hub scan");
    buf.release(temp);
  }
  int32_t last_flag = 0, last_index = 0;
  GOSH_TRY_HIP(hipMemcpy(&last_flag, flags + (n - 1), 4, hipMemcpyDeviceToHost), "read hub count");
  GOSH_TRY_HIP(hipMemcpy(&last_index, index + (n - 1), 4, hipMemcpyDeviceToHost), "read hub count");
  if (fine.map == nullptr)
    if (int rc = persistent(&fine.map, static_cast<size_t>(n), "map")) return rc;
  hipLaunchKernelGGL(number_hubs_kernel, dim3(flat_blocks), dim3(256), 0, nullptr, flags, index, order, n, fine.map);
  if (int rc = gosh::check_launch("number_hubs_kernel")) return rc;
  hipLaunchKernelGGL(join, dim3(group_blocks), dim3(256), 0, nullptr, xadj, adj, rk, status, order, n, fine.map);
  if (int rc = gosh::check_launch("join_kernel")) return rc;
  GOSH_TRY_HIP(hipDeviceSynchronize(), "marking");
  *n_coarse = static_cast<int64_t>(last_flag) + last_index;
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
