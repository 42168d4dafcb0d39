// Device blocks of freed hierarchies, kept for the next one.
//
// Releasing gigabytes to the driver is not free: it clears them in the background at some
// 33 GB/s, and an allocation that needs memory it has not cleared yet waits.  A program that
// coarsens one graph after another met such waits of up to seconds (a 4 M-vertex graph whose
// hierarchy takes 16 ms: 100 to 240 ms per call on average; with kept blocks 13 ms).
//
// Kept blocks are bounded per device (kept_limit), handed out to any thread, given back when an
// allocation of this library fails, when more would be kept than the bound (oldest first), and
// on request (block_trim, behind gosh_hierarchy_trim_scratch and _release_device, which also gives
// back the kept staging).  A block is kept only after everything that uses it has finished -- the device is waited for,
// unless the caller has waited for its own streams -- so whoever gets it next may use it on any stream.  Nobody
// waits for a device with the mutex held, except where an allocation fails or on request.
#include <hip/hip_runtime.h>

#include <deque>
#include <mutex>
#include <new>
#include <unordered_map>

#include "gosh_device_pool.h"

namespace gosh {
namespace {

struct Block {
  void *p;
  size_t bytes;
  int device;
};
constexpr int kStagingKept = 2, kMaxDevices = 64;
struct Store {
  std::mutex mutex;
  char *staging[kStagingKept] = {};
  int staging_kept = 0;
  std::unordered_map<void *, Block> handed_out;
  std::deque<Block> kept;  // oldest first
  size_t limit[kMaxDevices] = {};  // 0: not known yet
};
// Never destroyed: hierarchies may be freed during the end of the process.
Store &store() {
  static Store *s = new Store();
  return *s;
}

// A 64th of the device's memory.
size_t kept_limit(Store &s, int device) {
  if (device < 0 || device >= kMaxDevices) return 0;
  if (s.limit[device] != 0) return s.limit[device];
  size_t free_bytes = 0, total = 0;
  if (hipMemGetInfo(&free_bytes, &total) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return s.limit[device] = total / 64;
}

size_t kept_bytes(const Store &s, int device) {
  size_t sum = 0;
  for (const Block &b : s.kept)
    if (b.device == device) sum += b.bytes;
  return sum;
}

// Sixteen sizes per power of two, so that the blocks of one graph fit the next of its size.
size_t rounded(size_t bytes) {
  size_t step = 256;
  while (step * 32 <= bytes) step *= 2;
  return (bytes + step - 1) / step * step;
}

// Frees the kept blocks of a device; false if there were none.  The caller holds the mutex.
bool drop_kept(Store &s, int device) {
  bool any = false;
  for (size_t i = 0; i < s.kept.size();) {
    if (s.kept[i].device == device) {
      (void)hipFree(s.kept[i].p);
      s.kept.erase(s.kept.begin() + static_cast<std::ptrdiff_t>(i));
      any = true;
    } else {
      ++i;
    }
  }
  return any;
}

}  // namespace

hipError_t device_malloc_bytes(void **p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) return e;
  (void)hipGetLastError();
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return e;
  Store &s = store();
  {
    std::lock_guard<std::mutex> lock(s.mutex);
    if (!drop_kept(s, device)) return e;
  }
  e = hipMalloc(p, bytes);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

void *block_take(size_t bytes) {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return nullptr;
  Store &s = store();
  void *p = nullptr;
  try {
    {
      std::lock_guard<std::mutex> lock(s.mutex);
      auto best = s.kept.end();
      for (auto b = s.kept.begin(); b != s.kept.end(); ++b)
        if (b->device == device && b->bytes >= bytes && b->bytes <= bytes + bytes / 4 + (size_t(64) << 10) &&
            (best == s.kept.end() || b->bytes < best->bytes))
          best = b;
      if (best != s.kept.end()) {
        const Block b = *best;
        s.handed_out[b.p] = b;
        s.kept.erase(best);
        return b.p;
      }
    }
    size_t got = rounded(bytes);
    if (device_malloc(&p, got) != hipSuccess) {
      got = bytes;
      if (device_malloc(&p, got) != hipSuccess) return nullptr;
    }
    std::lock_guard<std::mutex> lock(s.mutex);
    s.handed_out[p] = Block{p, got, device};
    return p;
  } catch (const std::bad_alloc &) {  // no host memory to remember the block by
    if (p) (void)hipFree(p);
    return nullptr;
  }
}

namespace {

// One block of block_give, on a device whose queues have finished if `idle`.  What is freed waits for its device:
// without the mutex.
void give_one(Store &s, void *p, bool known_idle, uint64_t idle_devices) {
  std::unique_lock<std::mutex> lock(s.mutex);
  const auto known = s.handed_out.find(p);
  if (known == s.handed_out.end()) {
    lock.unlock();
    (void)hipFree(p);
    return;
  }
  const Block b = known->second;
  s.handed_out.erase(known);
  const bool idle = known_idle || (b.device >= 0 && b.device < kMaxDevices && (idle_devices >> b.device & 1) != 0);
  (void)hipSetDevice(b.device);  // whose memory the limit is a part of; block_give restores the current one
  const size_t limit = idle ? kept_limit(s, b.device) : 0;
  while (b.bytes <= limit && kept_bytes(s, b.device) + b.bytes > limit) {
    auto oldest = s.kept.begin();
    while (oldest->device != b.device) ++oldest;  // there is one: the block alone is within the limit
    void *const old = oldest->p;
    s.kept.erase(oldest);
    lock.unlock();
    (void)hipFree(old);
    lock.lock();
  }
  if (b.bytes <= limit) {
    try {
      s.kept.push_back(b);
      return;
    } catch (const std::bad_alloc &) {
    }
  }
  lock.unlock();
  (void)hipFree(p);
}

}  // namespace

void block_give(void *const *blocks, size_t count, bool idle) {
  bool any = false;
  for (size_t i = 0; i < count; ++i) any |= blocks[i] != nullptr;
  if (!any) return;
  Store &s = store();
  int current = -1;
  if (hipGetDevice(&current) != hipSuccess) current = -1;
  uint64_t devices = 0, finished = 0;  // of the blocks; those whose queues have finished
  static_assert(kMaxDevices == 64, "a bit per device");
  if (!idle) {
    {
      std::lock_guard<std::mutex> lock(s.mutex);
      for (size_t i = 0; i < count; ++i) {
        const auto known = blocks[i] != nullptr ? s.handed_out.find(blocks[i]) : s.handed_out.end();
        if (known != s.handed_out.end() && known->second.device >= 0 && known->second.device < kMaxDevices)
          devices |= uint64_t{1} << known->second.device;
      }
    }
    for (int device = 0; device < kMaxDevices; ++device)
      if ((devices >> device & 1) != 0 && hipSetDevice(device) == hipSuccess && hipDeviceSynchronize() == hipSuccess)
        finished |= uint64_t{1} << device;
  }
  for (size_t i = 0; i < count; ++i)
    if (blocks[i] != nullptr) give_one(s, blocks[i], idle, finished);
  if (current >= 0) (void)hipSetDevice(current);
}

void block_trim() {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) {
    (void)hipGetLastError();  // a host-built hierarchy on a machine without a device
    return;
  }
  Store &s = store();
  std::lock_guard<std::mutex> lock(s.mutex);
  (void)drop_kept(s, device);
  while (s.staging_kept > 0) (void)hipHostFree(s.staging[--s.staging_kept]);
}

size_t block_kept() {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return 0;
  Store &s = store();
  std::lock_guard<std::mutex> lock(s.mutex);
  return kept_bytes(s, device);
}

char *staging_take() {
  if (denied(kDenyStaging)) return nullptr;
  Store &s = store();
  {
    std::lock_guard<std::mutex> lock(s.mutex);
    if (s.staging_kept > 0) return s.staging[--s.staging_kept];
  }
  void *p = nullptr;
  if (hipHostMalloc(&p, 2 * kStagingBytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return static_cast<char *>(p);
}

void staging_give(char *both) {
  if (both == nullptr) return;
  Store &s = store();
  {
    std::lock_guard<std::mutex> lock(s.mutex);
    if (s.staging_kept < kStagingKept) {
      s.staging[s.staging_kept++] = both;
      return;
    }
  }
  (void)hipHostFree(both);
}

}  // namespace gosh
