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
// back the kept staging).  A block is kept only after the device has finished what was queued on it, so whoever gets it next may
// use it on any stream.
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

// One block of block_give; `idle` is the device known to have finished its queues.
void give_one(Store &s, void *p, int *idle) {
  const auto known = s.handed_out.find(p);
  if (known == s.handed_out.end()) {
    (void)hipFree(p);
    return;
  }
  const Block b = known->second;
  s.handed_out.erase(known);
  if (*idle != b.device && hipSetDevice(b.device) == hipSuccess && hipDeviceSynchronize() == hipSuccess) *idle = b.device;
  const size_t limit = *idle == b.device ? kept_limit(s, b.device) : 0;
  if (b.bytes <= limit) {
    size_t have = kept_bytes(s, b.device);
    for (size_t k = 0; k < s.kept.size() && have + b.bytes > limit;) {
      if (s.kept[k].device != b.device) {
        ++k;
        continue;
      }
      have -= s.kept[k].bytes;
      (void)hipFree(s.kept[k].p);
      s.kept.erase(s.kept.begin() + static_cast<std::ptrdiff_t>(k));
    }
    try {
      s.kept.push_back(b);
      return;
    } catch (const std::bad_alloc &) {
    }
  }
  (void)hipFree(p);
}

}  // namespace

void block_give(void *const *blocks, size_t count) {
  bool any = false;
  for (size_t i = 0; i < count; ++i) any |= blocks[i] != nullptr;
  if (!any) return;
  Store &s = store();
  std::lock_guard<std::mutex> lock(s.mutex);
  int current = -1, idle = -1;
  if (hipGetDevice(&current) != hipSuccess) current = -1;
  for (size_t i = 0; i < count; ++i)
    if (blocks[i] != nullptr) give_one(s, blocks[i], &idle);
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
