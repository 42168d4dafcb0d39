// The store of device blocks (gosh_device_pool) against a runtime that only keeps books: what is
// handed out, kept and given back, with every host allocation failing in turn.  No GPU.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <set>
#include <thread>

#include "gosh_device_pool.h"

namespace {
std::map<void *, size_t> device_blocks;
std::set<void *> pinned;
size_t device_total = size_t(64) << 20;
int64_t allocations_left = -1;  // -1: no limit
int waits = 0;         // for the device
bool probing = false;  // waits and frees, which wait too, must leave the store to other threads

[[noreturn]] void broken(const char *what) {
  std::printf("broken: %s\n", what);
  std::exit(1);
}
void expect(bool ok, const char *what) {
  if (!ok) broken(what);
}
size_t device_used() {
  size_t sum = 0;
  for (const auto &b : device_blocks) sum += b.second;
  return sum;
}
void *plain(size_t bytes) {
  void *p = std::malloc(bytes ? bytes : 1);
  if (p == nullptr) std::abort();
  return p;
}
// The books of the runtime are not the library's allocations.
struct Unlimited {
  int64_t left = allocations_left;
  Unlimited() { allocations_left = -1; }
  ~Unlimited() { allocations_left = left; }
};
void leave_the_store_to_others();
}  // namespace

void *operator new(size_t bytes) {
  if (allocations_left == 0) throw std::bad_alloc();
  if (allocations_left > 0) --allocations_left;
  return plain(bytes);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
  Unlimited u;
  if (device_used() + bytes > device_total) return hipErrorOutOfMemory;
  *p = plain(16);
  device_blocks[*p] = bytes;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  Unlimited u;
  leave_the_store_to_others();
  if (p != nullptr && device_blocks.erase(p) != 1) broken("freed what is no block");
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t, unsigned) {
  Unlimited u;
  *p = plain(16);
  pinned.insert(*p);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  Unlimited u;
  if (pinned.erase(p) != 1) broken("freed what is not pinned");
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total) {
  *free_bytes = device_total - device_used();
  *total = device_total;
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  ++waits;
  leave_the_store_to_others();
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

namespace gosh {
int fail(int code, const char *, ...) { return code; }
int64_t &seam(Seam) {
  static int64_t none = 0;
  return none;
}
}  // namespace gosh

namespace {
void leave_the_store_to_others() {
  if (!probing) return;
  Unlimited u;
  std::atomic<bool> done{false};
  std::thread other([&] {
    (void)gosh::block_kept();
    done = true;
  });
  for (int i = 0; i < 2000 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  if (!done) {
    std::printf("broken: the store is held while the device is waited for\n");
    std::fflush(stdout);
    std::_Exit(1);
  }
  other.join();
}

// A run like that of a hierarchy: scratch of several levels, arrays that outlive it, all given back.
void run() {
  gosh::Pool pool;
  void *arrays[2] = {};
  for (int i = 0; i < 200; ++i)
    if (pool.take(size_t(i % 7 + 1) << 10) == nullptr) break;
  {
    gosh::Buffers buf(pool);
    char *p = nullptr;
    for (int i = 0; i < 20; ++i) (void)buf.alloc(&p, size_t(100) << i % 5, "scratch");
  }
  arrays[0] = gosh::block_take(300 << 10);
  arrays[1] = gosh::block_take(5 << 10);
  gosh::block_give(arrays, 2);
}
}  // namespace

int main() {
  const size_t bound = device_total / 64;
  run();
  expect(device_used() > 0 && gosh::block_kept() == device_used() && device_used() <= bound, "kept blocks are bounded");
  char *s[3];
  for (char *&x : s) x = gosh::staging_take();
  for (char *x : s) gosh::staging_give(x);
  expect(pinned.size() == 2, "two pairs of staging are kept");
  gosh::block_trim();
  expect(device_blocks.empty() && gosh::block_kept() == 0, "a trim gives every block back");
  expect(pinned.empty(), "a trim gives the staging back");
  // an allocation of the library that would fail has the kept blocks back first
  void *p = gosh::block_take(200 << 10);
  gosh::block_give(&p, 1);
  expect(gosh::block_kept() > 0, "kept");
  void *all = nullptr;
  expect(gosh::device_malloc(&all, device_total - 1024) == hipSuccess, "kept blocks make room");
  (void)hipFree(all);
  // every host allocation of a run fails in turn: nothing ends the process, nothing is lost
  for (int64_t n = 0; n < 400; ++n) {
    allocations_left = n;
    try {
      run();
    } catch (const std::bad_alloc &) {
    }
    allocations_left = -1;
    expect(gosh::block_kept() == device_used(), "what is not kept has been freed");
    gosh::block_trim();
    expect(device_blocks.empty(), "blocks are lost after a failed host allocation");
  }
  // three blocks, two of which are kept: nobody waits with the store held, and not at all for idle blocks
  void *blocks[3];
  for (void *&b : blocks) b = gosh::block_take(400 << 10);
  probing = true;
  waits = 0;
  gosh::block_give(blocks, 3);
  expect(waits == 1 && device_blocks.size() == 2, "one wait for the blocks of a device, the oldest goes");
  probing = false;
  for (int i = 0; i < 2; ++i) blocks[i] = gosh::block_take(400 << 10);
  gosh::block_give(blocks, 2, true);
  expect(waits == 1 && device_blocks.size() == 2 && gosh::block_kept() == device_used(), "idle blocks are kept without a wait");
  gosh::block_trim();
  std::printf("pool ok\n");
  return 0;
}
