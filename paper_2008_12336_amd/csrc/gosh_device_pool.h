// Device memory of a coarsening run and what its translation units share.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "gosh_common.h"

namespace gosh {

// Device blocks recycled over the levels of one run: hipMalloc and hipFree of gigabyte
// blocks cost more than the kernels of a small level.  Levels only shrink, so the blocks
// of the first level serve all later ones (best fit).
struct Pool {
  struct Block {
    void *p;
    size_t bytes;
    bool busy;
  };
  std::vector<Block> blocks;
  ~Pool() { trim(); }
  void trim() {
    for (Block &b : blocks) (void)hipFree(b.p);
    blocks.clear();
  }
  void *take(size_t bytes) {
    // best fit, but a small request never occupies a block that a large one will want
    const size_t too_big = std::max<size_t>(bytes * 8, size_t(64) << 20);
    Block *best = nullptr;
    for (Block &b : blocks)
      if (!b.busy && b.bytes >= bytes && b.bytes <= too_big && (best == nullptr || b.bytes < best->bytes))
        best = &b;
    if (best != nullptr) {
      best->busy = true;
      return best->p;
    }
    void *p = nullptr;
    if (hipMalloc(&p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    blocks.push_back(Block{p, bytes, true});
    return p;
  }
  void give(void *p) {
    for (Block &b : blocks)
      if (b.p == p) b.busy = false;
  }
};

// The blocks one call holds; they go back to the pool on return.
struct Buffers {
  Pool &pool;
  std::vector<void *> ptrs;
  explicit Buffers(Pool &pl) : pool(pl) {}
  ~Buffers() {
    for (void *p : ptrs)
      if (p) pool.give(p);
  }
  template <typename T>
  int alloc(T **out, size_t count, const char *what) {
    const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    void *p = pool.take(bytes);
    if (p == nullptr) return fail(GOSH_ENOMEM, "cannot allocate %zu device bytes for %s", bytes, what);
    ptrs.push_back(p);
    *out = static_cast<T *>(p);
    return GOSH_OK;
  }
  void release(void *p) {
    for (void *&q : ptrs)
      if (q == p) {
        pool.give(q);
        q = nullptr;
      }
  }
};

inline int blocks_for(int64_t items, int per_block) {
  int64_t b = (items + per_block - 1) / per_block;
  return static_cast<int>(std::min<int64_t>(std::max<int64_t>(b, 1), 1 << 16));
}

// Exact-sized block that outlives the run (a level's array).
template <typename T>
int persistent(T **out, size_t count, const char *what) {
  void *p = nullptr;
  const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
  if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(GOSH_ENOMEM, "cannot allocate %zu device bytes for %s", bytes, what);
  }
  *out = static_cast<T *>(p);
  return GOSH_OK;
}

struct DeviceCoarsener {
  Pool pool;
  int threads = 1;
  // Two pinned staging slots for large downloads, made on first use and kept.  The copy
  // stream is NOT kept: a process has few hardware queues, and an idle stream of ours
  // would make the streams of a later training call share one.
  static constexpr size_t kSlotBytes = size_t(64) << 20;
  char *slot[2] = {nullptr, nullptr};
  ~DeviceCoarsener() {
    for (int i = 0; i < 2; ++i)
      if (slot[i]) (void)hipHostFree(slot[i]);
  }
};

}  // namespace gosh
