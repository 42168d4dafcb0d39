// Device memory of a coarsening run and what its translation units share.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "gosh_common.h"

namespace gosh {

// Device blocks that outlive a hierarchy (gosh_device_pool.cpp): at least `bytes` on the
// current device, or null; given back on any thread, whatever device is current (never throws),
// after a wait for their devices unless they are `idle`: nothing that is queued uses them any more;
// what is kept of them on the current device, freed, and the staging below.
void *block_take(size_t bytes);
void block_give(void *const *blocks, size_t count, bool idle = false);
void block_trim();

// Pinned staging for copies between pageable memory and the device: two slots of
// kStagingBytes, null if there is no memory for them.  A pair or two are kept.
constexpr size_t kStagingBytes = size_t(32) << 20;
char *staging_take();
void staging_give(char *both);

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
  void trim() {  // runs where a hierarchy is freed: needs no host memory
    constexpr size_t kBatch = 64;
    void *batch[kBatch];
    size_t held = 0;
    for (const Block &b : blocks) {
      batch[held++] = b.p;
      if (held == kBatch) {
        block_give(batch, held);
        held = 0;
      }
    }
    block_give(batch, held);
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
    blocks.reserve(blocks.size() + 1);  // throws before there is a block to lose
    void *const p = block_take(bytes);
    if (p == nullptr) return nullptr;
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
    ptrs.reserve(ptrs.size() + 1);
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

// Block that outlives the run (a level's array).
template <typename T>
int persistent(T **out, size_t count, const char *what) {
  const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
  void *const p = block_take(bytes);
  if (p == nullptr) return fail(GOSH_ENOMEM, "cannot allocate %zu device bytes for %s", bytes, what);
  *out = static_cast<T *>(p);
  return GOSH_OK;
}

struct DeviceCoarsener {
  Pool pool;
  int threads = 1;
};

}  // namespace gosh
