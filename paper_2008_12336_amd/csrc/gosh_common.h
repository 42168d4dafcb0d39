// Shared by the translation units of libgosh: error reporting and argument checks.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>

#include "gosh.h"

namespace gosh {

// Records a printf-style message for gosh_last_error() and returns `code`.
int fail(int code, const char *fmt, ...);

// Argument checks common to the device entry points.  Return GOSH_OK or record an
// error and return GOSH_EINVAL.
int check_dim(int32_t d);
int check_matrix(const float *M, int32_t d, const char *what);
int check_csr(const gosh_csr *g);
// The span [p, p + bytes) must be memory a kernel can reach: a device allocation that holds
// all of it, or pinned host memory.  GOSH_EINVAL otherwise (pageable host memory, a span
// running past its allocation) -- a kernel would fault on it.
int check_device_span(const void *p, size_t bytes, const char *what);
int check_device_csr(const gosh_csr *g);  // both arrays of a device-resident graph

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Turns a failed launch into GOSH_EHIP.
int check_launch(const char *kernel);

// Records the failure of a HIP call for gosh_last_error() and returns its status:
// GOSH_ENOMEM when device or pinned memory ran out, GOSH_EHIP otherwise.
int hip_fail(hipError_t e, const char *what);

// Seams for the library's own tests, one set per thread and not part of gosh.h:
// gosh_testing(which, value) sets one and returns what it was.
enum Seam : int32_t {
  kSeamHotMode,    // written by every launch of the training kernels: its HotMode
  kSeamDeny,       // memory that is not to be had: a sum of the Deny flags
  kSeamRadixFrom,  // if not 0: long coarse rows of graphs with more columns are sorted by radix
  kSeamWideSums,   // if not 0: multiplicities are summed in 64 bits from this weight on
  kSeamLockTries,  // if not 0: tries of a row lock before an update is added without it
  kSeamLocksHeld,  // if not 0: every lock of an epoch is held (1) or free (2) when its launch begins
  kSeamSwaps,      // written by every rotation: how many part swaps a kernel made
  kSeamWeightBits, // if not 0: at most so many bits of a weight lie beside its column while rows are merged
  kSeams
};
enum Deny : int64_t { kDenyLocks = 1, kDenyStaging = 2, kDenyRadix = 4, kDenyTable = 8, kDenyNarrow = 16,
                      kDenyRetired = 32 };
int64_t &seam(Seam which);
inline bool denied(Deny what) { return (seam(kSeamDeny) & what) != 0; }

// Returns from the enclosing function with that status if the call fails.
#define GOSH_TRY_HIP(call, what)                                 \
  do {                                                           \
    hipError_t e_ = (call);                                      \
    if (e_ != hipSuccess) return gosh::hip_fail(e_, what);       \
  } while (0)

// hipMalloc, tried again without the device blocks kept from freed hierarchies if it fails, and
// the number of bytes of those on the current device.
hipError_t device_malloc_bytes(void **p, size_t bytes);
template <typename T>
hipError_t device_malloc(T **p, size_t bytes) {
  return device_malloc_bytes(reinterpret_cast<void **>(p), bytes);
}
size_t block_kept();

// The process-wide tuning record behind gosh_set_tuning / gosh_get_tuning (fields documented
// in gosh.h).  Read at the start of every call that launches a training kernel.
gosh_tuning tuning();

// Wavefronts the device keeps resident (8 on each of the 4 SIMDs of every CU).
int resident_waves();

// Rows first_row .. first_row+count-1 of the initial matrix of a level, written to
// rows_dev (count x d): the arithmetic of gosh_init_embedding for a slice.
int init_rows(float *rows_dev, int64_t first_row, int64_t count, int32_t d, uint64_t seed,
              uint32_t level, hipStream_t st);

// True if [p, p + bytes) lies inside the mapped part of a matrix of gosh_matrix_place.
bool inside_placed_matrix(const void *p, size_t bytes);

// The launch behind gosh_row_probe, without its argument checks (the caller has made them).
int row_probe(float *M_dev, int64_t n, int32_t d, int64_t accesses, uint64_t seed, int32_t mode, hipStream_t st);

// Divergence check: largest finite |entry| (as the bits of the float) and the number of
// non-finite entries, accumulated on the device.  clear, then add any number of row ranges
// (all on one stream, or ordered by events), then read (copies the result and waits for the
// stream).
struct CheckResult {
  uint32_t max_bits;
  uint32_t pad;
  unsigned long long nonfinite;
};
// Where kernels on the current device reach `bytes` of host memory at p, or null unless all of it is
// pinned.
void *pinned_on_device(void *p, size_t bytes);

int matrix_check_clear(CheckResult *results_dev, hipStream_t st, int count = 1);
int matrix_check_add(const float *rows_dev, int64_t floats, CheckResult *result_dev, hipStream_t st);
int matrix_check_read(const CheckResult *result_dev, float *max_abs, int64_t *nonfinite, hipStream_t st);
// A per-device CheckResult owned by the library (allocated on first use, kept).
int check_scratch(CheckResult **out);

// Per-device scratch for the hot-row bitmap (one bit per vertex), grown on demand and, smaller
// blocks included, kept until the process ends.  Calls on one device must not overlap on different
// streams.
int hot_scratch(size_t bytes, void **out);
// Per-device words of the training kernels, per row: a lock, zero between launches, and two counts
// of draws that launches use in turns.  The launch counts in `draws`, which are zero, and clears
// the first `stale_rows` of `stale`, which the launch before may still be reading until then.
// Grown on demand, cleared on `stream` (a hipStream_t) and kept until the process ends.  GOSH_ENOMEM
// if there is no memory: the launch then does without.
struct LockWords {
  uint32_t *locks, *draws, *stale;
  int64_t stale_rows;
};
int lock_scratch(int64_t rows, void *stream, LockWords *out);

}  // namespace gosh
