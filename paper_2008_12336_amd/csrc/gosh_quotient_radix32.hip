// The radix merge of long coarse rows with 32-bit sums.
#include "gosh_quotient_radix.h"

namespace gosh {
template int merge_by_radix<uint32_t, false>(Pool &, const int64_t *, const int32_t *, int64_t, int64_t, Packing,
                                        uint32_t *, uint32_t *, int64_t *);
template int merge_by_radix<uint32_t, true>(Pool &, const int64_t *, const int32_t *, int64_t, int64_t, Packing,
                                       uint32_t *, uint32_t *, int64_t *);
}  // namespace gosh
