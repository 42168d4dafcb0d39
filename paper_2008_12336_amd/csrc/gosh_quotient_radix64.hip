// The radix merge of long coarse rows with 64-bit sums.
#include "gosh_quotient_radix.h"

namespace gosh {
template int merge_by_radix<unsigned long long, false>(Pool &, const int64_t *, const int32_t *, int64_t, int64_t, Packing,
                                        uint32_t *, unsigned long long *, int64_t *);
template int merge_by_radix<unsigned long long, true>(Pool &, const int64_t *, const int32_t *, int64_t, int64_t, Packing,
                                       uint32_t *, unsigned long long *, int64_t *);
}  // namespace gosh
