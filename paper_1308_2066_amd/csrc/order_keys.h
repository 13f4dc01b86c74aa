// Order keys of binary64 values for the sort and the selection (internal).
#pragma once

#include "ara_internal.h"

namespace ara {

// Unsigned keys whose order is the descending order of the values; -0.0 is +0.0, and NaNs come
// by their sign, positive ones before every other value and negative ones after.
__device__ __forceinline__ uint64_t desc_key(double d) {
    uint64_t u = __builtin_bit_cast(uint64_t, d + 0.0);   // -0.0 + 0.0 == +0.0
    u = (u >> 63) ? ~u : (u | 0x8000000000000000ull);       // ascending order key
    return ~u;                                             // descending
}

__device__ __forceinline__ double key_value(uint64_t k) {
    uint64_t u = ~k;
    u = (u >> 63) ? (u & 0x7FFFFFFFFFFFFFFFull) : ~u;
    return __builtin_bit_cast(double, u);
}

}  // namespace ara
