// Splitting FP64 values into BF16 parts, each the nearest BF16 (ties to even)
// of what the parts before it leave.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace bsm {

// Round-to-odd double -> float followed by round-to-nearest-even float ->
// bf16 gives the correctly rounded (RNE) bf16 of the double: the float keeps
// 24 significant bits, more than the 8 + 2 the second rounding needs.
__device__ inline uint32_t bf16_rne(double x) {
    float t = __double2float_rz(x);
    if (static_cast<double>(t) != x) t = __uint_as_float(__float_as_uint(t) | 1u);
    uint32_t u = __float_as_uint(t);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ inline double bf16_to_double(uint32_t h) {
    return static_cast<double>(__uint_as_float(h << 16));
}

// The first `parts` (2 or 3) parts of x.  What a part leaves is exact in FP64
// (the parts are roundings of the value they are subtracted from, far above
// its last bit).
__device__ inline void split_bf16(double x, int parts, uint32_t (&p)[3]) {
    p[0] = bf16_rne(x);
    const double r = x - bf16_to_double(p[0]);
    p[1] = bf16_rne(r);
    p[2] = parts == 3 ? bf16_rne(r - bf16_to_double(p[1])) : 0u;
}

}  // namespace bsm
