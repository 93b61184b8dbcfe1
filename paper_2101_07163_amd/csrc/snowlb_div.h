// snowlb_div.h -- division by a number known on the host, for the tile orders of the 2D and 3D steps.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace snowlb {

// n / d for 0 <= n < 2^31 by a multiplication: (n * m) >> (31 + ceil(log2 d)) with m rounded up (m < 2^32 for
// d >= 2; for d = 1, m = 0 and the mask of bit 5 adds n itself).  code: the shift beyond 32 (bits 0..4) and bit 5.
// No branch, so a uniform n stays in scalar registers.
struct FastDiv {
    uint32_t m, code;
};
inline FastDiv fast_div(uint32_t d) {
    if (d <= 1) return FastDiv{0u, 32u};
    uint32_t l = 1;
    while ((1ull << l) < d) ++l;
    return FastDiv{(uint32_t)(((1ull << (31 + l)) + d - 1) / d), l - 1};
}
__host__ __device__ __forceinline__ uint32_t div_by(uint32_t n, uint32_t m, uint32_t code) {
    return ((uint32_t)(((uint64_t)n * m) >> 32) >> (code & 31u)) + (n & (0u - ((code >> 5) & 1u)));
}

}  // namespace snowlb
