// Division by a divisor known on the host.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lce {

// Unsigned division n / d for n < 2^31 by multiply-high (Granlund-Montgomery
// round-up variant): q = (mulhi(n, magic) + n) >> shift.
struct FastDiv {
    uint32_t d, magic, shift;
};

__host__ inline FastDiv make_fastdiv(uint32_t d) {
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;                       // l = ceil(log2 d)
    const uint64_t magic = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
    return FastDiv{d, (uint32_t)magic, l};
}

__device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv &f) {
    return (__umulhi(n, f.magic) + n) >> f.shift;
}

}  // namespace lce
