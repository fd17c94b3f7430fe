// Division by an invariant, for kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pconv {

// n / d for n < 2^31 by one multiplication: Granlund and Montgomery's division by an invariant, with the
// multiplier floor(2^32 (2^s - d) / d) + 1 and s = ceil(log2 d)
struct FastDiv { uint32_t mul, shift; };
inline FastDiv make_fast_div(uint32_t d)
{
    uint32_t s = 0;
    while ((uint64_t(1) << s) < d) ++s;
    return {uint32_t(((uint64_t(1) << 32) * ((uint64_t(1) << s) - d)) / d + 1), s};
}
__device__ __forceinline__ int fast_div(int n, FastDiv d)
{
    return int((__umulhi(uint32_t(n), d.mul) + uint32_t(n)) >> d.shift);
}

}  // namespace pconv
