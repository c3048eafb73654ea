// Division of non-negative integers by a launch constant (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cdl {

// n / d for 0 <= n < 2^31 by one multiplication: with s = ceil(log2 d) and mul = ceil(2^(31 + s) / d) (below 2^32) the
// quotient is (n * mul) >> (31 + s), exactly (the excess mul * d - 2^(31 + s) is below d <= 2^s, so it adds less than
// one unit of the quotient over the whole range of n); sh = s - 1, or -1 for d = 1.
struct DivBy { uint32_t mul; int sh; };
inline DivBy make_div_by(uint32_t d)
{
    if (d <= 1) return DivBy{0u, -1};
    int s = 0;
    while ((1ull << s) < d) ++s;
    const unsigned long long mul = ((1ull << (31 + s)) + d - 1) / d;
    return DivBy{(uint32_t)mul, s - 1};
}
__device__ __forceinline__ int div_by(int n, uint32_t mul, int sh)
{
    return sh < 0 ? n : (int)(__umulhi((uint32_t)n, mul) >> sh);
}
__device__ __forceinline__ int div_by(int n, DivBy d) { return div_by(n, d.mul, d.sh); }

}  // namespace cdl
