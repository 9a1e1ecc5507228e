// Divisions of a kernel by what its launch knows: the host finds a factor and a shift, the kernel multiplies.  The
// host's part compiles without HIP, so that a test can take it by itself.
#pragma once
#include <stdint.h>

namespace tern {
namespace {

// Small numbers: e / d = (e * m) >> s for 0 <= e < emax <= 2^15
// (below 2^16 for d a power of two): with emax * d <= 2^s the error of m = ceil(2^s / d) stays below 1 / d, and
// e * m < 2^32.
struct Reciprocal {
    uint32_t m, s;
};
inline Reciprocal reciprocal(uint32_t d, uint32_t emax)
{
    uint32_t s = 0;
    while (((uint64_t)1 << s) < (uint64_t)emax * d) ++s;
    const Reciprocal r = {(uint32_t)((((uint64_t)1 << s) + d - 1) / d), s};
    return r;
}
// Block numbers, e below 2^31: the product takes 64 bits.  m = ceil(2^s / d) with s = 31 + ceil(log2 d) is below
// 2^32, and m * d exceeds 2^s by less than d <= 2^(s - 31).
struct Divisor {
    uint32_t m, s;
    int32_t d;
};
inline int32_t log2_up(int32_t x)
{
    int32_t l = 0;
    while (((int64_t)1 << l) < x) ++l;
    return l;
}
inline Divisor divisor(int32_t d)
{
    const uint32_t s = 31 + (uint32_t)log2_up(d);
    const Divisor r = {(uint32_t)((((uint64_t)1 << s) + (uint32_t)d - 1) / (uint32_t)d), s, d};
    return r;
}

#ifdef __HIP__
__device__ __forceinline__ uint32_t quotient(uint32_t e, Reciprocal r) { return __umul24(e, r.m) >> r.s; }
__device__ __forceinline__ int quotient(int e, Divisor d) { return (int)(((uint64_t)(uint32_t)e * d.m) >> d.s); }
#endif

}  // namespace
}  // namespace tern
