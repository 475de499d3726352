// Entries of the one-axis Gibbs factors, and their split into a pair of
// bfloat16 values (hi + lo).
#pragma once

#include <math.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace jko {

__device__ __forceinline__ uint16_t f2bf_rne(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Entry of the Gibbs factor of an axis of n cells, for cells `diff` apart, and
// the bfloat16 pair of one.
__device__ __forceinline__ double gibbs_entry(int diff, int n, double gamma) {
    const double d = (double)diff / (double)n;
    return exp(-(d * d) / gamma);
}
__device__ __forceinline__ void gibbs_split(double kd, uint16_t* hi, uint16_t* lo) {
    const uint16_t h = f2bf_rne((float)kd);
    *hi = h;
    *lo = f2bf_rne((float)(kd - (double)bf2f(h)));
}
// One entry as a kernel's table of them holds it: the float's bits, or hi and lo.
template <bool SPLIT>
__device__ __forceinline__ uint32_t gibbs_bits(int diff, int n, double gamma) {
    const double kd = gibbs_entry(diff, n, gamma);
    if (!SPLIT) return __float_as_uint((float)kd);
    uint16_t h, l;
    gibbs_split(kd, &h, &l);
    return h | ((uint32_t)l << 16);
}

}  // namespace jko
