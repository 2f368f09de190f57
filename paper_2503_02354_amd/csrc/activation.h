// SiLU of values that are rounded to bf16 next, for the epilogues of the convolution kernels (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace coe {
namespace k {

// SiLU as every kernel of this library defines it
__device__ __forceinline__ float silu_exact(float x) { return x / (1.f + expf(-x)); }

// With the bits that silu_exact gives after rounding to bf16: a short form decides unless it is so close to the middle between two
// bf16 values that kDistance units of fp32 could tip it (a value in 3000), or |x| is above kLargest (or x is not a number).  Those
// lanes evaluate silu_exact.  The short form errs by the rounding of its exponent, 0.7 2^-21 at |x| = 10, one unit each of the
// exponential and the reciprocal, and three roundings: compared over all 2^32 arguments, distance at most 10 for |x| <= 10, the
// same bf16 everywhere.
// What bounds an epilogue with SiLU is vector instructions: an exponential and a division of full precision are about 25 of them per
// value, this is 8.  us per launch, 250 images, 1x1 (silu_exact throughout / this / the same launch with ReLU): 64 -> 64 on 56 x 56
// 60 / 48 / 38, 128 -> 128 on 56 x 56 129 / 115 / 86, 256 -> 256 on 28 x 28 68 / 57 / 46, 512 -> 512 on 14 x 14 46 / 38 / 31.
template <int N> __device__ __forceinline__ void silu_for_bf16(float (&v)[N])
{
    constexpr uint32_t kDistance = 10;
    constexpr float kLargest = 10.f;
    float x[N], largest = 0.f;
    uint16_t off[N], nearest = 0xFFFF;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = v[i];
        v[i] = x[i] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x[i] * -1.44269504088896340736f));
        off[i] = (uint16_t)(__float_as_uint(v[i]) - (0x8000u - kDistance));
        nearest = min(nearest, off[i]);
        largest = fmaxf(largest, fabsf(x[i]));
    }
    if (nearest > 2 * kDistance && largest <= kLargest) return;
    uint32_t open = 0;                                        // a bit per value; one value of a lane at a time: little code
#pragma unroll
    for (int i = 0; i < N; ++i) open |= off[i] <= 2 * kDistance || !(fabsf(x[i]) <= kLargest) ? 1u << i : 0u;
    while (open) {
        const uint32_t one = open & (0u - open);
        float at = x[0];
#pragma unroll
        for (int i = 1; i < N; ++i) at = one == 1u << i ? x[i] : at;
        const float r = silu_exact(at);
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = one == 1u << i ? r : v[i];
        open ^= one;
    }
}

}  // namespace k
}  // namespace coe
