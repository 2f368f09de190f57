// SiLU of values that are rounded to bf16 next, for the epilogues of the convolution kernels (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace coe {
namespace k {

// SiLU as every kernel of this library defines it
__device__ __forceinline__ float silu_exact(float x) { return x / (1.f + expf(-x)); }

// x / (1 + 2^(x * -log2 e)) by the machine's exponential and reciprocal.  What the product's rounding and the constant leave out grows
// with -x: at most 10 units of the result from silu_exact from kSiluNear on (however large x is).  CORRECTED makes up for it to first
// order: 5 units from kSiluFar on.  (Arguments beyond 80 take 80's exponent: the sum with one is one.)
constexpr float kSiluNear = -10.f, kSiluFar = -80.f;
template <bool CORRECTED> __device__ __forceinline__ float silu_short(float x)
{
    constexpr float kExp = -1.44269504088896340736f, kExpRest = (float)(-1.44269504088896340736 - (double)kExp), kLn2 = 0.69314718055994530942f;
    if (!CORRECTED) return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x * kExp));
    const float m = fminf(x, 80.f), p = m * kExp;
    const float rest = fmaf(m, kExpRest, fmaf(m, kExp, -p));
    return x * __builtin_amdgcn_rcpf(fmaf(__builtin_amdgcn_exp2f(p), fmaf(rest, kLn2, 1.f), 1.f));
}

// With the bits that silu_exact gives after rounding to bf16: a short form decides unless it is so close to the middle between two
// bf16 values that kDistance units of fp32 could tip it (a value in 3000), or below kSiluFar.  Those lanes evaluate silu_exact.
// Wavefronts with a value below kSiluNear take the corrected form: with a widened distance or silu_exact for such values, launches with
// many of them took up to half as long again as with silu_exact throughout.  Compared over all 2^32 arguments, both forms: the same
// bf16 everywhere.
// What bounds an epilogue with SiLU is vector instructions: an exponential and a division of full precision are about 25 of them per
// value, the short form is 8, the corrected one 12.  us per launch, 250 images, 1x1, values of standard deviation 0.6 / 4.8 / 16 before
// the activation: 64 -> 64 on 56 x 56 45 / 48 / 48 (silu_exact throughout 59), 128 -> 128 on 56 x 56 108 / 112 / 113 (128), 256 -> 256 on
// 28 x 28 54 / 58 / 59 (66), 512 -> 512 on 14 x 14 37 / 40 / 40 (45); 3x3, 128 -> 128 on 28 x 28 61 / 64 / 64 (67).
template <int N> __device__ __forceinline__ void silu_for_bf16(float (&v)[N])
{
    constexpr uint32_t kDistance = 10;
    float x[N], lowest = 0.f;
    uint16_t off[N], nearest = 0xFFFF;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = v[i];
        lowest = fminf(lowest, x[i]);
    }
    if (__builtin_amdgcn_ballot_w64(lowest < kSiluNear)) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = silu_short<true>(x[i]);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = silu_short<false>(x[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        off[i] = (uint16_t)(__float_as_uint(v[i]) - (0x8000u - kDistance));
        nearest = min(nearest, off[i]);
    }
    if (nearest > 2 * kDistance && lowest >= kSiluFar) return;
    uint32_t open = 0;                                        // a bit per value; one value of a lane at a time: little code
#pragma unroll
    for (int i = 0; i < N; ++i) open |= off[i] <= 2 * kDistance || x[i] < kSiluFar ? 1u << i : 0u;
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
