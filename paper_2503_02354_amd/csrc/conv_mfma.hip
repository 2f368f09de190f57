// bf16 implicit-GEMM convolution on the gfx950 matrix cores.
//
// GEMM view: out[m][k] = sum_{r,s,c} x[n][p*stride-pad+r][q*stride-pad+s][c] * w[k][r][s][c], m = (n,p,q) flattened.
// NHWC activations make the reduction index contiguous in c, so a reduction step is one (r,s) position and a run
// of 32 channels.  A workgroup owns a BM x BN output tile.  Five kernels, picked by conv_mfma():
//   1. conv_igemm_ring_kernel  launches of few output tiles (conv_ring says how few): 32 x 32 or 64 x 64 tiles of four
//                              wavefronts, loads many reduction steps ahead; same bits as the kernel below that the shape
//                              otherwise takes;
//   2. conv3x3_slab_kernel     3x3, stride 1, pad 1, filter count a multiple of 64: the activation rows a tile needs are
//                              DMA'd into LDS once per 32-channel block and serve all nine window positions;
//   3. conv_gemm_persistent_kernel  other shapes with a filter count that is a multiple of 256 and a long reduction, in launches whose
//                              tiles fill the chip well (persistent_height): tiles of up to 256 x 256 by workgroups that stay;
//   4. conv_igemm_dma_kernel   any other shape with a filter count that is a multiple of 64: both operands DMA'd
//                              global -> LDS per reduction step;
//   5. conv_igemm_bf16_kernel  (below) the rest: operands staged through registers.
// Common to all five:
//   * Filters are repacked once, when an expert is registered, into matrix-core fragment order (pack_filters_mfma),
//     so a filter slab is contiguous in memory and in LDS and an operand read is one linear 1 KiB access.
//   * v_mfma_f32_32x32x16_bf16 (16x16x32 in the smallest tiles) is issued with the filter fragment as the first operand, so a lane ends up holding 4
//     consecutive output channels of one pixel per accumulator quad.
//   * Epilogue in fp32: + bias (+ residual), activation, one round-to-nearest-even to bf16 (v_cvt_pk_bf16_f32).
//   * Zero padding of the convolution and rows past the end of a tile come from buffer loads whose out-of-range
//     offsets return zero; which window positions fall inside the image is a per-row bit mask computed once.
// The register-staged kernel:
//   * Loads run kDepth steps ahead: each step's activation slab (BM x BK) and filter slab (BN x BK) travel
//     global -> registers (kDepth register stages) -> LDS (two stages) -> matrix-core operands.  Every step issues
//     the same loads unconditionally, so the wait before a register stage is moved to LDS can leave the younger
//     stages in flight.
//   * A wave64 vector instruction occupies a SIMD for 4 cycles and a step has only 16 matrix-core instructions per
//     wavefront, so per-step address arithmetic is kept to a few instructions per load (the position inside the
//     window is a scalar offset shared by all lanes).
//   * Activation rows are padded by 16 bytes in LDS so the 16-byte operand reads are bank-conflict free.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "activation.h"
#include "kernels.h"

namespace coe {
namespace k {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPad = 8;              // elements of padding per LDS activation row (16 bytes)
constexpr int kXcds = 8;
constexpr int kDepth = 3;            // register stages = how many steps ahead the global loads run
constexpr uint32_t kOutOfRange = 0x80000000u;   // buffer offset beyond any tensor: the load returns zeros

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));   // round to nearest even
}
// GELU as every kernel of this library defines it
__device__ __forceinline__ float gelu_erfc(float x)
{
    return 0.5f * x * erfcf(-x * 0.70710678118654752440f);
}
// The same within ten units in the last place of fp32, for x > -12 and NaN: max(x, 0) - |x| Q(|x|), Q(a) = exp(-a^2 / 2) h(a),
// h(a) = erfcx(a / sqrt 2) / 2 as t times a polynomial of degree 8 in t = 1 / (1 + 0.26 a): a weighted least-squares fit, iterated
// towards equal relative error on 0 <= a <= 14.5 (7e-8 with the coefficients in fp32).  The exponent is the square of the rounded
// argument that gelu_erfc passes on, to twice the precision: the rounding of that argument weighs far out.
__device__ __forceinline__ float gelu_fast(float x)
{
    const float a = fabsf(x > 64.f ? 64.f : x), t = __builtin_amdgcn_rcpf(fmaf(0.26f, a, 1.f));
    float p = 0.0302301552f;
    p = fmaf(p, t, -0.151493773f);
    p = fmaf(p, t, 0.248731926f);
    p = fmaf(p, t, -0.147787973f);
    p = fmaf(p, t, 0.158757895f);
    p = fmaf(p, t, 0.0519651659f);
    p = fmaf(p, t, 0.102788605f);
    p = fmaf(p, t, 0.103050984f);
    p = fmaf(p, t, 0.103757024f);
    constexpr float kLog2e = -1.44269504088896340736f, kLog2eLow = (float)(-1.44269504088896340736 - (double)kLog2e);
    const float y = a * 0.70710678118654752440f, z = y * y, h = z * kLog2e;
    const float low = fmaf(fmaf(z, kLog2eLow, fmaf(z, kLog2e, -h)), 0.69314718055994530942f, -fmaf(y, y, -z));
    const float e = __builtin_amdgcn_exp2f(h);
    return fmaf(-a, fmaf(e, low, e) * t * p, fmaxf(x, -0.f));
}
// GELU of values that are rounded to bf16 next, with the bits that gelu_erfc gives: the fast form decides unless it is so close to
// the middle between two bf16 values that ten units of fp32 could tip it (a value in 3000), or far out.  Those lanes evaluate
// gelu_erfc.  Compared over all 2^32 arguments: distance at most 10 for x > -12, the same bf16 everywhere, NaN for NaN and for
// minus infinity.  (Which way single roundings fall moves the logits after twelve transformer layers by 1 %.)  Its time is near
// that of the fast form alone: chain of 777 transformer requests 91.8 ms with the 128 x 128 tiles and erfcf throughout, 78.6 with
// today's tiles and erfcf, 73.9 with a fast form that differed in one rounding of 10,000, 75.1 with this (in groups of eight values
// on the persistent tiles; of four 2 % slower, of sixteen 7 %: too many registers).
template <int N> __device__ __forceinline__ void gelu_for_bf16(float (&v)[N])
{
    constexpr uint32_t kDistance = 10;
    float x[N], lowest = 0.f;
    uint16_t off[N], nearest = 0xFFFF;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = v[i];
        v[i] = gelu_fast(x[i]);
        off[i] = (uint16_t)(__float_as_uint(v[i]) - (0x8000u - kDistance));
        nearest = min(nearest, off[i]);
        lowest = fminf(lowest, x[i]);
    }
    if (nearest > 2 * kDistance && lowest > -12.f) return;
    if constexpr (N <= 4) {                                   // (as few registers as possible)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (off[i] <= 2 * kDistance || x[i] <= -12.f) v[i] = gelu_erfc(x[i]);
    } else {                                                  // (as little code as possible: one value of a lane at a time)
        uint32_t open = 0;                                    // a bit per value
#pragma unroll
        for (int i = 0; i < N; ++i) open |= off[i] <= 2 * kDistance || x[i] <= -12.f ? 1u << i : 0u;
        do {
            const uint32_t one = open & (0u - open);
            float at = x[0];
#pragma unroll
            for (int i = 1; i < N; ++i) at = one == 1u << i ? x[i] : at;
            const float r = gelu_erfc(at);
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = one == 1u << i ? r : v[i];
            open ^= one;
        } while (open);
    }
}
__device__ __forceinline__ float act_fn(float v, int act)
{
    if (act == 1) return v > 0.f ? v : 0.f;
    return v;
}
template <int ACT, int N> __device__ __forceinline__ void activate(float (&v)[N])
{
    if (ACT == 2) {
        gelu_for_bf16(v);
    } else if (ACT == 3) {
        silu_for_bf16(v);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = act_fn(v[i], ACT);
    }
}
// The activation is a launch parameter, but an epilogue that tests it per element compiles into hundreds of
// branches: dispatch ONCE per wave to a body specialised for the activation.  GELU's body takes up to 40 registers more than the
// others and would cost every launch of a kernel a wavefront per SIMD (conv_igemm_dma_kernel<128, 128, 2, 2>: 324 -> 362 us on the
// stride-2 layers of 4096 images), so it is in kernels of its own, which the launchers choose.  So is SiLU's where the others
// lose by it: conv_gemm_persistent_kernel spilled up to 18 registers for it in every launch (768 -> 2304, 197 positions of 64 images 49.5 us
// with, 47.0 without, of 100 images 75.3 / 71.3), and in conv_igemm_bf16_kernel it cost launches with ReLU 4 % (128 -> 32 on 17 x 13,
// 200 images 6.31 / 6.07); in conv_igemm_ring_kernel a pass of one request through ResNet-18 shapes took 1 to 2 % longer with it.
constexpr int kActsElse = 0,      // none, ReLU and SiLU, as the launch says
              kActsPlain = 1,     // none and ReLU, as the launch says
              kActsGelu = 2, kActsSilu = 3;
template <int ACTS, typename F> __device__ __forceinline__ void with_activation(int act, F&& body)
{
    if constexpr (ACTS == kActsGelu) {
        body(std::integral_constant<int, 2>{});
    } else if constexpr (ACTS == kActsSilu) {
        body(std::integral_constant<int, 3>{});
    } else {
        if (act == 1) body(std::integral_constant<int, 1>{});
        else if (ACTS == kActsElse && act == 3) body(std::integral_constant<int, ACTS == kActsElse ? 3 : 0>{});
        else body(std::integral_constant<int, 0>{});
    }
}
// raw buffer descriptor over [p, p + bytes): offsets at or beyond `bytes` read as zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, int ACTS>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void conv_igemm_bf16_kernel(const uint16_t* __restrict__ x,
                                                                    const uint16_t* __restrict__ wp,
                                                                    const float* __restrict__ bias,
                                                                    const uint16_t* __restrict__ res,
                                                                    uint16_t* __restrict__ y, ConvShape s, int M,
                                                                    int tiles_n)
{
    constexpr int kThreads = 64 * WAVES_M * WAVES_N;
    static_assert(kThreads == 256 || kThreads == 512, "four or eight wavefronts per workgroup");
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int MB = WM / 32, NB = WN / 32;
    static_assert(MB >= 1 && NB >= 1, "wave tile");
    constexpr int CH = BK / 8;                       // 16-byte chunks per activation slab row
    constexpr int ROWS_PER_PASS = kThreads / CH;
    constexpr int A_LOADS = BM / ROWS_PER_PASS;
    constexpr int KS = BK / 16;                      // matrix-core steps per slab
    constexpr int A_STRIDE = BK + kPad;
    constexpr int A_STAGE = BM * A_STRIDE;           // elements
    constexpr int B_STAGE = BN * BK;                 // elements, fragment order: [BN/32][KS][64 lanes][8]
    constexpr int B_CHUNKS = B_STAGE / 8;
    constexpr int B_LOADS = (B_CHUNKS + kThreads - 1) / kThreads;
    constexpr int B_PER_BLOCK = KS * 64;             // chunks per 32-filter block and step
    constexpr int STAGE = A_STAGE + B_STAGE;

    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // 2 * STAGE elements

    // XCD-aware tile order: consecutive workgroup ids land on different XCDs, so give each XCD a contiguous range
    // of tiles (filter tiles fastest) and the slabs shared by neighbouring tiles stay in one XCD's L2.
    int tile;
    {
        int L = blockIdx.x, total = gridDim.x;
        int xcd = L % kXcds, slot = L / kXcds;
        int base = total / kXcds, rem = total % kXcds;
        tile = xcd * base + (xcd < rem ? xcd : rem) + slot;
    }
    const int tile_n = tile % tiles_n, tile_m = tile / tiles_n;
    const int m0 = tile_m * BM, n0 = tile_n * BN;

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;
    const int chunk = tid % CH;
    const int row0 = tid / CH;

    const int cblocks = s.C / BK;
    const int RS = s.R * s.S;
    const int nsteps = RS * cblocks;
    const int ks16_total = nsteps * KS;               // 16-channel steps per filter

    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(wp, (uint32_t)s.K * (uint32_t)(RS * s.C) * 2u);

    // Per activation row this thread fetches: byte offset of window position (0,0), channel 0 (+ its 16-byte chunk),
    // and a mask with bit r*S+s set when that window position lies inside the image.  Rows past M have mask 0.
    int32_t a_off[A_LOADS];
    uint64_t a_mask[A_LOADS];
    {
        const int PQ = s.P * s.Q;
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {
            int m = m0 + row0 + ROWS_PER_PASS * j;
            bool ok = m < M;
            int mm = ok ? m : 0;
            int n = mm / PQ, pq = mm % PQ;
            int p = pq / s.Q, q = pq % s.Q;
            int ih0 = p * s.stride - s.pad, iw0 = q * s.stride - s.pad;
            a_off[j] = ((n * s.H + ih0) * s.W + iw0) * s.C * 2 + chunk * 16;
            uint64_t mask = 0;
            for (int rr = 0; rr < s.R; ++rr)
                for (int tt = 0; tt < s.S; ++tt)
                    if (ok && (unsigned)(ih0 + rr) < (unsigned)s.H && (unsigned)(iw0 + tt) < (unsigned)s.W)
                        mask |= 1ull << (rr * s.S + tt);
            a_mask[j] = mask;
        }
    }
    // filter slab: chunk c of a step lives at block (c / B_PER_BLOCK), offset (c % B_PER_BLOCK) inside the step's
    // KS fragments of that block; LDS keeps the same linear order
    uint32_t b_off[B_LOADS];
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) {
        int c = tid + kThreads * j;
        b_off[j] = c < B_CHUNKS
                       ? (uint32_t)((((n0 / 32 + c / B_PER_BLOCK) * ks16_total) * 512 + (c % B_PER_BLOCK) * 8) * 2)
                       : kOutOfRange;
    }

    // One register stage: the loads of one reduction step while they are in flight.
    struct RegStage {
        u32x4 a[A_LOADS];
        u32x4 b[B_LOADS];
    };
    RegStage st0, st1, st2;
    static_assert(kDepth == 3, "three named register stages");
    int r = 0, t = 0, cb = 0, f_step = 0;             // (r, s, channel block) and index of the step being fetched

    auto fetch = [&](RegStage& st) {
        const int rs = r * s.S + t;
        const int32_t win = ((r * s.W + t) * s.C + cb * BK) * 2;      // scalar: same for every lane
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j) {
            uint32_t off = ((a_mask[j] >> rs) & 1ull) ? (uint32_t)(a_off[j] + win) : kOutOfRange;
            st.a[j] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, off, 0, 0);
        }
        const uint32_t wstep = (uint32_t)f_step * (KS * 512 * 2);     // scalar
#pragma unroll
        for (int j = 0; j < B_LOADS; ++j) st.b[j] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, b_off[j], wstep, 0);
        // advance; past the last step the fetch position stays put, so a fetch issued beyond the end re-reads the
        // last step (never used) and every step issues the same number of loads
        if (f_step + 1 < nsteps) {
            ++f_step;
            if (++cb == cblocks) { cb = 0; if (++t == s.S) { t = 0; ++r; } }
        }
    };
    uint16_t* const a_dst = lds + row0 * A_STRIDE + chunk * 8;
    uint16_t* const b_dst = lds + A_STAGE + tid * 8;
    auto stash = [&](int stage, const RegStage& st) {
#pragma unroll
        for (int j = 0; j < A_LOADS; ++j)
            *(u32x4*)(a_dst + stage * STAGE + ROWS_PER_PASS * j * A_STRIDE) = st.a[j];
#pragma unroll
        for (int j = 0; j < B_LOADS; ++j)
            if (B_CHUNKS % kThreads == 0 || tid + kThreads * j < B_CHUNKS)
                *(u32x4*)(b_dst + stage * STAGE + kThreads * j * 8) = st.b[j];
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int frag_row = lane & 31;          // pixel row inside a 32-row block
    const int frag_k = (lane >> 5) * 8;      // which 8 of the 16 reduction elements this lane supplies

    // Operand fragments are read one matrix-core step ahead of their use, so the LDS latency of step ks+1 hides behind
    // the matrix-core work of step ks.
    const uint16_t* const a_src = lds + (wm * WM + frag_row) * A_STRIDE + frag_k;
    const uint16_t* const b_src = lds + A_STAGE + (wn * NB) * (KS * 512) + lane * 8;
    auto compute = [&](int stage) {
        const uint16_t* a_lds = a_src + stage * STAGE;
        const uint16_t* b_lds = b_src + stage * STAGE;
        bf16x8 af[2][MB], bfr[2][NB];
#pragma unroll
        for (int i = 0; i < MB; ++i) af[0][i] = *(const bf16x8*)(a_lds + i * 32 * A_STRIDE);
#pragma unroll
        for (int j = 0; j < NB; ++j) bfr[0][j] = *(const bf16x8*)(b_lds + (j * KS) * 512);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) {
#pragma unroll
                for (int i = 0; i < MB; ++i)
                    af[(ks + 1) & 1][i] = *(const bf16x8*)(a_lds + i * 32 * A_STRIDE + (ks + 1) * 16);
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    bfr[(ks + 1) & 1][j] = *(const bf16x8*)(b_lds + (j * KS + ks + 1) * 512);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][j], af[ks & 1][i], acc[i][j], 0, 0, 0);
        }
    };

    // prologue: three steps in flight, the first one staged
    fetch(st0);
    fetch(st1);
    fetch(st2);
    stash(0, st0);
    __syncthreads();

    // Step u: the register stage that held step u is free -> refill it with step u + 3; compute step u from LDS
    // stage u & 1; move step u + 1 (loads issued two steps ago) from its register stage to the other LDS stage.
    // Fetch and staging are unconditional (past the end they move data nobody reads): the number of loads in flight
    // at every wait is then a compile-time constant and the wait can leave the younger two stages outstanding.
    auto step = [&](int u, RegStage& refill, const RegStage& next) {
        fetch(refill);
        if (u < nsteps) compute(u & 1);
        stash((u + 1) & 1, next);
        __syncthreads();
    };
    for (int u0 = 0; u0 < nsteps; u0 += kDepth) {
        step(u0, st0, st1);
        step(u0 + 1, st1, st2);
        step(u0 + 2, st2, st0);
    }

    // Epilogue.  With the filter fragment as the first operand, accumulator element v of lane l belongs to pixel l%32
    // and filter 8*(v/4) + 4*(l/32) + v%4 of the 32x32 block: a quad of v is 4 consecutive channels of one pixel.
    const int f_hi = (lane >> 5) * 4;
    with_activation<ACTS>(s.act, [&](auto act_c) {
    constexpr int ACT = decltype(act_c)::value;
    // no load crosses SiLU's branches: its bias is fetched one quad ahead (192 -> 96, 20 x 20, 16 images 5.9 -> 5.6 us, 250 images 22.7 -> 22.0)
    constexpr bool kAhead = ACT == 3;
    auto bias_of = [&](int quad) { return *(const float4*)(bias + n0 + wn * WN + 8 * quad + f_hi); };
    float4 ahead = make_float4(0.f, 0.f, 0.f, 0.f);
    if (kAhead) ahead = bias_of(0);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int m = m0 + wm * WM + i * 32 + frag_row;
        if (m >= M) continue;
        const size_t orow = (size_t)m * s.K;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + wn * WN + j * 32 + 8 * g + f_hi;
                const float4 bv = kAhead ? ahead : bias_of(4 * j + g);
                if (kAhead) ahead = bias_of((4 * j + g + 1) % (4 * NB));
                float v0 = acc[i][j][4 * g + 0] + bv.x, v1 = acc[i][j][4 * g + 1] + bv.y;
                float v2 = acc[i][j][4 * g + 2] + bv.z, v3 = acc[i][j][4 * g + 3] + bv.w;
                if (res) {
                    uint2 rv = *(const uint2*)(res + orow + n);
                    v0 += bf16_to_f32(rv.x & 0xFFFFu); v1 += bf16_to_f32(rv.x >> 16);
                    v2 += bf16_to_f32(rv.y & 0xFFFFu); v3 += bf16_to_f32(rv.y >> 16);
                }
                float v[4] = {v0, v1, v2, v3};
                activate<ACT>(v);
                *(uint2*)(y + orow + n) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            }
        }
    }
    });
}

template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, int ACTS = kActsPlain>
hipError_t launch(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                  hipStream_t stream)
{
    if constexpr (ACTS == kActsPlain) {
        if (s.act == 2) return launch<BM, BN, BK, WAVES_M, WAVES_N, kActsGelu>(x, wp, bias, res, y, s, stream);
        if (s.act == 3) return launch<BM, BN, BK, WAVES_M, WAVES_N, kActsSilu>(x, wp, bias, res, y, s, stream);
    }
    long long M = (long long)s.N * s.P * s.Q;
    int tiles_m = (int)((M + BM - 1) / BM), tiles_n = s.K / BN;
    long long total = (long long)tiles_m * tiles_n;
    if (total > 0x7FFFFFFFll) return hipErrorInvalidValue;
    constexpr size_t kLdsBytes = 2 * (size_t)(BM * (BK + kPad) + BN * BK) * sizeof(uint16_t);
    constexpr int kThreads = 64 * WAVES_M * WAVES_N;
    static bool configured = false;
    if (!configured) {   // more than the default 64 KiB of LDS per workgroup needs an explicit opt-in
        hipError_t e = hipFuncSetAttribute((const void*)conv_igemm_bf16_kernel<BM, BN, BK, WAVES_M, WAVES_N, ACTS>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL((conv_igemm_bf16_kernel<BM, BN, BK, WAVES_M, WAVES_N, ACTS>), dim3((unsigned)total), dim3(kThreads), kLdsBytes,
                       stream, (const uint16_t*)x, (const uint16_t*)wp, bias, (const uint16_t*)res, (uint16_t*)y, s, (int)M,
                       tiles_n);
    return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------------------------
// Direct-to-LDS kernel.  Both operands of a reduction step are DMA'd from global memory straight into LDS (buffer
// loads with the LDS bit: lane i of a load lands at base + 16 i, one instruction fills 1 KiB).  No register staging
// and no LDS store instructions (an LDS store instruction moves 64 bytes per clock, half the read rate, and the
// staging registers cost occupancy).
//   * Filters: one load = one fragment of the repacked filter tensor, read back linearly.
//   * Activations: one load = 16 pixel rows x 64 bytes (a 32-channel run), four adjacent lanes per row so the global
//     access stays 64 bytes contiguous.  Inside the 1 KiB block the 16-byte chunk c of row r sits in slot
//     4 r + (c ^ f(r)), f(r) = ((r >> 1) & 3) ^ (r >> 3): the later operand read (lane = pixel row, fixed chunk) then
//     touches every LDS bank equally, whether the hardware resolves conflicts per 8 or per 16 lanes.  The lane that
//     fills slot i simply fetches the chunk that belongs there.
// Three LDS stages, loads two steps ahead, one barrier per step:
//     wait until this wave's loads of step u have landed | barrier | issue loads of step u+2 into the stage that
//     step u-1 was computed from (every wave is past that, it is behind the barrier) | compute step u.
// ---------------------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void;

// Which group a tile belongs to in a grouped launch, and what that means for the tile: its first output pixel, the end of
// the group's pixels, its position among the filter tiles, the group's filters and bias.  Tiles are numbered group by
// group, filter tiles fastest; every group starts a fresh row of tiles, so no tile mixes two experts' weights.
struct TileOrigin {
    int m0, m_end, tile_n;
    const uint16_t* wp;
    const float* bias;
};
template <int BM>
__device__ __forceinline__ TileOrigin locate_tile(int tile, int tiles_n, int PQ, int M, const uint16_t* wp, const float* bias,
                                                  const GroupTable& gt, uint32_t off_w, uint32_t off_b)
{
    TileOrigin o;
    if (gt.n == 0) {
        o.tile_n = tile % tiles_n;
        o.m0 = (tile / tiles_n) * BM;
        o.m_end = M;
        o.wp = wp;
        o.bias = bias;
        return o;
    }
    int g = 0, t = tile;
    for (;; ++g) {                                            // the launch has exactly sum-of-tiles workgroups
        const int rows = (gt.first_row[g + 1] - gt.first_row[g]) * PQ;
        const int tiles_g = ((rows + BM - 1) / BM) * tiles_n;
        if (t < tiles_g || g + 1 >= gt.n) break;
        t -= tiles_g;
    }
    o.tile_n = t % tiles_n;
    o.m0 = gt.first_row[g] * PQ + (t / tiles_n) * BM;
    o.m_end = gt.first_row[g + 1] * PQ;
    const char* base = (const char*)gt.weights[g];
    o.wp = (const uint16_t*)(base + off_w);
    o.bias = (const float*)(base + off_b);
    return o;
}


// Epilogue of the direct-to-LDS kernels: + bias (+ residual), activation, round to bf16 in the accumulator layout (a
// lane holds 4 consecutive channels of one pixel per accumulator quad), then through a wave-private LDS buffer of
// 32 rows so that the global stores are 16 bytes per lane and cover whole rows of the wave tile (full cache lines
// instead of 8-byte pieces of 32 different lines per instruction).  LDS operations of one wave execute in program
// order, so the wave-private buffer needs no barrier between its writes and reads.
template <int MB, int NB, int ACT, bool RES>
__device__ __forceinline__ void store_tile_via_lds_act(f32x16 (&acc)[MB][NB], uint16_t* stage, const float* __restrict__ bias,
                                                   const uint16_t* __restrict__ res, uint16_t* __restrict__ y, int m_wave,
                                                   int n_wave, int M, int K, int lane)
{
    constexpr int WN = NB * 32, ROW = WN + 8;             // elements; 16 bytes of padding per staged row
    constexpr int CPR = WN / 8;                            // 16-byte chunks per row
    constexpr int T = 32 * CPR / 64;                       // chunks per lane and 32-row block
    constexpr int kQuads = ACT == 3 ? 2 : 1;               // accumulator quads that are finished together: SiLU shares a test
    const int frag_row = lane & 31, f_hi = (lane >> 5) * 4;
    // no load crosses SiLU's branches: its bias is fetched one test ahead (256 -> 256, 28 x 28, 12 images 10.4 -> 10.25 us)
    constexpr bool kAhead = ACT == 3;
    auto bias_of = [&](int quad) { return *(const float4*)(bias + n_wave + 8 * quad + f_hi); };
    float4 ahead[kQuads];
    if (kAhead) {
#pragma unroll
        for (int h = 0; h < kQuads; ++h) ahead[h] = bias_of(h);
    }
    // the residual takes the same road in the other direction: row-contiguous 16-byte loads (all issued up front),
    // staged in LDS, picked up in the accumulator layout
    u32x4 rres[MB][T];
    if (RES) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int idx = lane + 64 * t;
                const int mo = m_wave + i * 32 + idx / CPR;
                rres[i][t] = mo < M ? *(const u32x4*)(res + (size_t)mo * K + n_wave + (idx % CPR) * 8) : u32x4{0u, 0u, 0u, 0u};
            }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (RES) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int idx = lane + 64 * t;
                *(u32x4*)(stage + (idx / CPR) * ROW + (idx % CPR) * 8) = rres[i][t];
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int g = 0; g < 4; g += kQuads) {
                float v[4 * kQuads];
#pragma unroll
                for (int h = 0; h < kQuads; ++h) {
                    const int nl = j * 32 + 8 * (g + h) + f_hi;
                    const float4 bv = kAhead ? ahead[h] : bias_of(4 * j + g + h);
                    if (kAhead) ahead[h] = bias_of((4 * j + g + kQuads) % (4 * NB) + h);
                    v[4 * h] = acc[i][j][4 * (g + h)] + bv.x; v[4 * h + 1] = acc[i][j][4 * (g + h) + 1] + bv.y;
                    v[4 * h + 2] = acc[i][j][4 * (g + h) + 2] + bv.z; v[4 * h + 3] = acc[i][j][4 * (g + h) + 3] + bv.w;
                    if (RES) {
                        const uint2 rv = *(const uint2*)(stage + frag_row * ROW + nl);
                        v[4 * h] += bf16_to_f32(rv.x & 0xFFFFu); v[4 * h + 1] += bf16_to_f32(rv.x >> 16);
                        v[4 * h + 2] += bf16_to_f32(rv.y & 0xFFFFu); v[4 * h + 3] += bf16_to_f32(rv.y >> 16);
                    }
                }
                activate<ACT>(v);
#pragma unroll
                for (int h = 0; h < kQuads; ++h)
                    *(uint2*)(stage + frag_row * ROW + j * 32 + 8 * (g + h) + f_hi) =
                        make_uint2(pack_bf16(v[4 * h], v[4 * h + 1]), pack_bf16(v[4 * h + 2], v[4 * h + 3]));
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int idx = lane + 64 * t;
            const int row = idx / CPR, ch = idx % CPR;
            const int mo = m_wave + i * 32 + row;
            const u32x4 v = *(const u32x4*)(stage + row * ROW + ch * 8);
            if (mo < M) *(u32x4*)(y + (size_t)mo * K + n_wave + ch * 8) = v;
        }
    }
}

template <int ACTS, int MB, int NB>
__device__ __forceinline__ void store_tile_via_lds(f32x16 (&acc)[MB][NB], uint16_t* stage, const float* __restrict__ bias,
                                                   const uint16_t* __restrict__ res, uint16_t* __restrict__ y, int m_wave,
                                                   int n_wave, int M, int K, int act, int lane)
{
    with_activation<ACTS>(act, [&](auto a) {
        if (res) store_tile_via_lds_act<MB, NB, decltype(a)::value, true>(acc, stage, bias, res, y, m_wave, n_wave, M, K, lane);
        else store_tile_via_lds_act<MB, NB, decltype(a)::value, false>(acc, stage, bias, res, y, m_wave, n_wave, M, K, lane);
    });
}

// A 1x1 convolution over the concatenation of up to kMaxSources maps of equal shape reads them where they lie (SOURCES): the shape
// says C channels a map and R maps, and map k takes the place of window position k.  The order of the reduction is that of the
// concatenated map.  Concatenating cost a read and a write of every map and a launch: in a pass of 1000 requests through detectors, of
// 13 ms, 28 launches, 1.0 ms in all.
struct Sources {
    const uint16_t* rest[kMaxSources - 1];      // the maps after the first
};
[[maybe_unused]] __device__ __forceinline__ const uint16_t* source_at(const uint16_t* first, const Sources& from, int k)
{
    const uint16_t* p = first;                                // (k is uniform, the table a kernel argument: no indexed access)
#pragma unroll
    for (int i = 0; i + 1 < kMaxSources; ++i) p = k == i + 1 ? from.rest[i] : p;
    return p;
}

// host side of a grouped launch: the table and where a layer's filters and bias sit inside every group's blob
struct Grouping {
    GroupTable table{};              // table.n == 0: plain launch
    uint32_t off_w = 0, off_b = 0;
};
inline long long count_tiles(long long M, long long PQ, int BM, int tiles_n, const GroupTable& gt)
{
    if (gt.n == 0) return (M + BM - 1) / BM * tiles_n;
    long long total = 0;
    for (int g = 0; g < gt.n; ++g) total += ((gt.first_row[g + 1] - gt.first_row[g]) * PQ + BM - 1) / BM * tiles_n;
    return total;
}

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    // s_waitcnt with only the vector-memory counter armed (expcnt and lgkmcnt fields at their maxima)
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The wait in front of a step's barrier.  Besides the wave's own loads of the step (all but the newest N vector-memory
// operations) it also drains the wave's LDS reads: the compiler is free to sink the last matrix-core instructions of a
// step below the barrier, and with them the wait for their operand reads, so a wave could pass the barrier with reads of
// the previous step still queued while another wave's DMA of a later step already targets the same LDS stage.
template <int N> __device__ __forceinline__ void wait_before_barrier()
{
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool GELU, bool SOURCES>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void conv_igemm_dma_kernel(const uint16_t* __restrict__ x,
                                                                   const uint16_t* __restrict__ wp_all,
                                                                   const float* __restrict__ bias_all,
                                                                   const uint16_t* __restrict__ res,
                                                                   uint16_t* __restrict__ y, ConvShape s, int M,
                                                                   int tiles_n, GroupTable gt, uint32_t off_w, uint32_t off_b, Sources from)
{
#if defined(__HIP_DEVICE_COMPILE__)      // the host pass only needs the launch stub (LDS address-space casts do not exist there)
    constexpr int BK = 32, KS = 2, kStages = 3;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int MB = WM / 32, NB = WN / 32;
    constexpr int FA = BM / 16, FB = BN / 32 * KS;           // 1 KiB blocks per step: 16-row activation blocks, filter fragments
    static_assert(FA % NW == 0 && FB % NW == 0, "every wave issues the same number of loads");
    constexpr int A_PER_WAVE = FA / NW, B_PER_WAVE = FB / NW;
    constexpr int LOADS = A_PER_WAVE + B_PER_WAVE;
    constexpr int FRAG = 512;                                 // elements per 1 KiB block
    constexpr int STAGE = (FA + FB) * FRAG;                   // elements

    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // kStages * STAGE elements

    int tile;
    {
        int L = blockIdx.x, total = gridDim.x;
        int xcd = L % kXcds, slot = L / kXcds;
        int base = total / kXcds, rem = total % kXcds;
        tile = xcd * base + (xcd < rem ? xcd : rem) + slot;
    }
    const TileOrigin org = locate_tile<BM>(tile, tiles_n, s.P * s.Q, M, wp_all, bias_all, gt, off_w, off_b);
    const int m0 = org.m0, n0 = org.tile_n * BN;
    M = org.m_end;                                            // rows of this tile's group end here
    const uint16_t* const wp = org.wp;
    const float* const bias = org.bias;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;

    const int cblocks = s.C / BK;
    const int RS = s.R * s.S;
    const int nsteps = RS * cblocks;
    const int ks16_total = nsteps * KS;

    __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(wp, (uint32_t)s.K * (uint32_t)(RS * s.C) * 2u);

    // rows this lane fetches: block (wid * A_PER_WAVE + j), row lane / 4 of the block; which 16-byte chunk of the
    // 32-channel run follows from the slot the lane fills
    auto swz = [](int r16) { return ((r16 >> 1) & 3) ^ (r16 >> 3); };
    int32_t a_off[A_PER_WAVE];
    uint64_t a_mask[A_PER_WAVE];
    {
        const int PQ = s.P * s.Q;
        const int chunk = (lane & 3) ^ swz(lane >> 2);
#pragma unroll
        for (int j = 0; j < A_PER_WAVE; ++j) {
            int m = m0 + (wid * A_PER_WAVE + j) * 16 + (lane >> 2);
            bool ok = m < M;
            int mm = ok ? m : 0;
            int n = mm / PQ, pq = mm % PQ;
            int p = pq / s.Q, q = pq % s.Q;
            int ih0 = p * s.stride - s.pad, iw0 = q * s.stride - s.pad;
            a_off[j] = ((n * s.H + ih0) * s.W + iw0) * s.C * 2 + chunk * 16;
            uint64_t mask = SOURCES && ok ? ~0ull : 0;
            for (int rr = 0; rr < (SOURCES ? 0 : s.R); ++rr)
                for (int tt = 0; tt < s.S; ++tt)
                    if (ok && (unsigned)(ih0 + rr) < (unsigned)s.H && (unsigned)(iw0 + tt) < (unsigned)s.W)
                        mask |= 1ull << (rr * s.S + tt);
            a_mask[j] = mask;
        }
    }
    // filter fragments of this wave: (wid * B_PER_WAVE + j) = nb * KS + ks
    uint32_t b_off[B_PER_WAVE];
#pragma unroll
    for (int j = 0; j < B_PER_WAVE; ++j) {
        int fb = wid * B_PER_WAVE + j;
        b_off[j] = (uint32_t)((((n0 / 32 + fb / KS) * ks16_total + fb % KS) * FRAG + lane * 8) * 2);
    }

    int r = 0, t = 0, cb = 0, f_step = 0;
    auto issue = [&](int stage) {
        uint16_t* const st = lds + stage * STAGE;
        const int rs = r * s.S + t;
        const int32_t win = ((SOURCES ? 0 : r * s.W + t) * s.C + cb * BK) * 2;
#pragma unroll
        for (int j = 0; j < A_PER_WAVE; ++j) {
            uint32_t off = ((a_mask[j] >> rs) & 1ull) ? (uint32_t)(a_off[j] + win) : kOutOfRange;
            // (the immediate offset of such a load would also shift the LDS destination: keep it 0)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void*)(st + (wid * A_PER_WAVE + j) * FRAG), 16, off, 0, 0, 0);
        }
        const uint32_t wstep = (uint32_t)f_step * (KS * FRAG * 2);
#pragma unroll
        for (int j = 0; j < B_PER_WAVE; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void*)(st + (FA + wid * B_PER_WAVE + j) * FRAG), 16, b_off[j],
                                                     wstep, 0, 0);
        if (f_step + 1 < nsteps) {
            ++f_step;
            if (++cb == cblocks) {
                cb = 0;
                if (++t == s.S) { t = 0; ++r; }
                if (SOURCES) x_rsrc = make_rsrc(source_at(x, from, r), (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
            }
        }
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // operand read: pixel row lane % 32 of a 32-row block, chunk 2 ks + lane / 32 -> element offset inside the
    // two 1 KiB blocks; the chunk of ks = 1 is the one of ks = 0 with bit 1 flipped (32 bytes = 16 elements)
    static_assert(KS == 2, "two 16-channel halves per step");
    const int rd_row = lane & 31;
    const int rd0 = (rd_row >> 4) * FRAG + ((rd_row & 15) * 4 + ((lane >> 5) ^ swz(rd_row & 15))) * 8;
    auto compute = [&](int stage) {
        const uint16_t* a_lds = lds + stage * STAGE + (wm * MB * 2) * FRAG;
        const uint16_t* b_lds = lds + stage * STAGE + (FA + wn * NB * KS) * FRAG + lane * 8;
        bf16x8 af[KS][MB], bfr[KS][NB];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < MB; ++i) af[ks][i] = *(const bf16x8*)(a_lds + i * 2 * FRAG + (rd0 ^ (ks * 16)));
#pragma unroll
            for (int j = 0; j < NB; ++j) bfr[ks][j] = *(const bf16x8*)(b_lds + (j * KS + ks) * FRAG);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
    };

    issue(0);
    issue(1);
    int stage_c = 0, stage_l = 2;
    for (int u = 0; u < nsteps; ++u) {
        wait_before_barrier<LOADS>();        // step u has landed; step u + 1 may still be in flight
        __builtin_amdgcn_s_barrier();
        issue(stage_l);
        compute(stage_c);
        stage_c = stage_c == kStages - 1 ? 0 : stage_c + 1;
        stage_l = stage_l == kStages - 1 ? 0 : stage_l + 1;
    }
    wait_before_barrier<0>();
    __builtin_amdgcn_s_barrier();        // every wave is done with the operand stages: LDS is free for the epilogue
    store_tile_via_lds<GELU ? kActsGelu : kActsElse, MB, NB>(acc, lds + wid * (32 * (WN + 8)), bias, res, y, m0 + wm * WM, n0 + wn * WN, M, s.K, s.act, lane);
#endif
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool GELU = false, bool SOURCES = false>
hipError_t launch_dma(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                      hipStream_t stream, const Grouping& grp = Grouping(), const Sources* from = nullptr)
{
    if constexpr (!GELU && !SOURCES)
        if (from) return launch_dma<BM, BN, WAVES_M, WAVES_N, false, true>(x, wp, bias, res, y, s, stream, grp, from);
    if constexpr (!GELU && !SOURCES)
        if (s.act == 2) return launch_dma<BM, BN, WAVES_M, WAVES_N, true>(x, wp, bias, res, y, s, stream, grp);
    long long M = (long long)s.N * s.P * s.Q;
    int tiles_n = s.K / BN;
    long long total = count_tiles(M, (long long)s.P * s.Q, BM, tiles_n, grp.table);
    if (total > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (total == 0) return hipSuccess;
    constexpr size_t kLdsBytes = 3 * (size_t)(BM + BN) * 32 * sizeof(uint16_t);
    constexpr int kThreads = 64 * WAVES_M * WAVES_N;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void*)conv_igemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, GELU, SOURCES>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL((conv_igemm_dma_kernel<BM, BN, WAVES_M, WAVES_N, GELU, SOURCES>), dim3((unsigned)total), dim3(kThreads), kLdsBytes, stream,
                       (const uint16_t*)x, (const uint16_t*)wp, bias, (const uint16_t*)res, (uint16_t*)y, s, (int)M, tiles_n,
                       grp.table, grp.off_w, grp.off_b, from ? *from : Sources{});
    return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------------------------
// 3x3, stride 1, pad 1: the activation slab is loaded ONCE per 32-channel block and shared by the nine window
// positions.  Output pixels are numbered m = (n, p, q) flattened and, with "same" padding, input pixel (n, h, w) has
// the same number; window position (r, s) of output pixel m reads input pixel m + (r-1) W + (s-1) whenever that
// position is inside the image.  A tile of BM consecutive output pixels therefore needs the BM + 2W + 2 consecutive
// input pixels starting at m0 - W - 1: they are DMA'd into LDS as 16-row blocks (same swizzle as above) while the
// previous channel block is being computed, one block per wave and step.  Window positions outside the image are
// redirected to a 64-byte row of zeros; every lane keeps its nine LDS addresses per 32-row block in registers, so the
// inner loop has no address arithmetic beyond adding the slab buffer's base.  Filters: as above, three stages.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kSlabMaxW = 56;

template <int BM, int BN, int WAVES_M, int WAVES_N, int ACTS>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void conv3x3_slab_kernel(const uint16_t* __restrict__ x,
                                                                    const uint16_t* __restrict__ wp_all,
                                                                    const float* __restrict__ bias_all,
                                                                    const uint16_t* __restrict__ res,
                                                                    uint16_t* __restrict__ y, ConvShape s, int M,
                                                                    int tiles_n, GroupTable gt, uint32_t off_w, uint32_t off_b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BK = 32, KS = 2, kTaps = 9;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int MB = WM / 32, NB = WN / 32;
    constexpr int FRAG = 512;                                             // elements per 1 KiB block
    constexpr int SB_CAP = (BM + 2 * kSlabMaxW + 2 + 15) / 16;            // slab blocks per channel block (capacity)
    static_assert(SB_CAP <= 8 * NW, "the slab must be complete one step before it is used");
    constexpr int SLAB = SB_CAP * FRAG + 64;                              // + the row of zeros (32 elements) + padding
    constexpr int ZERO_OFF = SB_CAP * FRAG;                               // elements, inside either slab buffer
    constexpr int FB = BN / 32 * KS;
    static_assert(FB % NW == 0, "every wave issues the same number of loads");
    constexpr int B_PER_WAVE = FB / NW;
    constexpr int B_STAGE = FB * FRAG;
    constexpr int SPARE = 2 * SLAB;                                       // 1 KiB that absorbs the padding loads
    constexpr int B_BASE = SPARE + FRAG;
    // 64-row wave tiles have registers for two sets of operands: ALL operands of step u + 1 (filters too) are read while
    // step u is multiplied, so after a step's barrier the matrix cores start at once instead of waiting for the filter
    // reads.  A wave then keeps its SIMD's matrix core busy on its own, which matters whenever the other workgroup of the
    // compute unit is in its epilogue.  The filters then have to be in LDS one step earlier: four stages, loads three
    // steps ahead.
    constexpr bool kDeep = MB <= 2;

    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // 2 slabs | spare block | 3 or 4 filter stages

    int tile;
    {
        int L = blockIdx.x, total = gridDim.x;
        int xcd = L % kXcds, slot = L / kXcds;
        int base = total / kXcds, rem = total % kXcds;
        tile = xcd * base + (xcd < rem ? xcd : rem) + slot;
    }
    const TileOrigin org = locate_tile<BM>(tile, tiles_n, s.H * s.W, M, wp_all, bias_all, gt, off_w, off_b);
    const int m0 = org.m0, n0 = org.tile_n * BN;
    M = org.m_end;                                            // rows of this tile's group end here
    const uint16_t* const wp = org.wp;
    const float* const bias = org.bias;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;
    const int W = s.W, H = s.H;
    const int cblocks = s.C / BK;
    const int ks16_total = kTaps * cblocks * KS;
    const int total_px = s.N * H * W;
    const int slab_rows = BM + 2 * W + 2;

    const __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)total_px * (uint32_t)s.C * 2u);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(wp, (uint32_t)s.K * (uint32_t)(kTaps * s.C) * 2u);

    auto swz = [](int r16) { return ((r16 >> 1) & 3) ^ (r16 >> 3); };

    // the rows of zeros
    if (tid < 8) {
        *(u32x4*)(lds + ZERO_OFF + (tid & 3) * 8 + (tid >> 2) * SLAB) = u32x4{0u, 0u, 0u, 0u};
    }
    __syncthreads();

    // slab loader: row lane / 4 of a block, chunk chosen by the slot this lane fills
    const int ld_row = lane >> 2;
    const int ld_chunk = (lane & 3) ^ swz(ld_row);
    const int g_base = m0 - (W + 1) + ld_row;                 // input pixel of slab row ld_row
    auto issue_slab = [&](int cb, int tap, int parity) {
        const int sb = tap * NW + wid;                        // wave-uniform
        const int rho = sb * 16 + ld_row;
        const int g = g_base + sb * 16;
        const bool ok = sb < SB_CAP && cb < cblocks && rho < slab_rows && (unsigned)g < (unsigned)total_px;
        const uint32_t off = ok ? (uint32_t)((g * s.C + cb * BK + ld_chunk * 8) * 2) : kOutOfRange;
        uint16_t* dst = sb < SB_CAP ? lds + parity * SLAB + sb * FRAG : lds + SPARE;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void*)dst, 16, off, 0, 0, 0);
    };
    uint32_t b_off[B_PER_WAVE];
#pragma unroll
    for (int j = 0; j < B_PER_WAVE; ++j) {
        int fb = wid * B_PER_WAVE + j;
        b_off[j] = (uint32_t)((((n0 / 32 + fb / KS) * ks16_total + fb % KS) * FRAG + lane * 8) * 2);
    }
    auto issue_b = [&](int cb, int tap, int stage) {
        if (tap >= kTaps) { tap -= kTaps; ++cb; }
        if (cb >= cblocks) { cb = cblocks - 1; tap = kTaps - 1; }          // past the end: re-read the last step
        const uint32_t wstep = (uint32_t)((tap * cblocks + cb) * KS) * (FRAG * 2);
#pragma unroll
        for (int j = 0; j < B_PER_WAVE; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void*)(lds + B_BASE + stage * B_STAGE + (wid * B_PER_WAVE + j) * FRAG),
                                                     16, b_off[j], wstep, 0, 0);
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // prologue: the whole first slab, then filters of steps 0 and 1 (and 2) with one padding load between them so that
    // the order of outstanding loads is the steady-state one (slab piece, filters, slab piece, filters)
#pragma unroll
    for (int t = 0; t < (SB_CAP + NW - 1) / NW; ++t) issue_slab(0, t, 0);
    issue_b(0, 0, 0);
    issue_slab(cblocks, 8, 0);                                              // lands in the spare block
    issue_b(0, 1, 1);
    if (kDeep) {
        issue_slab(cblocks, 8, 0);
        issue_b(0, 2, 2);
    }

    // (built while the first loads are in flight)
    // operand addresses (elements, relative to a slab buffer) of this lane's pixel rows for the nine positions.
    // Slab row rho, chunk c sits at element 32 rho + 8 (c ^ f(rho & 15)) (16-row blocks of 512 elements are contiguous).
    // Kept free of branches and integer divisions: this runs once per tile and a 64-channel layer has only 18 steps
    // to amortise it over.  Pixel coordinates come from the tile's first pixel (one wave-uniform division) plus small
    // exact float divisions (numerators below 2^13, divisors up to 56^2).
    int32_t a_addr[MB][kTaps];
    {
        const int HW = H * W;
        const int pq0 = __builtin_amdgcn_readfirstlane(m0 % HW);
        const float inv_hw = 1.0f / (float)HW, inv_w = 1.0f / (float)W;
        const int khalf = lane >> 5;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int ml = wm * WM + i * 32 + (lane & 31);
            const int ok = (m0 + ml) < M;
            const int t0 = pq0 + ml;                                       // < H*W + BM
            const int pq = t0 - (int)(((float)t0 + 0.5f) * inv_hw) * HW;
            const int p = (int)(((float)pq + 0.5f) * inv_w), q = pq - p * W;
            const int row_in[3] = {ok & (p > 0), ok, ok & (p < H - 1)};
            const int col_in[3] = {q > 0, 1, q < W - 1};
#pragma unroll
            for (int rr = 0; rr < 3; ++rr)
#pragma unroll
                for (int tt = 0; tt < 3; ++tt) {
                    const int rho = ml + rr * W + tt;                      // = ml + (W + 1) + (rr - 1) W + (tt - 1)
                    const int chunk = (khalf ^ (rho >> 1) ^ ((rho >> 3) & 1)) & 3;
                    const int a = rho * 32 + chunk * 8;
                    a_addr[i][rr * 3 + tt] = (row_in[rr] & col_in[tt]) ? a : ZERO_OFF + khalf * 8;
                }
        }
    }

    // Activation operands of position tap+1 are read while position tap is multiplied: the slab does not change
    // inside a channel block, so only the filter operands have to wait for the step's barrier.  (With 128-row wave
    // tiles there are no registers left for that; there the reads of the second 16-channel half are slipped between
    // the matrix-core instructions of the first.)
    constexpr bool kAhead = MB <= 2;
    if constexpr (kDeep) {
        bf16x8 af[2][KS][MB], bfr[2][KS][NB];   // [step parity]
        auto read_a = [&](int par, const uint16_t* slab, int tap) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < MB; ++i) af[par][ks][i] = *(const bf16x8*)(slab + (a_addr[i][tap] ^ (ks * 16)));
        };
        auto read_b = [&](int par, int stage) {
            const uint16_t* b_lds = lds + B_BASE + stage * B_STAGE + (wn * NB * KS) * FRAG + lane * 8;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int j = 0; j < NB; ++j) bfr[par][ks][j] = *(const bf16x8*)(b_lds + (j * KS + ks) * FRAG);
        };
        // operands of step 0: its filters and the first slab have landed when all but the newest two steps' loads have
        wait_before_barrier<2 * (1 + B_PER_WAVE)>();
        __builtin_amdgcn_s_barrier();
        read_a(0, lds, 0);
        read_b(0, 0);
        static_assert(SB_CAP <= 7 * NW, "the next slab is complete one step before its first operands are read ahead");
        int stage_rd = 1, stage_ld = 3;          // stage of the NEXT step's filters; stage the loads three steps ahead go to
        // one step; TAP and the register set CUR of its operands are compile-time (a channel block has nine positions, so
        // the sets swap roles from one block to the next: blocks are walked in pairs)
        auto step = [&](auto tap_c, auto cur_c, int cb) {
            constexpr int tap = decltype(tap_c)::value, cur = decltype(cur_c)::value, nxt = cur ^ 1;
            constexpr int kReads = KS * MB + KS * NB, kMfma = KS * MB * NB;
            const bool more = cb + 1 < cblocks;
            // the filters of the next step (and, at a channel block's last position, the whole next slab: its last piece
            // was issued at least two steps ago) have landed; only this wave's newest loads may still be in flight
            wait_before_barrier<1 + B_PER_WAVE>();
            __builtin_amdgcn_s_barrier();
            issue_slab(cb + 1, tap, (cb + 1) & 1);
            issue_b(cb, tap + 3, stage_ld);
            // operands of the next step: next position of this channel block, or position 0 of the next block
            if (tap + 1 < kTaps) { read_a(nxt, lds + (cb & 1) * SLAB, tap + 1); read_b(nxt, stage_rd); }
            else if (more) { read_a(nxt, lds + ((cb + 1) & 1) * SLAB, 0); read_b(nxt, stage_rd); }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cur][ks][j], af[cur][ks][i], acc[i][j], 0, 0, 0);
            // issue order inside the step (0x100 = LDS read, 0x008 = matrix core): matrix-core instructions from the start,
            // the next step's operand reads slipped in between them one by one
            if (tap + 1 < kTaps || more) {
#pragma unroll
                for (int t = 0; t < (kReads < kMfma ? kReads : kMfma); ++t) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                if (kReads > kMfma) __builtin_amdgcn_sched_group_barrier(0x100, kReads - kMfma, 0);
                if (kReads < kMfma) __builtin_amdgcn_sched_group_barrier(0x008, kMfma - kReads, 0);
            } else {
                __builtin_amdgcn_sched_group_barrier(0x008, kMfma, 0);
            }
            stage_rd = (stage_rd + 1) & 3;
            stage_ld = (stage_ld + 1) & 3;
        };
        auto block = [&](auto first_c, int cb) {        // the nine positions of channel block cb, starting in register set FIRST
            constexpr int f = decltype(first_c)::value;
            step(std::integral_constant<int, 0>{}, std::integral_constant<int, f>{}, cb);
            step(std::integral_constant<int, 1>{}, std::integral_constant<int, f ^ 1>{}, cb);
            step(std::integral_constant<int, 2>{}, std::integral_constant<int, f>{}, cb);
            step(std::integral_constant<int, 3>{}, std::integral_constant<int, f ^ 1>{}, cb);
            step(std::integral_constant<int, 4>{}, std::integral_constant<int, f>{}, cb);
            step(std::integral_constant<int, 5>{}, std::integral_constant<int, f ^ 1>{}, cb);
            step(std::integral_constant<int, 6>{}, std::integral_constant<int, f>{}, cb);
            step(std::integral_constant<int, 7>{}, std::integral_constant<int, f ^ 1>{}, cb);
            step(std::integral_constant<int, 8>{}, std::integral_constant<int, f>{}, cb);
        };
        for (int cb = 0; cb < cblocks; cb += 2) {
            block(std::integral_constant<int, 0>{}, cb);
            if (cb + 1 < cblocks) block(std::integral_constant<int, 1>{}, cb + 1);
        }
    } else
    for (int cb = 0; cb < cblocks; ++cb) {
        const uint16_t* slab = lds + (cb & 1) * SLAB;
        bf16x8 af[2][KS][MB];               // [tap parity]
#pragma unroll
        for (int tap = 0; tap < kTaps; ++tap) {
            wait_before_barrier<1 + B_PER_WAVE>();      // everything up to this step's filters has landed
            __builtin_amdgcn_s_barrier();
            issue_slab(cb + 1, tap, (cb + 1) & 1);
            issue_b(tap + 2 < kTaps ? cb : cb + 1, (tap + 2) % kTaps, (tap + 2) % 3);
            const uint16_t* b_lds = lds + B_BASE + (tap % 3) * B_STAGE + (wn * NB * KS) * FRAG + lane * 8;
            bf16x8 bfr[KS][NB];
            if (!kAhead || tap == 0) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int i = 0; i < MB; ++i) af[tap & 1][ks][i] = *(const bf16x8*)(slab + (a_addr[i][tap] ^ (ks * 16)));
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int j = 0; j < NB; ++j) bfr[ks][j] = *(const bf16x8*)(b_lds + (j * KS + ks) * FRAG);
            if (kAhead && tap + 1 < kTaps) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
                        af[(tap + 1) & 1][ks][i] = *(const bf16x8*)(slab + (a_addr[i][tap + 1] ^ (ks * 16)));
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks][j], af[tap & 1][ks][i], acc[i][j], 0, 0, 0);
            // issue order inside the step (0x100 = LDS read, 0x008 = matrix core)
            if (kAhead) {
                // this step's operands first (filters; at position 0 also the activations), then the matrix-core
                // instructions with the next position's activation reads slipped in between
                if (tap == 0) __builtin_amdgcn_sched_group_barrier(0x100, KS * NB + KS * MB, 0);
                else __builtin_amdgcn_sched_group_barrier(0x100, KS * NB, 0);
                if (tap + 1 < kTaps) {
#pragma unroll
                    for (int t = 0; t < KS * MB; ++t) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, KS * MB * NB - KS * MB, 0);
                } else {
                    __builtin_amdgcn_sched_group_barrier(0x008, KS * MB * NB, 0);
                }
            } else {
                // the operands of the first 16-channel half, then matrix-core instructions with the reads of the second
                // half slipped in between them
                __builtin_amdgcn_sched_group_barrier(0x100, MB + NB, 0);
#pragma unroll
                for (int t = 0; t < MB + NB; ++t) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, KS * MB * NB - (MB + NB), 0);
            }
        }
    }
    wait_before_barrier<0>();
    __builtin_amdgcn_s_barrier();        // every wave is done with the operand stages: LDS is free for the epilogue
    store_tile_via_lds<ACTS, MB, NB>(acc, lds + wid * (32 * (WN + 8)), bias, res, y, m0 + wm * WM, n0 + wn * WN, M, s.K, s.act, lane);
#endif
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int ACTS = kActsPlain>
hipError_t launch_slab(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                       hipStream_t stream, const Grouping& grp = Grouping())
{
    if constexpr (ACTS == kActsPlain) {
        if (s.act == 2) return launch_slab<BM, BN, WAVES_M, WAVES_N, kActsGelu>(x, wp, bias, res, y, s, stream, grp);
        if (s.act == 3) return launch_slab<BM, BN, WAVES_M, WAVES_N, kActsSilu>(x, wp, bias, res, y, s, stream, grp);
    }
    long long M = (long long)s.N * s.P * s.Q;
    int tiles_n = s.K / BN;
    long long total = count_tiles(M, (long long)s.P * s.Q, BM, tiles_n, grp.table);
    if (total > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (total == 0) return hipSuccess;
    constexpr int kSbCap = (BM + 2 * kSlabMaxW + 2 + 15) / 16;
    constexpr int kStagesB = (BM / WAVES_M) / 32 <= 2 ? 4 : 3;             // as in the kernel: 64-row wave tiles read one step ahead
    constexpr size_t kLdsBytes = (2 * (size_t)(kSbCap * 512 + 64) + 512 + kStagesB * (size_t)BN * 32) * sizeof(uint16_t);
    constexpr int kThreads = 64 * WAVES_M * WAVES_N;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute((const void*)conv3x3_slab_kernel<BM, BN, WAVES_M, WAVES_N, ACTS>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e != hipSuccess) return e;
        configured = true;
    }
    hipLaunchKernelGGL((conv3x3_slab_kernel<BM, BN, WAVES_M, WAVES_N, ACTS>), dim3((unsigned)total), dim3(kThreads), kLdsBytes, stream,
                       (const uint16_t*)x, (const uint16_t*)wp, bias, (const uint16_t*)res, (uint16_t*)y, s, (int)M, tiles_n,
                       grp.table, grp.off_w, grp.off_b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Few output tiles: with a handful of requests the kernels above leave most of the chip idle (512 filters over the 49
// pixels of one 7 x 7 image are four 256 x 128 tiles) and each of their few workgroups walks the whole reduction with
// its loads only two short steps ahead.  Splitting the reduction would change the order of the sums, and with it the
// bits of a request's result with the number of requests that happen to run beside it; so the tile shrinks instead and
// the loads run further ahead.  Same operands and same order of accumulation as the kernel that the
// shape otherwise takes (slab_order: channel blocks outside, window positions inside), hence the same bits.
//   * STAGES stages of UN 32-channel steps each in LDS, all but two of them in flight; one barrier per stage.
//   * operands of a stage are read into registers while the stage before it is multiplied, and the loads of a later one issued,
//     each between two products: a wave issues in order, and what stands in front of the products delays them.  us, 64 x 64
//     tiles, reads, then loads, then products / this order: 3072 -> 768, 985 rows 16.0 / 13.9; 3x3 stride 2, 256 -> 512 on 14 x 14, 29 images
//     13.4 / 11.2; 3x3 stride 1, 512 -> 512 on 7 x 7, 29 images 14.1 / 13.2; but 3x3, 64 -> 256 on 14 x 14, 30 images 6.7 / 6.85.
//   * 32 x 32 tiles are four wavefronts of 16 x 16 (T = 16): a product of 16 x 16 x 32 sums in the order of two of 32 x 32 x 16 one after the
//     other (also with exponents far apart, cancelling terms and denormals) and the chain of them, which bounds a tile of one wavefront (144
//     steps of 64 cycles where 512 channels go into a 3x3 window), takes a quarter of the time; a step's four loads are one per
//     wavefront, so more of them are in flight; bias and residual are fetched first and 8-byte stores leave straight from the
//     accumulators.  us per launch, one image, a tile of one wavefront / of four: 3x3 512 -> 512 on 7 x 7 9.3 / 8.1, 256 -> 256 on
//     14 x 14 7.2 / 6.3, 128 -> 128 on 28 x 28 5.6 / 5.2, 64 -> 64 on 56 x 56 4.9 / 4.5; one ResNet-18 request 297 / 268.
//   * row tiles run fastest: the workgroups of one XCD take all rows of a few filter tiles, so filters - most of the
//     bytes here - come from memory once and not once per XCD.
// ---------------------------------------------------------------------------------------------------------------
template <int BEGIN, int END, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (BEGIN < END) {
        f(std::integral_constant<int, BEGIN>{});
        static_for<BEGIN + 1, END>(f);
    }
}

constexpr int kRingWaves = 4;

// The other convolution of a launch that does two (PAIR): its tiles follow the first one's
struct RingSecond {
    ConvShape s;
    int32_t M, tiles_n;
    uint32_t off_w, off_b;
    uint32_t first_tiles;      // tiles of the first convolution
};

template <bool SLAB_ORDER, int T, int UN, int STAGES, int ACTS, bool PAIR, bool SOURCES>
__global__ __launch_bounds__(64 * kRingWaves) void conv_igemm_ring_kernel(const uint16_t* __restrict__ x,
                                                                   const uint16_t* __restrict__ wp_all,
                                                                   const float* __restrict__ bias_all,
                                                                   const uint16_t* __restrict__ res,
                                                                   uint16_t* __restrict__ y, ConvShape s, int M,
                                                                   int tiles_n, GroupTable gt, uint32_t off_w, uint32_t off_b,
                                                                   const uint16_t* __restrict__ x2, const uint16_t* __restrict__ wp2,
                                                                   const float* __restrict__ bias2, const uint16_t* __restrict__ res2,
                                                                   uint16_t* __restrict__ y2, RingSecond second, Sources from)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BK = 32, KS = 2;
    constexpr bool QUARTERS = T == 16;
    constexpr int BM = 2 * T, BN = 2 * T;                     // waves 2 x 2, T x T accumulators each
    constexpr int FA = BM / 16, FB = BN / 32 * KS;            // 1 KiB blocks per step
    // every wave issues the same number of loads: of a step's 4 KiB in quarters one block each (two waves pixel rows, two filters)
    static_assert(QUARTERS ? FA + FB == kRingWaves : FA == kRingWaves && FB == kRingWaves, "blocks of a step");
    constexpr int PER_STEP = QUARTERS ? 1 : 2;
    constexpr int LOADS = UN * PER_STEP;                      // of a wave and stage
    constexpr int FRAG = 512;                                 // elements per 1 KiB block
    constexpr int STEP = (FA + FB) * FRAG, STAGE = UN * STEP;
    static_assert(STAGES >= 3 && (STAGES - 2) * LOADS <= 63, "what is in flight at a wait fits its counter");

    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // STAGES * STAGE elements

    int tile;
    {
        int L = blockIdx.x, total = gridDim.x;
        if (PAIR) {
            const int first = (int)second.first_tiles;
            const bool is_second = L >= first;
            L = is_second ? L - first : L;
            total = is_second ? total - first : first;
            x = is_second ? x2 : x;
            wp_all = is_second ? wp2 : wp_all;
            bias_all = is_second ? bias2 : bias_all;
            res = is_second ? res2 : res;
            y = is_second ? y2 : y;
            // (member by member: a choice between the two structures would go through scratch memory)
            auto pick = [&](int32_t& a, int32_t b) { a = is_second ? b : a; };
            pick(s.N, second.s.N); pick(s.H, second.s.H); pick(s.W, second.s.W); pick(s.C, second.s.C);
            pick(s.K, second.s.K); pick(s.R, second.s.R); pick(s.S, second.s.S); pick(s.stride, second.s.stride);
            pick(s.pad, second.s.pad); pick(s.P, second.s.P); pick(s.Q, second.s.Q); pick(s.act, second.s.act);
            M = is_second ? second.M : M;
            tiles_n = is_second ? second.tiles_n : tiles_n;
            off_w = is_second ? second.off_w : off_w;
            off_b = is_second ? second.off_b : off_b;
        }
        int xcd = L % kXcds, slot = L / kXcds;
        int base = total / kXcds, rem = total % kXcds;
        tile = xcd * base + (xcd < rem ? xcd : rem) + slot;
    }
    const int PQ = s.P * s.Q;
    int m_first = 0;
    const uint16_t* wp = wp_all;
    const float* bias = bias_all;
    int g = 0, tiles_m = (M + BM - 1) / BM;
    if (gt.n > 0) {
        for (;; ++g) {                                        // the launch has exactly sum-of-tiles workgroups
            tiles_m = ((gt.first_row[g + 1] - gt.first_row[g]) * PQ + BM - 1) / BM;
            if (tile < tiles_m * tiles_n || g + 1 >= gt.n) break;
            tile -= tiles_m * tiles_n;
        }
        m_first = gt.first_row[g] * PQ;
        M = gt.first_row[g + 1] * PQ;
        wp = (const uint16_t*)((const char*)gt.weights[g] + off_w);
        bias = (const float*)((const char*)gt.weights[g] + off_b);
    }
    const int m0 = m_first + (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / 2, wn = wid % 2;

    const int cblocks = s.C / BK;
    const int RS = s.R * s.S;
    const int ks16_total = RS * cblocks * KS;

    __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(wp, (uint32_t)s.K * (uint32_t)(RS * s.C) * 2u);

    auto swz = [](int r16) { return ((r16 >> 1) & 3) ^ (r16 >> 3); };
    // Byte offset of this lane's piece of an activation row, out of range where the window position is outside the image:
    // for all nine positions at once in slab order, else for the position that is being fetched.  The channel block is
    // a scalar offset, so a load needs no vector arithmetic (a wave's instruction issue is what bounds these tiles).
    constexpr int kPos = SLAB_ORDER ? 9 : 1;
    constexpr int kParts = SLAB_ORDER ? 9 / UN : 1;           // stages per channel block (slab order)
    static_assert(!SLAB_ORDER || 9 % UN == 0, "whole stages per channel block");
    uint32_t a_at[kPos];
    int32_t a_off, a_ih, a_iw;
    auto place = [&](int rr, int tt) __attribute__((always_inline)) -> uint32_t {
        const bool in = (unsigned)(a_ih + rr) < (unsigned)s.H && (unsigned)(a_iw + tt) < (unsigned)s.W;
        return in ? (uint32_t)(a_off + (rr * s.W + tt) * s.C * 2) : kOutOfRange;
    };
    const bool rows = !QUARTERS || wid < FA;                  // this wave fetches pixel rows
    {
        const int chunk = (lane & 3) ^ swz(lane >> 2);
        const int m = m0 + wid * 16 + (lane >> 2);
        const bool ok = m < M && rows;
        const int mm = ok ? m : 0;
        const int n = mm / PQ, pq = mm % PQ;
        const int p = pq / s.Q, q = pq % s.Q;
        a_ih = ok ? p * s.stride - s.pad : -0x10000;          // a row past the end: no position is inside
        a_iw = q * s.stride - s.pad;
        a_off = ((n * s.H + p * s.stride - s.pad) * s.W + a_iw) * s.C * 2 + chunk * 16;
#pragma unroll
        for (int i = 0; i < kPos; ++i) a_at[i] = place(i / 3, i % 3);
    }
    const int fb = QUARTERS ? (rows ? 0 : wid - FA) : wid;    // filter fragment of this wave
    const uint32_t b_off = (uint32_t)((((n0 / 32 + fb / KS) * ks16_total + fb % KS) * FRAG + lane * 8) * 2);
    // in quarters a wave has one kind of load: descriptor and lane offsets are picked once, the scalar offset per load
    __amdgpu_buffer_rsrc_t own_rsrc = rows ? x_rsrc : w_rsrc;
    if (!rows)
#pragma unroll
        for (int i = 0; i < kPos; ++i) a_at[i] = b_off;

    // the stage that is fetched next: scalar offsets of its first channel block in a row and of its first filter fragment
    uint32_t f_c = 0, f_w = 0, r_pos = 0, t_pos = 0;
    const uint32_t c_end = (uint32_t)s.C * 2, tap_w = (uint32_t)cblocks * (KS * FRAG * 2);
    // part (slab order): which UN of the nine positions
    auto load_one = [&](auto part_c, auto k_c, int stage) __attribute__((always_inline)) {
        constexpr int part = decltype(part_c)::value, u = decltype(k_c)::value / PER_STEP, j = decltype(k_c)::value % PER_STEP;
        uint16_t* const st = lds + stage * STAGE + u * STEP;
        const uint32_t at = a_at[SLAB_ORDER ? part * UN + u : 0];
        const uint32_t c_at = SLAB_ORDER ? f_c : f_c + u * (BK * 2), w_at = SLAB_ORDER ? f_w + (part * UN + u) * tap_w : f_w + u * (KS * FRAG * 2);
        if constexpr (QUARTERS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(own_rsrc, (lds_void*)(st + wid * FRAG), 16, at, rows ? c_at : w_at, 0, 0);
        else if constexpr (j == 0)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void*)(st + wid * FRAG), 16, at, c_at, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void*)(st + (FA + wid) * FRAG), 16, b_off, w_at, 0, 0);
    };
    auto advance = [&](auto part_c) __attribute__((always_inline)) {
        constexpr int part = decltype(part_c)::value;
        // past the last stage the position stays put: what is fetched there is never used
        if (SLAB_ORDER) {
            if (part == kParts - 1 && f_c + BK * 2 < c_end) { f_c += BK * 2; f_w += KS * FRAG * 2; }
        } else if (f_c + UN * BK * 2 < c_end) {
            f_c += UN * BK * 2;
            f_w += UN * KS * FRAG * 2;
        } else {                                              // on to the next window position
            const bool row_end = t_pos + 1 == (uint32_t)s.S;
            if (!row_end || r_pos + 1 < (uint32_t)s.R) {
                t_pos = row_end ? 0 : t_pos + 1;
                r_pos = row_end ? r_pos + 1 : r_pos;
                f_c = 0;
                f_w += UN * KS * FRAG * 2;
                if (SOURCES) {
                    x_rsrc = make_rsrc(source_at(x, from, (int)r_pos), (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
                    own_rsrc = rows ? x_rsrc : w_rsrc;
                } else if (rows) {
                    a_at[0] = place(r_pos, t_pos);
                }
            }
        }
    };

    // Operands.  In quarters a product takes a whole step: lane l holds pixel row (and filter) l % 16 and the 8 channels l / 16 of 32.
    constexpr int PRODUCTS = QUARTERS ? 1 : KS;               // of a step
    std::conditional_t<QUARTERS, f32x4, f32x16> acc;
#pragma unroll
    for (int v = 0; v < (QUARTERS ? 4 : 16); ++v) acc[v] = 0.f;
    const int l16 = lane & 15, g16 = lane >> 4;
    const int rd_row = lane & 31;
    const int rd_a = QUARTERS ? wm * FRAG + (l16 * 4 + (g16 ^ swz(l16))) * 8
                              : (wm * 2 + (rd_row >> 4)) * FRAG + ((rd_row & 15) * 4 + ((lane >> 5) ^ swz(rd_row & 15))) * 8;
    const int rd_b = QUARTERS ? (FA + (g16 >> 1)) * FRAG + ((g16 & 1) * 32 + wn * 16 + l16) * 8 : (FA + wn * KS) * FRAG + lane * 8;
    bf16x8 af[2][UN][PRODUCTS], bfr[2][UN][PRODUCTS];         // [stage parity]
    constexpr int kReads = UN * PRODUCTS * 2, kMfma = UN * PRODUCTS;
    auto read_one = [&](auto set_c, auto k_c, int stage) __attribute__((always_inline)) {
        constexpr int set = decltype(set_c)::value, k = decltype(k_c)::value, u = k / (PRODUCTS * 2), ks = k / 2 % PRODUCTS;
        const uint16_t* const st = lds + stage * STAGE + u * STEP;
        if constexpr (k % 2 == 0) af[set][u][ks] = *(const bf16x8*)(st + (rd_a ^ (ks * 16)));
        else bfr[set][u][ks] = *(const bf16x8*)(st + rd_b + ks * FRAG);
    };
    auto multiply_one = [&](auto set_c, auto k_c) __attribute__((always_inline)) {
        constexpr int set = decltype(set_c)::value, k = decltype(k_c)::value, u = k / PRODUCTS, ks = k % PRODUCTS;
        if constexpr (QUARTERS) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[set][u][ks], af[set][u][ks], acc, 0, 0, 0);
        else acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][u][ks], af[set][u][ks], acc, 0, 0, 0);
    };
    // in quarters the bias and the residual are fetched before everything else
    const int q_px = m0 + wm * 16 + l16, q_f = n0 + wn * 16 + g16 * 4;
    float4 q_bias = make_float4(0.f, 0.f, 0.f, 0.f);
    uint2 q_res = make_uint2(0u, 0u);
    if constexpr (QUARTERS) {
        q_bias = *(const float4*)(bias + q_f);
        if (res && q_px < M) q_res = *(const uint2*)(res + (size_t)q_px * s.K + q_f);
    }

    typedef std::integral_constant<int, 0> c0;
    typedef std::integral_constant<int, 1> c1;
    // stages are fetched in order; in slab order stage k holds part k % kParts of channel block k / kParts
    static_for<0, STAGES - 1>([&](auto k) __attribute__((always_inline)) {
        typedef std::integral_constant<int, decltype(k)::value % kParts> part;
        static_for<0, LOADS>([&](auto l) __attribute__((always_inline)) { load_one(part{}, l, decltype(k)::value); });
        advance(part{});
    });
    wait_before_barrier<(STAGES - 2) * LOADS>();
    __builtin_amdgcn_s_barrier();
    static_for<0, kReads>([&](auto k) __attribute__((always_inline)) { read_one(c0{}, k, 0); });
    // body of stage i: the loads of stage i + 1 have landed (its successors may be in flight) | barrier | stage i + STAGES - 1
    // goes where stage i - 1 was: every wave has its operands in registers since before this barrier | operands of stage
    // i + 1 | products of stage i.  Past the end stale stages are read into registers that nothing uses.
    int next = 1, fill = STAGES - 1;
    auto body = [&](auto part_c, auto cur_c, auto nxt_c) __attribute__((always_inline)) {
        constexpr int part = decltype(part_c)::value;
        wait_before_barrier<(STAGES - 3) * LOADS>();
        __builtin_amdgcn_s_barrier();
        typedef std::integral_constant<int, (part + STAGES - 1) % kParts> fill_part;
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, kMfma>([&](auto m_c) __attribute__((always_inline)) {
            constexpr int m = decltype(m_c)::value;
            multiply_one(cur_c, m_c);
            __builtin_amdgcn_sched_barrier(0);
            static_for<kReads * m / kMfma, kReads * (m + 1) / kMfma>([&](auto k) __attribute__((always_inline)) { read_one(nxt_c, k, next); });
            static_for<LOADS * m / kMfma, LOADS * (m + 1) / kMfma>([&](auto l) __attribute__((always_inline)) { load_one(fill_part{}, l, fill); });
            __builtin_amdgcn_sched_barrier(0);
        });
        advance(fill_part{});
        next = next == STAGES - 1 ? 0 : next + 1;
        fill = fill == STAGES - 1 ? 0 : fill + 1;
    };
    if constexpr (SLAB_ORDER) {
        for (int cb = 0; cb < cblocks; cb += 2) {             // kParts is odd: register sets swap roles from block to block
            static_for<0, kParts>([&](auto k) __attribute__((always_inline)) {
                constexpr int set = decltype(k)::value & 1;
                body(k, std::integral_constant<int, set>{}, std::integral_constant<int, set ^ 1>{});
            });
            if (cb + 1 == cblocks) break;
            static_for<0, kParts>([&](auto k) __attribute__((always_inline)) {
                constexpr int set = decltype(k)::value & 1;
                body(k, std::integral_constant<int, set ^ 1>{}, std::integral_constant<int, set>{});
            });
        }
    } else {
        const int n_stages = RS * cblocks / UN;               // the launcher picks UN so that it divides the channel blocks
        for (int i = 0; i < n_stages; i += 2) {
            body(c0{}, c0{}, c1{});
            if (i + 1 == n_stages) break;
            body(c0{}, c1{}, c0{});
        }
    }
    wait_before_barrier<0>();
    if constexpr (QUARTERS) {
        with_activation<ACTS>(s.act, [&](auto a) {
            float v[4] = {acc[0] + q_bias.x, acc[1] + q_bias.y, acc[2] + q_bias.z, acc[3] + q_bias.w};
            if (res) {
                v[0] += bf16_to_f32(q_res.x & 0xFFFFu); v[1] += bf16_to_f32(q_res.x >> 16);
                v[2] += bf16_to_f32(q_res.y & 0xFFFFu); v[3] += bf16_to_f32(q_res.y >> 16);
            }
            activate<decltype(a)::value>(v);
            if (q_px < M) *(uint2*)(y + (size_t)q_px * s.K + q_f) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        });
    } else {
        __builtin_amdgcn_s_barrier();    // every wave is done with the operand stages: LDS is free for the epilogue
        f32x16 (&tile_acc)[1][1] = reinterpret_cast<f32x16 (&)[1][1]>(acc);
        store_tile_via_lds<ACTS, 1, 1>(tile_acc, lds + wid * (32 * (T + 8)), bias, res, y, m0 + wm * T, n0 + wn * T, M, s.K, s.act, lane);
    }
#endif
}

struct ConvArgs {
    const void *x, *wp;
    const float* bias;
    const void* res;
    void* y;
    ConvShape s;
    Grouping grp;
    const Sources* from = nullptr;      // a concatenation: its maps after x
};

// b != nullptr: a second convolution, over the same groups, in the same launch
template <bool SLAB_ORDER, int T, int UN, int STAGES, int ACTS = kActsPlain, bool PAIR = false, bool SOURCES = false>
hipError_t launch_ring(const ConvArgs& a, hipStream_t stream, const ConvArgs* b = nullptr)
{
    if constexpr (ACTS == kActsPlain) {                       // (pairs and sources, which never have GELU: the others in one)
        if constexpr (!SLAB_ORDER) {
            if (a.from) return launch_ring<SLAB_ORDER, T, UN, STAGES, kActsElse, false, true>(a, stream);
            if (b) return launch_ring<SLAB_ORDER, T, UN, STAGES, kActsElse, true>(a, stream, b);
        }
        if (a.s.act == 2) return launch_ring<SLAB_ORDER, T, UN, STAGES, kActsGelu>(a, stream);
        if (a.s.act == 3) return launch_ring<SLAB_ORDER, T, UN, STAGES, kActsSilu>(a, stream);
    }
    constexpr int BM = 2 * T, BN = 2 * T;
    const long long M = (long long)a.s.N * a.s.P * a.s.Q;
    long long total = count_tiles(M, (long long)a.s.P * a.s.Q, BM, a.s.K / BN, a.grp.table);
    RingSecond second{};
    if (PAIR) {
        const long long M2 = (long long)b->s.N * b->s.P * b->s.Q;
        second = {b->s, (int32_t)M2, b->s.K / BN, b->grp.off_w, b->grp.off_b, (uint32_t)total};
        total += count_tiles(M2, (long long)b->s.P * b->s.Q, BM, b->s.K / BN, b->grp.table);
    }
    if (total > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (total == 0) return hipSuccess;
    constexpr size_t kLdsBytes = STAGES * UN * (size_t)(BM + BN) * 32 * sizeof(uint16_t);
    static_assert(kLdsBytes <= 160 * 1024 && kLdsBytes >= (T == 16 ? 0 : (size_t)kRingWaves * 32 * (T + 8) * 2), "operand stages and epilogue rows");
    static const hipError_t configured = hipFuncSetAttribute((const void*)conv_igemm_ring_kernel<SLAB_ORDER, T, UN, STAGES, ACTS, PAIR, SOURCES>,
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
    if (configured != hipSuccess) return configured;
    hipLaunchKernelGGL((conv_igemm_ring_kernel<SLAB_ORDER, T, UN, STAGES, ACTS, PAIR, SOURCES>), dim3((unsigned)total), dim3(64 * kRingWaves),
                       kLdsBytes, stream, (const uint16_t*)a.x, (const uint16_t*)a.wp, a.bias, (const uint16_t*)a.res, (uint16_t*)a.y, a.s, (int)M,
                       a.s.K / BN, a.grp.table, a.grp.off_w, a.grp.off_b, b ? (const uint16_t*)b->x : nullptr, b ? (const uint16_t*)b->wp : nullptr,
                       b ? b->bias : nullptr, b ? (const uint16_t*)b->res : nullptr, b ? (uint16_t*)b->y : nullptr, second, a.from ? *a.from : Sources{});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Long GEMM-like launches (token GEMMs, 1x1 and strided convolutions with long reductions): tiles of 64 MB x 256 of eight
// wavefronts, 32 MB x 64 each (MB = 4: 256 x 256), by workgroups that stay for several tiles, one per compute unit.
// What bounds it: with 0.75 KiB of operand reads per matrix-core instruction the LDS moves 96 B/clk of reads and 32 B/clk of
// arriving loads when the matrix cores run at their full rate, which is all it can do; timing copies on 3072 -> 768 over
// 76,633 rows (us): matrix cores only 207, with operand reads 288, with loads 310, with both 380, so what counts is that
// the three overlap.  A wave issues in order and stalls where a queue is full: a run of reads or loads in front of the
// matrix-core instructions leaves these waiting.  Hence the fixed order inside a half step (one read or load after each
// matrix-core instruction), and loads of filters and of pixel rows in different halves.
//   * A step is 32 channels, its two 16-channel halves alternate: the operands of one are read while the other is
//     multiplied; in the middle of a step one barrier says that the next stage has landed and this one has been read.
//   * Three stages; the fetches run on into the next tile, so a tile starts with its operands in LDS and the epilogue
//     of the tile before, with the stores still on their way, costs no pipeline start.
// Measured, us (128 x 128 tiles of conv_igemm_dma_kernel / here), 76,633 rows: 768 -> 2304 434 / 324 (0.84 PFLOP/s),
// 768 -> 768 with residual 154 / 122, 3072 -> 768 with residual 447 / 337 (1.07 PFLOP/s); 25,216 rows: 768 -> 2304 112 / 87;
// 256 images: 1x1 1024 -> 256 on 14 x 14 39 / 30; 3x3 stride 2, 512 images: 256 -> 512 on 14 x 14 78 / 58.
// ---------------------------------------------------------------------------------------------------------------
// Epilogue with an exact number of memory operations: MB * T stores (and loads, with a residual) per wave, rows past the end
// dropped by the buffer's range check.
template <int MB, int NB, int ACT, bool RES>
__device__ __forceinline__ void store_tile_counted_act(f32x16 (&acc)[MB][NB], uint16_t* stage, const float* __restrict__ bias,
                                                       __amdgpu_buffer_rsrc_t res, __amdgpu_buffer_rsrc_t y, int m_wave, int n_wave,
                                                       int M, int K, int lane)
{
    constexpr int WN = NB * 32, ROW = WN + 8;
    constexpr int CPR = WN / 8;
    constexpr int T = 32 * CPR / 64;
    constexpr int kQuads = ACT >= 2 ? 2 : 1;               // accumulator quads that are finished together: GELU and SiLU share a test
    const int frag_row = lane & 31, f_hi = (lane >> 5) * 4;
    auto at = [&](int i, int t) -> uint32_t {
        const int idx = lane + 64 * t, mo = m_wave + i * 32 + idx / CPR;
        return mo < M ? ((uint32_t)mo * (uint32_t)K + (uint32_t)(n_wave + (idx % CPR) * 8)) * 2u : kOutOfRange;
    };
    float* const bl = (float*)(stage + 32 * ROW);             // the wave's bias values, next to its rows
    static_assert(WN == 64, "one bias value per lane");
    bl[lane] = bias[n_wave + lane];
    u32x4 rres[2][T];
    if (RES) {
#pragma unroll
        for (int t = 0; t < T; ++t) rres[0][t] = __builtin_amdgcn_raw_buffer_load_b128(res, at(0, t), 0, 0);
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (RES) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int idx = lane + 64 * t;
                *(u32x4*)(stage + (idx / CPR) * ROW + (idx % CPR) * 8) = rres[i & 1][t];
                if (i + 1 < MB) rres[(i + 1) & 1][t] = __builtin_amdgcn_raw_buffer_load_b128(res, at(i + 1, t), 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
#pragma unroll
            for (int g = 0; g < 4; g += kQuads) {
                float v[4 * kQuads];
#pragma unroll
                for (int h = 0; h < kQuads; ++h) {
                    const int nl = j * 32 + 8 * (g + h) + f_hi;
                    const float4 bv = *(const float4*)(bl + nl);
                    v[4 * h] = acc[i][j][4 * (g + h)] + bv.x; v[4 * h + 1] = acc[i][j][4 * (g + h) + 1] + bv.y;
                    v[4 * h + 2] = acc[i][j][4 * (g + h) + 2] + bv.z; v[4 * h + 3] = acc[i][j][4 * (g + h) + 3] + bv.w;
                    if (RES) {
                        const uint2 rv = *(const uint2*)(stage + frag_row * ROW + nl);
                        v[4 * h] += bf16_to_f32(rv.x & 0xFFFFu); v[4 * h + 1] += bf16_to_f32(rv.x >> 16);
                        v[4 * h + 2] += bf16_to_f32(rv.y & 0xFFFFu); v[4 * h + 3] += bf16_to_f32(rv.y >> 16);
                    }
                }
                activate<ACT>(v);
#pragma unroll
                for (int h = 0; h < kQuads; ++h)
                    *(uint2*)(stage + frag_row * ROW + j * 32 + 8 * (g + h) + f_hi) =
                        make_uint2(pack_bf16(v[4 * h], v[4 * h + 1]), pack_bf16(v[4 * h + 2], v[4 * h + 3]));
            }
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int idx = lane + 64 * t;
            const u32x4 v = *(const u32x4*)(stage + (idx / CPR) * ROW + (idx % CPR) * 8);
            __builtin_amdgcn_raw_buffer_store_b128(v, y, at(i, t), 0, 0);
        }
    }
}

template <bool ROWS, int MB, int NB, int WAVES_M, int WAVES_N, int ACTS, bool SOURCES>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 2) void conv_gemm_persistent_kernel(const uint16_t* __restrict__ x,
                                                                   const uint16_t* __restrict__ wp_all,
                                                                   const float* __restrict__ bias_all,
                                                                   const uint16_t* __restrict__ res,
                                                                   uint16_t* __restrict__ y, ConvShape s, int M_all,
                                                                   int tiles_n, int total, GroupTable gt, uint32_t off_w, uint32_t off_b, Sources from)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BK = 32, KS = 2, STAGES = 3;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = 32 * MB, WN = 32 * NB, BM = WM * WAVES_M, BN = WN * WAVES_N;
    // every wave issues the same number of loads; blocks of rows past the tile's last read nothing and fill spare LDS
    constexpr int A_PER_WAVE = (BM / 16 + NW - 1) / NW, FA = A_PER_WAVE * NW, FB = BN / 32 * KS;
    static_assert(FB % NW == 0, "");
    constexpr int B_PER_WAVE = FB / NW, LOADS = A_PER_WAVE + B_PER_WAVE;
    constexpr int FRAG = 512;
    constexpr int STAGE = (FA + FB) * FRAG;
    constexpr int kStores = MB * NB * 2;                      // of a wave's epilogue
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // STAGES * STAGE | rows of the epilogue per wave

    // every XCD takes a contiguous range of tiles (filter tiles fastest), its workgroups take turns
    const int xcd = blockIdx.x % kXcds, n_x = (gridDim.x - xcd + kXcds - 1) / kXcds;
    const int t_begin = xcd * (total / kXcds) + (xcd < total % kXcds ? xcd : total % kXcds);
    const int t_end = t_begin + total / kXcds + (xcd < total % kXcds ? 1 : 0);
    int tile = t_begin + blockIdx.x / kXcds;
    if (tile >= t_end) return;

    const int PQ = s.P * s.Q;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;
    const int cblocks = s.C / BK;
    const int RS = s.R * s.S;
    const int nsteps = RS * cblocks;
    const int ks16_total = nsteps * KS;
    static_assert(ROWS || !SOURCES, "maps of equal shape: rows");
    __amdgpu_buffer_rsrc_t x_rsrc = make_rsrc(x, (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
    const __amdgpu_buffer_rsrc_t y_rsrc = make_rsrc(y, (uint32_t)s.N * (uint32_t)(PQ * s.K) * 2u);
    const __amdgpu_buffer_rsrc_t r_rsrc = make_rsrc(res, res ? (uint32_t)s.N * (uint32_t)(PQ * s.K) * 2u : 0u);
    auto swz = [](int r16) { return ((r16 >> 1) & 3) ^ (r16 >> 3); };

    // ---- what is fetched: tile f_tile, position (r_pos, t_pos), channel offset f_c, filter offset f_w ----
    uint32_t a_at[A_PER_WAVE], b_off[B_PER_WAVE];
    int32_t a_off[A_PER_WAVE], a_ih[A_PER_WAVE], a_iw[A_PER_WAVE];
    __amdgpu_buffer_rsrc_t w_rsrc;
    uint32_t f_c = 0, f_w = 0;
    int r_pos = 0, t_pos = 0;
    const uint32_t c_end = (uint32_t)s.C * 2;
    auto place = [&](int j, int rr, int tt) __attribute__((always_inline)) -> uint32_t {
        const bool in = (unsigned)(a_ih[j] + rr) < (unsigned)s.H && (unsigned)(a_iw[j] + tt) < (unsigned)s.W;
        return in ? (uint32_t)(a_off[j] + (rr * s.W + tt) * s.C * 2) : kOutOfRange;
    };
    auto fetch_tile = [&](int t) __attribute__((always_inline)) {
        const TileOrigin o = locate_tile<BM>(t, tiles_n, PQ, M_all, wp_all, bias_all, gt, off_w, off_b);
        w_rsrc = make_rsrc(o.wp, (uint32_t)s.K * (uint32_t)(RS * s.C) * 2u);
        const int chunk = (lane & 3) ^ swz(lane >> 2);
#pragma unroll
        for (int j = 0; j < A_PER_WAVE; ++j) {
            const int m = o.m0 + (wid * A_PER_WAVE + j) * 16 + (lane >> 2);
            const bool ok = m < o.m_end && (FA * 16 == BM || m < o.m0 + BM);
            if (ROWS) {
                a_at[j] = ok ? (uint32_t)(m * s.C * 2 + chunk * 16) : kOutOfRange;
            } else {
                const int mm = ok ? m : 0;
                const int n = mm / PQ, pq = mm - n * PQ, p = pq / s.Q, q = pq - p * s.Q;
                a_ih[j] = ok ? p * s.stride - s.pad : -0x10000;
                a_iw[j] = q * s.stride - s.pad;
                a_off[j] = ((n * s.H + p * s.stride - s.pad) * s.W + a_iw[j]) * s.C * 2 + chunk * 16;
                a_at[j] = place(j, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < B_PER_WAVE; ++j) {
            const int fb = wid * B_PER_WAVE + j;
            b_off[j] = (uint32_t)((((o.tile_n * BN / 32 + fb / KS) * ks16_total + fb % KS) * FRAG + lane * 8) * 2);
        }
        f_c = f_w = 0;
        r_pos = t_pos = 0;
        if (SOURCES) x_rsrc = make_rsrc(x, (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
    };
    auto issue_a = [&](int stage, auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (lds_void*)(lds + stage * STAGE + (wid * A_PER_WAVE + j) * FRAG), 16, a_at[j], f_c, 0, 0);
    };
    auto issue_b = [&](int stage, auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void*)(lds + stage * STAGE + (FA + wid * B_PER_WAVE + j) * FRAG), 16, b_off[j], f_w, 0, 0);
    };
    auto advance = [&]() __attribute__((always_inline)) {     // never past the tile's last step
        f_w += KS * FRAG * 2;
        if ((ROWS && !SOURCES) || f_c + BK * 2 < c_end) {
            f_c += BK * 2;
        } else if (SOURCES) {
            f_c = 0;
            x_rsrc = make_rsrc(source_at(x, from, ++r_pos), (uint32_t)s.N * (uint32_t)(s.H * s.W * s.C) * 2u);
        } else {
            const bool row_end = t_pos + 1 == s.S;
            t_pos = row_end ? 0 : t_pos + 1;
            r_pos = row_end ? r_pos + 1 : r_pos;
            f_c = 0;
#pragma unroll
            for (int j = 0; j < A_PER_WAVE; ++j) a_at[j] = place(j, r_pos, t_pos);
        }
    };

    f32x16 acc[MB][NB];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    };
    const int rd_row = lane & 31;
    const int rd0 = (rd_row >> 4) * FRAG + ((rd_row & 15) * 4 + ((lane >> 5) ^ swz(rd_row & 15))) * 8;
    bf16x8 af[KS][MB], bfr[KS][NB];
    // operand k of a half step: filters first, then pixel rows
    auto read_one = [&](auto ks_c, auto k_c, int stage) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_c)::value, k = decltype(k_c)::value;
        if constexpr (k < NB) bfr[ks][k] = *(const bf16x8*)(lds + stage * STAGE + (FA + (wn * NB + k) * KS + ks) * FRAG + lane * 8);
        else af[ks][k - NB] = *(const bf16x8*)(lds + stage * STAGE + (wm * MB * 2) * FRAG + (rd0 ^ (ks * 16)) + (k - NB) * 2 * FRAG);
    };
    typedef std::integral_constant<int, 0> c0;
    typedef std::integral_constant<int, 1> c1;
    // Half a step: the products of half MUL with the operands of the other half (of stage rd) and `loads` loads of a stage
    // slipped in between, in this very order: a wave issues in order, and with its reads and loads in one run the
    // matrix core would idle while they queue.
    auto half = [&](auto mul_c, int rd, auto n_loads_c, auto&& load) __attribute__((always_inline)) {
        constexpr int mul = decltype(mul_c)::value, n_loads = decltype(n_loads_c)::value, kMfma = MB * NB, kReads = MB + NB;
        static_assert(n_loads <= kMfma, "");
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, kMfma>([&](auto t) __attribute__((always_inline)) {
            constexpr int k = decltype(t)::value;
            constexpr int upto = (k + 1) * n_loads / kMfma, from = k * n_loads / kMfma;
            acc[k / NB][k % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[mul][k % NB], af[mul][k / NB], acc[k / NB][k % NB], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            constexpr int r0 = k * kReads / kMfma, r1 = (k + 1) * kReads / kMfma;
            if constexpr (r1 > r0) {
                read_one(std::integral_constant<int, mul ^ 1>{}, std::integral_constant<int, r0>{}, rd);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            static_assert(r1 - r0 <= 1, "at most one read after each product");
            if constexpr (upto > from) {
                load(std::integral_constant<int, from>{});
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    int cur = 0;
    // Step u multiplies stage u and fetches stage u + 3: its pixel rows in the second half, once everybody has read stage u,
    // its filters in the first half of step u + 1.  SWITCH: the fetches go on with the next tile.  LAST: all loads in the
    // second half (they are older than the epilogue's stores then), FIRST: none in the first half.  EXTRA: stores that
    // may still be outstanding.
    auto step = [&](auto first_c, auto last_c, auto switch_c, auto extra_c) __attribute__((always_inline)) {
        constexpr bool first = decltype(first_c)::value, last = decltype(last_c)::value, swt = decltype(switch_c)::value;
        constexpr int extra = decltype(extra_c)::value;
        const int nxt = cur == STAGES - 1 ? 0 : cur + 1, prv = cur == 0 ? STAGES - 1 : cur - 1;
        half(c0{}, cur, std::integral_constant<int, first ? 0 : B_PER_WAVE>{}, [&](auto k) __attribute__((always_inline)) { issue_b(prv, k); });
        if (swt) fetch_tile(tile + n_x < t_end ? tile + n_x : tile);      // (after the last tile: loads that nobody uses)
        else if (!first) advance();
        wait_before_barrier<(STAGES - 2) * LOADS + extra>();
        __builtin_amdgcn_s_barrier();
        half(c1{}, nxt, std::integral_constant<int, last ? LOADS : A_PER_WAVE>{}, [&](auto k) __attribute__((always_inline)) {
            if constexpr (decltype(k)::value < A_PER_WAVE) issue_a(cur, k);
            else issue_b(cur, std::integral_constant<int, decltype(k)::value - A_PER_WAVE>{});
        });
        if (last) advance();
        cur = nxt;
    };
    typedef std::integral_constant<bool, true> yes;
    typedef std::integral_constant<bool, false> no;
    typedef std::integral_constant<int, kStores> stores;

    fetch_tile(tile);
#pragma unroll
    for (int k = 0; k < STAGES; ++k) {
        static_for<0, A_PER_WAVE>([&](auto j) __attribute__((always_inline)) { issue_a(k, j); });
        static_for<0, B_PER_WAVE>([&](auto j) __attribute__((always_inline)) { issue_b(k, j); });
        advance();
    }
    wait_before_barrier<(STAGES - 1) * LOADS>();
    __builtin_amdgcn_s_barrier();
    static_for<0, MB + NB>([&](auto k) __attribute__((always_inline)) { read_one(c0{}, k, 0); });
    clear();
    step(yes{}, no{}, no{}, c0{});
    step(no{}, no{}, no{}, c0{});
    for (;;) {                                                // at least five steps: the launcher sees to it
        for (int u = 2; u < nsteps - 3; ++u) step(no{}, no{}, no{}, c0{});
        step(no{}, no{}, yes{}, c0{});
        step(no{}, no{}, no{}, c0{});
        step(no{}, yes{}, no{}, c0{});
        const TileOrigin o = locate_tile<BM>(tile, tiles_n, PQ, M_all, wp_all, bias_all, gt, off_w, off_b);
        uint16_t* const stage = lds + STAGES * STAGE + wid * (32 * (WN + 8) + 128);
        with_activation<ACTS>(s.act, [&](auto a) {
            constexpr int ACT = decltype(a)::value;
            const int m = o.m0 + wm * WM, n = o.tile_n * BN + wn * WN;
            if (res) store_tile_counted_act<MB, NB, ACT, true>(acc, stage, o.bias, r_rsrc, y_rsrc, m, n, o.m_end, s.K, lane);
            else store_tile_counted_act<MB, NB, ACT, false>(acc, stage, o.bias, r_rsrc, y_rsrc, m, n, o.m_end, s.K, lane);
        });
        tile += n_x;
        if (tile >= t_end) break;
        clear();
        step(yes{}, no{}, no{}, stores{});
        step(no{}, no{}, no{}, stores{});
    }
    wait_vmcnt<0>();                                          // no load may land in LDS after the workgroup has ended
#endif
}

template <bool ROWS, int MB, int NB, int WAVES_M, int WAVES_N, int ACTS = kActsPlain, bool SOURCES = false>
hipError_t launch_gemm_persistent(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                       hipStream_t stream, const Grouping& grp = Grouping(), const Sources* from = nullptr)
{
    if constexpr (ACTS == kActsPlain && !SOURCES) {
        if (s.act == 2) return launch_gemm_persistent<ROWS, MB, NB, WAVES_M, WAVES_N, kActsGelu>(x, wp, bias, res, y, s, stream, grp);
        if (s.act == 3) return launch_gemm_persistent<ROWS, MB, NB, WAVES_M, WAVES_N, kActsSilu>(x, wp, bias, res, y, s, stream, grp, from);
    }
    if constexpr (ACTS != kActsGelu && !SOURCES && ROWS)
        if (from) return launch_gemm_persistent<ROWS, MB, NB, WAVES_M, WAVES_N, ACTS, true>(x, wp, bias, res, y, s, stream, grp, from);
    constexpr int BM = 32 * MB * WAVES_M, BN = 32 * NB * WAVES_N;
    long long M = (long long)s.N * s.P * s.Q;
    int tiles_n = s.K / BN;
    long long total = count_tiles(M, (long long)s.P * s.Q, BM, tiles_n, grp.table);
    if (total > 0x7FFFFFFFll) return hipErrorInvalidValue;
    if (total == 0) return hipSuccess;
    constexpr int NW = WAVES_M * WAVES_N, kRowsLds = (BM / 16 + NW - 1) / NW * NW * 16;
    constexpr size_t kLdsBytes = (3 * (size_t)(kRowsLds + BN) * 32 + WAVES_M * WAVES_N * (32 * (32 * NB + 8) + 128)) * sizeof(uint16_t);
    static const hipError_t configured = hipFuncSetAttribute((const void*)conv_gemm_persistent_kernel<ROWS, MB, NB, WAVES_M, WAVES_N, ACTS, SOURCES>,
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
    if (configured != hipSuccess) return configured;
    const unsigned grid = (unsigned)(total < 256 ? total : 256);
    hipLaunchKernelGGL((conv_gemm_persistent_kernel<ROWS, MB, NB, WAVES_M, WAVES_N, ACTS, SOURCES>), dim3(grid), dim3(64 * WAVES_M * WAVES_N),
                       kLdsBytes, stream, (const uint16_t*)x, (const uint16_t*)wp, bias, (const uint16_t*)res, (uint16_t*)y, s, (int)M,
                       tiles_n, (int)total, grp.table, grp.off_w, grp.off_b, from ? *from : Sources{});
    return hipGetLastError();
}

}  // namespace

bool conv_mfma_uses_slab(const ConvShape& s)
{
    return s.R == 3 && s.S == 3 && s.stride == 1 && s.pad == 1 && s.W <= kSlabMaxW && s.C % 32 == 0 && s.K % 64 == 0;
}

namespace {

// Launches with few output tiles go to conv_igemm_ring_kernel (same bits).  us a launch, launches one behind the other (kernel the shape
// otherwise takes / 32 x 32 tiles / 64 x 64 tiles; in brackets how many of these):
//   512 -> 512, 3x3, 7 x 7:   1 image 53 / 7.5 / 12,   20 (496, 128) 57 / 11.8 / 12.3,  24 (592, 152) 57 / 16.6 / 12.3,  100 (2464, 616) 58 / 53 / 39
//   256 -> 256, 3x3, 14 x 14: 1 image 32 / 5.5 / 7.8,  8 (392, 100) 32 / 7.7 / 8.0,     12 (592, 148) 33 / 10.7 / 8.2,   50 (2456, 616) 33 / 33 / 22
//   128 -> 128, 3x3, 28 x 28: 1 image 20 / 4.6 / 5.8,  5 (492, 124) 20 / 6.0 / 5.9,     6 (588, 148) 20 / 7.9 / 6.0,     24 (2352, 588) 21 / 21 / 14
//   64 -> 64, 3x3, 56 x 56:   1 image 8.1 / 4.1 / 4.8, 2 (392, 98) 8.2 / 4.8 / 4.9,     3 (588, 147) 8.2 / 6.4 / 5.0,    12 (2352, 588) 8.9 / 15 / 10.2
//   3072 -> 768, 1x1, 197 positions: 1 image 32 / 7.9 / 11.8,  3 (456, 120) 33 / 12.1 / 13.4,  4 (600, 156) 33 / 20 / 13.9,  8 (1200, 300) 33 / 37 / 24
//   768 -> 768, 1x1, 197 positions:  1 image 11.4 / 4.7 / 5.7, 3 (456, 120) 11.5 / 5.2 / 5.8,  4 (600, 156) 11.6 / 7.2 / 5.8, 16 (2376, 600) 12.4 / 25 / 14.2
// 32 x 32 tiles are ahead while the chip holds all of them at once, two per compute unit; 64 x 64 tiles, which share operands between four
// wavefronts, while there are about two of them (three: 3x3) per compute unit.
constexpr long long kRingTiles32 = 512, kRingTiles64 = 512, kRingTiles64Slab = 768;

// Which tiles a long GEMM-like launch takes: height / 64 of conv_gemm_persistent_kernel's tiles, or 0 for the 128 x 128 tiles of
// conv_igemm_dma_kernel.  The unit is the time of one turn of 256 x 256 tiles on all 256 compute units; a turn of 192- and
// 128-row tiles measured 0.72-0.84 and 0.53-0.58 of it (their operand reads per product are more), 128 x 128 tiles, three
// workgroups per compute unit that share it as they come, 0.5 for up to 256 and one more per 681.  What decides is how
// well the turns fill; us at 4 / 3 / 2 / 0: 25,216 rows 3072 -> 768 137 / 115 / 122 / 134; 5910 rows 768 -> 2304 25 / 32 / 29 / 33,
// 3072 -> 768 59 / 49 / 39 / 44; 12,544 rows 2048 -> 512 42 / 36 / 31 / 33; 11,760 rows 3x3 128 -> 256 26 / 22 / 17 / 17.
// Short reductions stay on the 128 x 128 tiles: eight steps, 256 -> 1024 on 14 x 14, 64 / 59 / 52 / 52 (bound by memory).
int persistent_height(const ConvShape& s, const GroupTable& gt)
{
    if (s.K % 256 || s.R * s.S * s.C < 16 * 32) return 0;
    const long long PQ = (long long)s.P * s.Q, M = s.N * PQ;
    if (M * s.K * 2 >= 0x7FFFFFFFll) return 0;                // 31-bit offsets into the output as well
    const long long small = count_tiles(M, PQ, 128, s.K / 128, gt);
    double best = 0.5 + (small > 256 ? (double)(small - 256) / 681.0 : 0.0);
    int height = 0;
    const double turn[5] = {0.0, 0.0, 0.54, 0.80, 1.0};
    for (int h = 2; h <= 4; ++h) {
        const double cost = (double)((count_tiles(M, PQ, 64 * h, s.K / 256, gt) + 255) / 256) * turn[h];
        if (cost <= best) { best = cost; height = h; }
    }
    return height;
}
template <int MB>
hipError_t conv_persistent(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                           hipStream_t stream, const Grouping& grp, const Sources* from)
{
    if (from || (s.R == 1 && s.S == 1 && s.stride == 1 && s.pad == 0))
        return launch_gemm_persistent<true, MB, 2, 2, 4>(x, wp, bias, res, y, s, stream, grp, from);
    return launch_gemm_persistent<false, MB, 2, 2, 4>(x, wp, bias, res, y, s, stream, grp);
}
// the launches that neither the slab kernel nor few-tile kernels take
hipError_t conv_gemm(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s, hipStream_t stream,
                     const Grouping& grp = Grouping(), const Sources* from = nullptr)
{
    switch (persistent_height(s, grp.table)) {
    case 4: return conv_persistent<4>(x, wp, bias, res, y, s, stream, grp, from);
    case 3: return conv_persistent<3>(x, wp, bias, res, y, s, stream, grp, from);
    case 2: return conv_persistent<2>(x, wp, bias, res, y, s, stream, grp, from);
    }
    // 128-row tiles: three workgroups per compute unit; measured ahead of 256-row tiles on the ResNet layer shapes
    if (s.K % 128 == 0) return launch_dma<128, 128, 2, 2>(x, wp, bias, res, y, s, stream, grp, from);
    return launch_dma<128, 64, 2, 2>(x, wp, bias, res, y, s, stream, grp, from);
}

// The tiles of a launch with few of them; none: not a launch for these tiles
enum class Ring { none, slab32_9, slab32_3, deep32_9, deep32_4, shallow32, slab64_3, slab64_1, tile64 };
long long tiles32(const ConvShape& s, const GroupTable& gt)
{
    const long long PQ = (long long)s.P * s.Q;
    return count_tiles(s.N * PQ, PQ, 32, s.K / 32, gt);
}
Ring ring_tiles(const ConvShape& s, const GroupTable& gt)
{
    const bool slab = conv_mfma_uses_slab(s);
    const int cblocks = s.C / 32;
    if (!slab && cblocks % 2) return Ring::none;                 // a stage holds channel blocks of one window position
    const long long M = (long long)s.N * s.P * s.Q, PQ = (long long)s.P * s.Q;
    const long long few = tiles32(s, gt);
    if (few <= kRingTiles32) {                                   // one workgroup per compute unit, or two that share its LDS
        if (slab) return few <= 256 ? Ring::slab32_9 : Ring::slab32_3;
        return cblocks % 4 ? Ring::shallow32 : few <= 256 ? Ring::deep32_9 : Ring::deep32_4;
    }
    const long long tiles64 = count_tiles(M, PQ, 64, s.K / 64, gt);
    if (s.K % 64 == 0 && tiles64 <= (slab ? kRingTiles64Slab : kRingTiles64)) {
        // 3x3: one workgroup per compute unit has its LDS to itself, with more tiles than that two share it.  Nine steps in
        // three stages (72 KB) were too shallow for filters that come from memory: 512 -> 512 over 29 images of 15 groups
        // took 42 us, with five stages or nine single-step ones in flight 22.
        return !slab ? Ring::tile64 : tiles64 <= 256 ? Ring::slab64_3 : Ring::slab64_1;
    }
    return Ring::none;
}
// hipErrorNotSupported: not a launch for these tiles.  b: a second convolution, of the same tiles
hipError_t conv_ring(const ConvArgs& a, hipStream_t stream, const ConvArgs* b = nullptr)
{
    Ring tiles = ring_tiles(a.s, a.grp.table);
    if (b && tiles == Ring::deep32_9 && tiles32(a.s, a.grp.table) + tiles32(b->s, b->grp.table) > 256) tiles = Ring::deep32_4;
    switch (tiles) {
    case Ring::slab32_9: return launch_ring<true, 16, 9, 4>(a, stream);
    case Ring::slab32_3: return launch_ring<true, 16, 3, 6>(a, stream);
    case Ring::deep32_9: return launch_ring<false, 16, 4, 9>(a, stream, b);
    case Ring::deep32_4: return launch_ring<false, 16, 4, 4>(a, stream, b);
    case Ring::shallow32: return launch_ring<false, 16, 2, 9>(a, stream, b);
    case Ring::slab64_3: return launch_ring<true, 32, 3, 5>(a, stream);
    case Ring::slab64_1: return launch_ring<true, 32, 1, 10>(a, stream);
    case Ring::tile64: return launch_ring<false, 32, 2, 5>(a, stream, b);
    case Ring::none: break;
    }
    return hipErrorNotSupported;
}

// 31-bit byte offsets inside the kernels (buffer offsets; bit 31 marks "out of range")
bool offsets_fit(const ConvShape& s)
{
    return (long long)s.N * s.H * s.W * s.C * 2 < 0x7FFFFFFFll && (long long)s.K * s.R * s.S * s.C * 2 < 0x7FFFFFFFll &&
           (long long)s.N * s.P * s.Q < 0x7FFFFFFFll - 256;
}

template <int BK>
hipError_t pick_tile(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                     hipStream_t stream)
{
    if (s.K % 128 == 0) return launch<128, 128, BK, 2, 2>(x, wp, bias, res, y, s, stream);
    if (s.K % 64 == 0) return launch<128, 64, BK, 2, 2>(x, wp, bias, res, y, s, stream);
    return launch<128, 32, BK, 4, 1>(x, wp, bias, res, y, s, stream);
}

}  // namespace

bool conv_mfma_supported(const ConvShape& s)
{
    return s.C > 0 && s.K > 0 && s.C % 32 == 0 && s.K % 32 == 0 && s.R * s.S <= 64;
}

void pack_filters_mfma(const uint16_t* w, uint16_t* out, int K, int red)
{
    // out[((nb * red/16 + ks) * 64 + lane) * 8 + i] = w[nb*32 + lane%32][ks*16 + (lane/32)*8 + i]
    const int ks_total = red / 16;
    for (int nb = 0; nb < K / 32; ++nb)
        for (int ks = 0; ks < ks_total; ++ks)
            for (int lane = 0; lane < 64; ++lane) {
                const uint16_t* src = w + (size_t)(nb * 32 + lane % 32) * red + ks * 16 + (lane / 32) * 8;
                uint16_t* dst = out + (((size_t)nb * ks_total + ks) * 64 + lane) * 8;
                for (int i = 0; i < 8; ++i) dst[i] = src[i];
            }
}

hipError_t conv_mfma(const void* x, const void* wp, const float* bias, const void* res, void* y, const ConvShape& s,
                     hipStream_t stream)
{
    if (!conv_mfma_supported(s)) return hipErrorInvalidValue;
    long long M = (long long)s.N * s.P * s.Q;
    if (M <= 0) return hipSuccess;
    if (!offsets_fit(s)) return hipErrorInvalidValue;
    const hipError_t ring = conv_ring(ConvArgs{x, wp, bias, res, y, s, Grouping()}, stream);
    if (ring != hipErrorNotSupported) return ring;
    // 32-channel steps everywhere: measured equal or better than 64-channel steps on every ResNet layer shape
    if (conv_mfma_uses_slab(s)) {
        // 256-row and 128-row tiles measured within a few percent of each other on every ResNet-18 layer shape
        if (s.K % 128 == 0) return launch_slab<256, 128, 2, 2>(x, wp, bias, res, y, s, stream);
        return launch_slab<256, 64, 4, 1>(x, wp, bias, res, y, s, stream);
    }
    if (s.K % 64 == 0) return conv_gemm(x, wp, bias, res, y, s, stream);
    // filter counts that are not a multiple of 64: the register-staged kernel
    return pick_tile<32>(x, wp, bias, res, y, s, stream);
}

bool conv_mfma_sources_supported(const ConvShape& one, int32_t n_sources)
{
    // (K = 64 m: every kernel that such a launch may take knows sources; GELU's instantiations do not)
    return n_sources >= 2 && n_sources <= kMaxSources && one.R == 1 && one.S == 1 && one.stride == 1 && one.pad == 0 && one.act != 2 &&
           one.C > 0 && one.C % 32 == 0 && one.K > 0 && one.K % 64 == 0;
}

hipError_t conv_mfma_sources(const void* const* x, int32_t n_sources, const void* wp, const float* bias, const void* res, void* y,
                             const ConvShape& one, hipStream_t stream)
{
    if (!conv_mfma_sources_supported(one, n_sources)) return hipErrorInvalidValue;
    ConvShape s = one;
    s.R = n_sources;
    if ((long long)s.N * s.P * s.Q <= 0) return hipSuccess;
    if (!offsets_fit(s)) return hipErrorInvalidValue;
    Sources from{};
    for (int k = 1; k < n_sources; ++k) from.rest[k - 1] = (const uint16_t*)x[k];
    const hipError_t ring = conv_ring(ConvArgs{x[0], wp, bias, res, y, s, Grouping(), &from}, stream);
    if (ring != hipErrorNotSupported) return ring;
    return conv_gemm(x[0], wp, bias, res, y, s, stream, Grouping(), &from);
}

bool conv_mfma_groupable(const ConvShape& s)
{
    return conv_mfma_supported(s) && s.K % 64 == 0;
}

static bool valid_groups(const GroupTable& groups, size_t off_w, size_t off_b, const ConvShape& s)
{
    if (!conv_mfma_groupable(s) || groups.n <= 0 || groups.n > kMaxGroups || groups.first_row[0] != 0 ||
        groups.first_row[groups.n] != s.N || off_w > 0x7FFFFFFFull || off_b > 0x7FFFFFFFull)
        return false;
    for (int g = 0; g < groups.n; ++g)
        if (groups.first_row[g + 1] < groups.first_row[g] || !groups.weights[g]) return false;
    return true;
}

hipError_t conv_mfma_grouped(const void* x, const GroupTable& groups, size_t off_w, size_t off_b, const void* res, void* y,
                             const ConvShape& s, hipStream_t stream)
{
    if (!valid_groups(groups, off_w, off_b, s)) return hipErrorInvalidValue;
    long long M = (long long)s.N * s.P * s.Q;
    if (M <= 0) return hipSuccess;
    if (!offsets_fit(s)) return hipErrorInvalidValue;
    const Grouping grp{groups, (uint32_t)off_w, (uint32_t)off_b};
    const hipError_t ring = conv_ring(ConvArgs{x, nullptr, nullptr, res, y, s, grp}, stream);
    if (ring != hipErrorNotSupported) return ring;
    // every group starts a fresh row of tiles: 128-row tiles waste fewer rows past the end of a small group, 256-row
    // tiles (twice the accumulator rows per wave and operand read) are the faster ones where that waste stays small
    if (conv_mfma_uses_slab(s)) {
        const long long PQ = (long long)s.P * s.Q;
        const bool tall = 256 * count_tiles(M, PQ, 256, 1, groups) * 100 <= 128 * count_tiles(M, PQ, 128, 1, groups) * 104;
        if (s.K % 128 == 0)
            return tall ? launch_slab<256, 128, 2, 2>(x, nullptr, nullptr, res, y, s, stream, grp)
                        : launch_slab<128, 128, 2, 2>(x, nullptr, nullptr, res, y, s, stream, grp);
        return tall ? launch_slab<256, 64, 4, 1>(x, nullptr, nullptr, res, y, s, stream, grp)
                    : launch_slab<128, 64, 4, 1>(x, nullptr, nullptr, res, y, s, stream, grp);
    }
    return conv_gemm(x, nullptr, nullptr, res, y, s, stream, grp);
}

// Two launches of few tiles each leave most of the chip idle, and the second waits for the first for nothing: one launch has the
// tiles of both.  The tiles are those that each would take by itself, so the bits are the same; how deep their pipeline is goes by
// the tiles of both, so that all are resident where they can be.  us, two launches / one, 1x1 512 -> 512 twice on 7 x 7: 1 image 10.4 / 5.4,
// 8 images (208 tiles each) 10.6 / 6.0, 16 11.4 / 9.5, 24 13.5 / 8.8, 64 18.3 / 15.3; with the depth of one convolution's tiles 8 images took 8.9.
// Launches that fill the chip gain nothing by sharing it, and pairs whose tiles differ would need a kernel per combination: these
// stay apart.
bool conv_mfma_pairable(const ConvShape& a, const ConvShape& b, const GroupTable* groups)
{
    const GroupTable none{};
    for (const ConvShape* s : {&a, &b})
        if (!conv_mfma_supported(*s) || (long long)s->N * s->P * s->Q <= 0 || !offsets_fit(*s) || s->act == 2 || conv_mfma_uses_slab(*s))
            return false;
    const Ring tiles = ring_tiles(a, groups ? *groups : none);
    return tiles != Ring::none && tiles == ring_tiles(b, groups ? *groups : none);
}

hipError_t conv_mfma_pair(const ConvCall& a, const ConvCall& b, const GroupTable* groups, hipStream_t stream)
{
    if (!conv_mfma_pairable(a.s, b.s, groups)) return hipErrorInvalidValue;
    if (groups && (!valid_groups(*groups, a.off_w, a.off_b, a.s) || !valid_groups(*groups, b.off_w, b.off_b, b.s))) return hipErrorInvalidValue;
    const GroupTable& gt = groups ? *groups : GroupTable{};
    const ConvArgs a1{a.x, a.wp, a.bias, a.res, a.y, a.s, Grouping{gt, (uint32_t)a.off_w, (uint32_t)a.off_b}};
    const ConvArgs b1{b.x, b.wp, b.bias, b.res, b.y, b.s, Grouping{gt, (uint32_t)b.off_w, (uint32_t)b.off_b}};
    return conv_ring(a1, stream, &b1);
}

}  // namespace k
}  // namespace coe
