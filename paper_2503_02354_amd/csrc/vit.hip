// gfx950 kernels for transformer-shaped experts (bf16): patch gathering, class token + positions, layer norm,
// multi-head attention on the matrix cores.  Token tensors are [N][T][D], D contiguous.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace coe {
namespace k {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));   // round to nearest even
}
// a product that is rounded before it is used (not contracted into a multiply-add)
__device__ __forceinline__ float scaled(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float wave_sum_lds(float v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}
template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// the same sum without LDS: v + the value of lane ^ 32, then ^ 16, 8, 4, 2 and 1
__device__ __forceinline__ float wave_sum(float v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kRor8 = 0x128, kMirror8 = 0x141, kXor3 = 0x1B, kXor2 = 0x4E, kXor1 = 0xB1;    // row rotate, half-row mirror, quad permutations
    auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(halves[0]) + __uint_as_float(halves[1]);
    auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(rows[0]) + __uint_as_float(rows[1]);
    v += dpp<kRor8>(v);
    v += dpp<kXor3>(dpp<kMirror8>(v));                        // 7 - i, then ^ 3: ^ 4
    v += dpp<kXor2>(v);
    v += dpp<kXor1>(v);
#endif
    return v;
}

// ---- patches of a non-overlapping convolution laid out as GEMM rows -------------------------------------------
// x [N][H][W][C] -> out [N][H/R][W/S][R][S*C]: one 16-byte chunk per thread; S*C*2 bytes is a multiple of 16.
__global__ __launch_bounds__(256) void patchify_kernel(const uint4* __restrict__ x, uint4* __restrict__ out, int N, int H, int W,
                                                       int R, int gh, int gw, int run_chunks)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)N * gh * gw * R * run_chunks;
    if (idx >= total) return;
    int ch = (int)(idx % run_chunks);
    size_t t = idx / run_chunks;
    int r = (int)(t % R); t /= R;
    int pw = (int)(t % gw); t /= gw;
    int ph = (int)(t % gh);
    int n = (int)(t / gh);
    // a source row holds W*C elements = gw * run_chunks chunks
    size_t src = (((size_t)n * H + (size_t)ph * R + r) * gw + pw) * run_chunks + ch;
    out[idx] = x[src];
}

// first tensor of the group that image n belongs to, `off` bytes into its expert's weights
__device__ __forceinline__ const void* group_tensor(const GroupTable& gt, int n, uint32_t off)
{
    int g = 0;
    while (g + 1 < gt.n && n >= gt.first_row[g + 1]) ++g;
    return (const char*)gt.weights[g] + off;
}

// ---- class token + position embedding: out[n][0] = cls + pos[0]; out[n][1+i] = x[n][i] + pos[1+i] -----------------
template <bool GROUPED>
__global__ __launch_bounds__(256) void tokens_kernel(const uint4* __restrict__ x, const uint4* __restrict__ cls,
                                                     const uint4* __restrict__ pos, uint4* __restrict__ out, int N, int T, int D8,
                                                     GroupTable gt, uint32_t off_cls, uint32_t off_pos)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)N * T * D8;
    if (idx >= total) return;
    int c = (int)(idx % D8);
    size_t r = idx / D8;
    int t = (int)(r % T);
    int n = (int)(r / T);
    if (GROUPED) {
        cls = (const uint4*)group_tensor(gt, n, off_cls);
        pos = (const uint4*)group_tensor(gt, n, off_pos);
    }
    uint4 a = t == 0 ? cls[c] : x[((size_t)n * (T - 1) + (t - 1)) * D8 + c];
    uint4 p = pos[(size_t)t * D8 + c];
    uint4 o;
    o.x = pack_bf16(bf16_lo(a.x) + bf16_lo(p.x), bf16_hi(a.x) + bf16_hi(p.x));
    o.y = pack_bf16(bf16_lo(a.y) + bf16_lo(p.y), bf16_hi(a.y) + bf16_hi(p.y));
    o.z = pack_bf16(bf16_lo(a.z) + bf16_lo(p.z), bf16_hi(a.z) + bf16_hi(p.z));
    o.w = pack_bf16(bf16_lo(a.w) + bf16_lo(p.w), bf16_hi(a.w) + bf16_hi(p.w));
    out[idx] = o;
}

// ---- layer norm over channels, one wavefront per token, the token held in registers ---------------------------------
// A launch of a few requests is a chain of latencies: the token, two sums over the wavefront, scale and shift.  Scale and shift are
// on their way from the start, up to 1024 channels (beyond, their registers would cost long launches half the wavefronts), and
// the sums exchange lanes by register operations instead of through LDS, in the same order.  us per launch, 985 tokens of 768 channels:
// 5.5 / 4.3 (6.3 / 4.6 with a group table); five requests, 48 launches, 1975 / 1877.  Beyond 1280 channels and the tokens that the chip
// holds at once, the sums go through LDS again: us in LDS / in registers, 1536 channels 4000 tokens 7.7 / 7.5, 16,000 23.4 / 25.2, 32,000
// 40.0 / 42.3; 2048 channels 4000 tokens 9.8 / 9.5, 8000 18.6 / 19.6, 32,000 53.8 / 56.9; but 1280 channels 16,000 tokens 20.1 / 20.8, 50,432 50.4 / 48.9.
constexpr int kLnMaxPairs = 16;     // D <= 64 lanes * 2 * 16 = 2048
constexpr int kLnAtOnce = 256 * 28; // tokens of more than 1024 channels: seven wavefronts per SIMD
template <bool GROUPED, int PAIRS>
__global__ __launch_bounds__(256) void layernorm_kernel(const uint32_t* __restrict__ x, const float* __restrict__ gamma,
                                                        const float* __restrict__ beta, uint32_t* __restrict__ y, int rows,
                                                        int D2 /* pairs per token */, GroupTable gt, int tokens_per_image,
                                                        uint32_t off_gamma, uint32_t off_beta)
{
    int row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (row >= rows) return;
    if (GROUPED) {
        gamma = (const float*)group_tensor(gt, row / tokens_per_image, off_gamma);
        beta = (const float*)group_tensor(gt, row / tokens_per_image, off_beta);
    }
    int lane = threadIdx.x & 63;
    const uint32_t* xp = x + (size_t)row * D2;
    float v[2 * PAIRS];
    uint32_t w[PAIRS];
    constexpr bool kAhead = PAIRS <= 8;
    float2 g[PAIRS], b[PAIRS];
    auto scale_shift = [&](int j) {
        const int c = lane + 64 * j;
        g[j] = c < D2 ? *(const float2*)(gamma + 2 * c) : make_float2(0.f, 0.f);
        b[j] = c < D2 ? *(const float2*)(beta + 2 * c) : make_float2(0.f, 0.f);
    };
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        const int c = lane + 64 * j;
        w[j] = c < D2 ? xp[c] : 0u;
    }
#pragma unroll
    for (int j = 0; j < PAIRS; ++j)
        if (kAhead) scale_shift(j);
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        v[2 * j] = bf16_lo(w[j]);
        v[2 * j + 1] = bf16_hi(w[j]);
        sum += v[2 * j] + v[2 * j + 1];
    }
    const float inv_d = 1.f / (float)(2 * D2);
    const bool by_lds = !kAhead && D2 > 640 && rows > kLnAtOnce;
    const float mean = (by_lds ? wave_sum_lds(sum) : wave_sum(sum)) * inv_d;
    float sq = 0.f;
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        if (lane + 64 * j < D2) {
            float p = v[2 * j] - mean, q = v[2 * j + 1] - mean;
            sq += p * p + q * q;
        }
    }
    const float rstd = rsqrtf((by_lds ? wave_sum_lds(sq) : wave_sum(sq)) * inv_d + 1e-6f);
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        const int c = lane + 64 * j;
        if (!kAhead) scale_shift(j);
        if (c < D2)
            y[(size_t)row * D2 + c] = pack_bf16((v[2 * j] - mean) * rstd * g[j].x + b[j].x, (v[2 * j + 1] - mean) * rstd * g[j].y + b[j].y);
    }
}

// ---- attention, head width 64, up to 224 tokens ---------------------------------------------------------------------
// Scores are computed transposed, S^T = K Q^T, with the key fragment as the first matrix-core operand: a lane then
// owns ONE query (column l%32) and, per 32-key block, the keys 8*(v/4) + 4*(l/32) + v%4.  Softmax statistics of a
// query therefore live in two lanes (l and l^32), and the exponentials, rounded to bf16, are already laid out as the
// second operand of the next product O^T = V^T P^T (keys may be visited in any order as long as V^T uses the same
// one), so the probabilities never leave registers.  A lane ends with 4 consecutive head channels of its query per
// accumulator quad and stores 8 bytes at a time.
// Numerics: scores in fp32, e = exp(s - max), probabilities p = e / sum(e) rounded to bf16 (they are a tensor of their
// own in storage precision), output = sum_j p_j v_j accumulated in fp32 and rounded to bf16.
// What bounds it: q, k, v and the output through HBM, 0.47 GB for 389 requests of 197 tokens and 12 heads (96 us at the
// 4.9 TB/s a large copy reaches); the softmax is about 80 us of vector instructions.  A head of a request is a load of
// 75 KB and a few microseconds of work, so what counts is that loads are always in flight: workgroups of eight wavefronts
// stay, one per compute unit; K and V of the next unit of work come by DMA into a second buffer, its queries into
// registers, while every wavefront does one block of 32 queries of this one.  V stays as it is in memory: the transposing
// LDS read (four rows of sixteen 16-bit elements per 16 lanes, a lane gets one column) delivers V^T.  With fewer than five
// 32-token blocks a unit of work is several heads.
// Measured there: 380 us (two workgroups of four wavefronts per compute unit, each loading and transposing its K and V
// through registers, then two rounds of query blocks) -> 140 us; 12 heads of one request 17 -> 9 us.
constexpr int kDh = 64;
constexpr int kMaxKeyBlocks = 7;
constexpr int kAttnWaves = 8;
typedef __attribute__((address_space(3))) void lds_void;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
[[maybe_unused]] constexpr uint32_t kOutOfRange = 0x80000000u;   // buffer offset beyond any tensor: loads return zeros, stores are dropped

template <int TB>
__global__ __launch_bounds__(64 * kAttnWaves, 2) void attention_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ out,
                                                                       int N, int T, int D, int heads, float scale)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int kHeads = kAttnWaves / TB;           // heads per unit of work
    constexpr int kRows8 = 4 * TB;                    // 1 KiB blocks of eight 128-byte rows in K, the same in V
    constexpr int kBuf = kHeads * 2 * kRows8 * 1024;  // bytes; a wavefront loads kHeads * TB blocks of it
    extern __shared__ __attribute__((aligned(1024))) char lds[];      // two buffers
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int items = N * heads, units = (items + kHeads - 1) / kHeads;
    const uint32_t row_bytes = (uint32_t)D * 6u;      // a token of qkv
    const __amdgpu_buffer_rsrc_t in_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(qkv), 0, (int)((uint32_t)N * (uint32_t)T * row_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t out_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)((uint32_t)N * (uint32_t)T * (uint32_t)D * 2u), 0x00020000);

    // Row r of K keeps its 16-byte chunk c in slot c ^ ((r >> 1) & 7), row r of V in slot c ^ (r & 7): operand reads (32 rows
    // of one chunk; four rows of sixteen channels) then spread over the LDS banks.  Lane i of a load fills slot i % 8 of row
    // i / 8 and fetches the chunk that belongs there.
    const int ld_row = lane >> 3, ld_slot = lane & 7;
    auto load_unit = [&](int unit, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kHeads * TB; ++j) {
            const int blk = wid + kAttnWaves * j, in_item = blk % (2 * kRows8), b = in_item % kRows8;
            const int item = unit * kHeads + blk / (2 * kRows8), is_v = in_item / kRows8;
            const int n = item / heads, head = item - n * heads;
            const int chunk = ld_slot ^ (is_v ? ld_row : ((b & 1) * 4 + (ld_row >> 1)));
            const bool ok = item < items && 8 * b + ld_row < T;
            const uint32_t at = ok ? (uint32_t)ld_row * row_bytes + (uint32_t)chunk * 16u : kOutOfRange;
            const uint32_t base = ((uint32_t)n * (uint32_t)T + 8u * b) * row_bytes + (uint32_t)((1 + is_v) * D + head * kDh) * 2u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (lds_void*)(lds + buf * kBuf + blk * 1024), 16, at,
                                                     __builtin_amdgcn_readfirstlane(base), 0, 0);
        }
    };
    const int sub = wid / TB, qb = wid % TB;          // this wavefront's head of the unit and block of queries
    const bool works = wid < kHeads * TB;
    const int query = qb * 32 + l32;
    u32x4 q_next[kDh / 16];
    auto load_queries = [&](int unit) __attribute__((always_inline)) {
        const int item = unit * kHeads + sub, n = item / heads, head = item - n * heads;
        const uint32_t at = item < items && query < T ? (uint32_t)l32 * row_bytes + (uint32_t)half * 16u : kOutOfRange;
        const uint32_t base = __builtin_amdgcn_readfirstlane(((uint32_t)n * (uint32_t)T + 32u * qb) * row_bytes + (uint32_t)(head * kDh) * 2u);
#pragma unroll
        for (int ks = 0; ks < kDh / 16; ++ks) q_next[ks] = __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, at, base + ks * 32, 0);
    };

    // operand addresses inside a buffer (bytes): K, for the low bit of the 16-channel step; V, for the two 32-channel halves
    const char* const item_lds = lds + (works ? sub : 0) * (2 * kRows8 * 1024);
    uint32_t k_at[kDh / 16], v_at[2];
#pragma unroll
    for (int ks = 0; ks < kDh / 16; ++ks) k_at[ks] = (uint32_t)(l32 * 128 + (((ks * 2 + half) ^ ((l32 >> 1) & 7)) * 16));
#pragma unroll
    for (int db = 0; db < 2; ++db) {
        const int r = 4 * half + ((lane >> 2) & 3), chunk = db * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
        v_at[db] = (uint32_t)(kRows8 * 1024 + r * 128 + ((chunk ^ r) * 16) + (lane & 1) * 8);
    }
    const float scale2 = scale * 1.44269504088896340736f;

    int buf = 0;
    bool stored = false;
    load_unit(blockIdx.x, 0);
    if (works) load_queries(blockIdx.x);
    for (int unit = blockIdx.x; unit < units; unit += gridDim.x) {
        // this unit's loads have landed; the eight stores of the unit before, if any, are younger and may be on their way
        if (works && stored) __builtin_amdgcn_s_waitcnt(8 | (7 << 4) | (0 << 8));
        else __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (0 << 8));
        __builtin_amdgcn_s_barrier();
        bf16x8 qf[kDh / 16];
#pragma unroll
        for (int ks = 0; ks < kDh / 16; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, q_next[ks]);
        if (unit + (int)gridDim.x < units) {
            load_unit(unit + gridDim.x, buf ^ 1);
            if (works) load_queries(unit + gridDim.x);
        }
        if (works) {
            const char* const kv = item_lds + buf * kBuf;
            f32x16 sc[TB];
            float m = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < TB; ++kb) {
#pragma unroll
                for (int v = 0; v < 16; ++v) sc[kb][v] = 0.f;
#pragma unroll
                for (int ks = 0; ks < kDh / 16; ++ks) {
                    const bf16x8 kf = *(const bf16x8*)(kv + k_at[ks] + kb * 4096);
                    sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sc[kb], 0, 0, 0);
                }
                if (kb == TB - 1) {                   // the last block may hold rows past the last token
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        if (kb * 32 + 8 * (v >> 2) + 4 * half + (v & 3) >= T) sc[kb][v] = -INFINITY;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sc[kb][v] = scaled(sc[kb][v], scale2);    // scores in units of ln 2
                    m = fmaxf(m, sc[kb][v]);
                }
            }
            m = fmaxf(m, __shfl_xor(m, 32, 64));
            float lsum = 0.f;
#pragma unroll
            for (int kb = 0; kb < TB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    // 2^x on the transcendental unit (one instruction; exp(s - max) = 2^((s - max) / ln 2))
                    sc[kb][v] = __builtin_amdgcn_exp2f(sc[kb][v] - m);
                    sc[kb][v + 1] = __builtin_amdgcn_exp2f(sc[kb][v + 1] - m);
                    lsum += sc[kb][v] + sc[kb][v + 1];
                }
            lsum += __shfl_xor(lsum, 32, 64);
            const float inv = 1.f / lsum;
            f32x16 oacc[2];
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
#pragma unroll
            for (int kb = 0; kb < TB; ++kb)
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2) {      // 16 keys per matrix-core step: accumulator quads 2 t2 and 2 t2 + 1
                    const int v0 = 8 * t2;
                    u32x4 pv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) pv[e] = pack_bf16(sc[kb][v0 + 2 * e] * inv, sc[kb][v0 + 2 * e + 1] * inv);
                    const bf16x8 pf = __builtin_bit_cast(bf16x8, pv);
#pragma unroll
                    for (int db = 0; db < 2; ++db) {
                        const char* vp = kv + v_at[db] + kb * 4096 + t2 * 2048;
                        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp));
                        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp + 1024));
                        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, oacc[db], 0, 0, 0);
                    }
                }
            const int item = unit * kHeads + sub, n = item / heads, head = item - n * heads;
            const uint32_t at = item < items && query < T ? (uint32_t)l32 * (uint32_t)(D * 2) + (uint32_t)half * 8u : kOutOfRange;
            const uint32_t base =
                __builtin_amdgcn_readfirstlane(((uint32_t)n * (uint32_t)T + 32u * qb) * (uint32_t)(D * 2) + (uint32_t)(head * kDh) * 2u);
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    u32x2 o;
                    o[0] = pack_bf16(oacc[db][4 * gq], oacc[db][4 * gq + 1]);
                    o[1] = pack_bf16(oacc[db][4 * gq + 2], oacc[db][4 * gq + 3]);
                    __builtin_amdgcn_raw_buffer_store_b64(o, out_rsrc, at, base + db * 64 + gq * 16, 0);
                }
        }
        stored = true;
        buf ^= 1;
    }
#endif
}

template <int TB>
hipError_t launch_attention(const void* qkv, void* out, int32_t N, int32_t T, int32_t D, int32_t heads, hipStream_t stream)
{
    constexpr int kHeads = kAttnWaves / TB;
    constexpr size_t kLds = 2 * (size_t)kHeads * 8 * TB * 1024;
    static const hipError_t configured =
        hipFuncSetAttribute((const void*)attention_kernel<TB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (configured != hipSuccess) return configured;
    const long long units = ((long long)N * heads + kHeads - 1) / kHeads;
    hipLaunchKernelGGL(attention_kernel<TB>, dim3((unsigned)(units < 256 ? units : 256)), dim3(64 * kAttnWaves), kLds, stream,
                       (const uint16_t*)qkv, (uint16_t*)out, N, T, D, heads, 1.0f / sqrtf((float)kDh));
    return hipGetLastError();
}

}  // namespace

hipError_t patchify(const void* x, void* out, int32_t N, int32_t H, int32_t W, int32_t C, int32_t R, int32_t S, hipStream_t stream)
{
    if (R <= 0 || S <= 0 || H % R || W % S || (S * C * 2) % 16) return hipErrorInvalidValue;
    int gh = H / R, gw = W / S, run_chunks = S * C * 2 / 16;
    size_t total = (size_t)N * gh * gw * R * run_chunks;
    if (total == 0) return hipSuccess;
    size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(patchify_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4*)x, (uint4*)out, N, H, W, R, gh,
                       gw, run_chunks);
    return hipGetLastError();
}

namespace {

template <bool GROUPED>
hipError_t launch_tokens(const void* x, const void* cls, const void* pos, void* out, int32_t N, int32_t T, int32_t D,
                         const GroupTable& gt, uint32_t off_cls, uint32_t off_pos, hipStream_t stream)
{
    if (D % 8) return hipErrorInvalidValue;
    size_t total = (size_t)N * T * (D / 8);
    if (total == 0) return hipSuccess;
    size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(tokens_kernel<GROUPED>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4*)x, (const uint4*)cls,
                       (const uint4*)pos, (uint4*)out, N, T, D / 8, gt, off_cls, off_pos);
    return hipGetLastError();
}

template <bool GROUPED>
hipError_t launch_layernorm(const void* x, const float* gamma, const float* beta, void* y, int64_t rows, int32_t D, const GroupTable& gt,
                            int32_t tokens_per_image, uint32_t off_gamma, uint32_t off_beta, hipStream_t stream)
{
    if (D % 2 || D > 128 * kLnMaxPairs) return hipErrorInvalidValue;
    if (rows == 0) return hipSuccess;
    int64_t blocks = (rows + 3) / 4;
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint32_t*)x, gamma, beta, (uint32_t*)y, (int)rows, D / 2,
                           gt, tokens_per_image, off_gamma, off_beta);
    };
    if (D <= 128 * 4) launch(layernorm_kernel<GROUPED, 4>);
    else if (D <= 128 * 6) launch(layernorm_kernel<GROUPED, 6>);
    else if (D <= 128 * 8) launch(layernorm_kernel<GROUPED, 8>);
    else launch(layernorm_kernel<GROUPED, kLnMaxPairs>);
    return hipGetLastError();
}

bool table_ok(const GroupTable& groups, int32_t N, size_t off_a, size_t off_b)
{
    return groups.n > 0 && groups.n <= kMaxGroups && groups.first_row[0] == 0 && groups.first_row[groups.n] == N &&
           off_a <= 0x7FFFFFFFull && off_b <= 0x7FFFFFFFull;
}

}  // namespace

hipError_t tokens(const void* x, const void* cls, const void* pos, void* out, int32_t N, int32_t T, int32_t D, hipStream_t stream)
{
    return launch_tokens<false>(x, cls, pos, out, N, T, D, GroupTable{}, 0, 0, stream);
}

hipError_t tokens_grouped(const void* x, const GroupTable& groups, size_t off_cls, size_t off_pos, void* out, int32_t N, int32_t T,
                          int32_t D, hipStream_t stream)
{
    if (!table_ok(groups, N, off_cls, off_pos)) return hipErrorInvalidValue;
    return launch_tokens<true>(x, nullptr, nullptr, out, N, T, D, groups, (uint32_t)off_cls, (uint32_t)off_pos, stream);
}

hipError_t layernorm(const void* x, const float* gamma, const float* beta, void* y, int64_t rows, int32_t D, hipStream_t stream)
{
    return launch_layernorm<false>(x, gamma, beta, y, rows, D, GroupTable{}, 1, 0, 0, stream);
}

hipError_t layernorm_grouped(const void* x, const GroupTable& groups, size_t off_gamma, size_t off_beta, void* y, int32_t N, int32_t T,
                             int32_t D, hipStream_t stream)
{
    if (!table_ok(groups, N, off_gamma, off_beta) || T <= 0) return hipErrorInvalidValue;
    return launch_layernorm<true>(x, nullptr, nullptr, y, (int64_t)N * T, D, groups, T, (uint32_t)off_gamma, (uint32_t)off_beta, stream);
}

bool attention_supported(int32_t T, int32_t D, int32_t heads)
{
    return heads > 0 && D == heads * kDh && T > 0 && T <= kMaxKeyBlocks * 32;
}

hipError_t attention(const void* qkv, void* out, int32_t N, int32_t T, int32_t D, int32_t heads, hipStream_t stream)
{
    if (!attention_supported(T, D, heads)) return hipErrorInvalidValue;
    if (N == 0) return hipSuccess;
    if ((long long)N * T * D * 6 >= 0x7FFFFFFFll) return hipErrorInvalidValue;      // 31-bit byte offsets inside the kernel
    switch ((T + 31) / 32) {
    case 1: return launch_attention<1>(qkv, out, N, T, D, heads, stream);
    case 2: return launch_attention<2>(qkv, out, N, T, D, heads, stream);
    case 3: return launch_attention<3>(qkv, out, N, T, D, heads, stream);
    case 4: return launch_attention<4>(qkv, out, N, T, D, heads, stream);
    case 5: return launch_attention<5>(qkv, out, N, T, D, heads, stream);
    case 6: return launch_attention<6>(qkv, out, N, T, D, heads, stream);
    default: return launch_attention<7>(qkv, out, N, T, D, heads, stream);
    }
}

}  // namespace k
}  // namespace coe
