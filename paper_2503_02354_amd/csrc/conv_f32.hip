// fp32 convolution on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32: full fp32 products and accumulation).
//
// A workgroup of eight wavefronts owns a 16 x 16 tile of output pixels and up to 64 filters; a wavefront holds 32 pixels
// (two tile rows).  Per block of CB input channels the input patch of the tile and the filters are staged in LDS; the
// reduction runs over 8-element chunks, four per half wavefront, so that one 16-byte operand read feeds four matrix-core
// instructions (which reduction element an instruction pairs with which is free as long as both operands agree).
//   C % 8 == 0: a chunk is 8 channels of one window position; a patch pixel takes CB + 4 floats in LDS, which puts the
//     16-byte reads of 16 neighbouring pixels on different banks.
//   other C (images): patch rows are contiguous, a chunk is 8 of the S*C elements of a window row, zeros on both sides where
//     it overhangs (what lies there in the patch are the next pixels, and zero times an infinite one is not zero).
// Zero padding is multiplied like any pixel, so the filters have to be finite (conv_direct's caller says whether they are).
// Bound: the fp32 matrix cores (157 TFLOP/s; a large library product reaches 153).  An instruction takes 64 cycles and the
// operands of four take one LDS read each, so neither LDS nor L2 is near its limit; two workgroups per compute unit (LDS
// up to 78 KB each) keep the matrix cores busy while the other one stages.
// Measured on 256 requests through two experts of 3->16->32->64 channels, 3x3, 64x64 images (98 GFLOP), the whole pass: 86.6 ms
// with one thread per output and scalar loads, 1.37 here.
// Error against 64 bits, 2-norm, plain kernel / here: 3 -> 16 9.54e-8 / 9.56e-8, 32 -> 64 3.02e-7 / 3.02e-7, 256 -> 512 8.32e-7 / 8.30e-7.
// Small maps: a wavefront whose two tile rows lie below the map has no products to add, and a launch of at most 256 tiles of 64 filters
// takes tiles of 32.  us, plain kernel / without these two / with them: 2x2 map, 512 -> 512, 3x3, 64 images 559 / 657 / 305,
// 512 images 7467 / 4833 / 2218; 2x2, 64 -> 64, 3x3, 64 images 40 / 48 / 21; 28x28, 3 -> 64, 3x3, one image 7.8 / 11.4 / 9.1.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace coe {
namespace k {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kTile = 16;                  // output pixels per tile side
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr size_t kLdsTwo = 78 * 1024;      // two workgroups per compute unit
constexpr size_t kLdsOne = 158 * 1024;

template <int ACT> __device__ __forceinline__ float act_fn(float v)
{
    if (ACT == 1) return v > 0.f ? v : 0.f;
    if (ACT == 2) return 0.5f * v * erfcf(-v * 0.70710678118654752440f);
    if (ACT == 3) return v / (1.f + expf(-v));
    return v;
}

struct Geom {
    int tiles_p, tiles_q, pixel_tiles, ktiles;
    int patch_rows, patch_cols;   // pixels
    int CB, cblocks;              // channels per block
    int px;                       // floats per patch pixel in LDS
    int row;                      // floats per patch row in LDS
    int sub, chunks;              // a window row is `sub` runs (px floats apart) of `chunks` 8-element chunks
};

template <int NB, bool CHAN8>
__global__ __launch_bounds__(kThreads, 4) void conv_f32_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                               const float* __restrict__ bias, const float* __restrict__ res,
                                                               float* __restrict__ y, ConvShape s, Geom g)
{
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float* const wl = smem;                                            // [R * sub * chunks][NB][64 lanes][4]
    float* const patch = smem + s.R * g.sub * g.chunks * NB * 256;     // [patch_rows][row]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int prow = 2 * wid + (l32 >> 4), pcol = l32 & 15;            // this lane's pixel of the tile
    const float* const a_src = patch + prow * s.stride * g.row + pcol * s.stride * g.px + 4 * half;
    const float* const b_src = wl + lane * 4;

    int staged = -1;
    const int total = g.pixel_tiles * g.ktiles;
    for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
        const int kt = tile / g.pixel_tiles, pt = tile % g.pixel_tiles;
        const int n = pt / (g.tiles_p * g.tiles_q), tp = (pt / g.tiles_q) % g.tiles_p, tq = pt % g.tiles_q;
        const int ih0 = tp * kTile * s.stride - s.pad, iw0 = tq * kTile * s.stride - s.pad;
        const float* const img = x + (size_t)n * s.H * s.W * s.C;
        const bool works = tp * kTile + 2 * wid < s.P;                 // this wavefront's rows exist (on small maps most do not)

        f32x16 acc[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

        for (int cb = 0; cb < g.cblocks; ++cb) {
            if (staged != kt || g.cblocks > 1) {
                const int pieces = s.R * g.sub * g.chunks * NB * 64;
                for (int i = tid; i < pieces; i += kThreads) {
                    const int l = i & 63, j = (i >> 6) % NB, c = (i >> 6) / NB;
                    const int f = (kt * NB + j) * 32 + (l & 31), e = (c % g.chunks) * 8 + (l >> 5) * 4;
                    f32x4 v = {0.f, 0.f, 0.f, 0.f};
                    if (f < s.K) {
                        if (CHAN8) {
                            v = *(const f32x4*)(w + ((size_t)f * s.R * s.S + c / g.chunks) * s.C + cb * g.CB + e);
                        } else {
                            const int sc = s.S * s.C, r = c / g.chunks;
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                if (e + t < sc) v[t] = w[((size_t)f * s.R + r) * sc + e + t];
                        }
                    }
                    *(f32x4*)(wl + (size_t)i * 4) = v;
                }
                staged = kt;
            }
            if (CHAN8) {
                const int per_px = g.CB / 4, pieces = g.patch_rows * g.patch_cols * per_px;
                for (int i = tid; i < pieces; i += kThreads) {
                    const int c4 = i % per_px, p = i / per_px, pr = p / g.patch_cols, pc = p % g.patch_cols;
                    const int ih = ih0 + pr, iw = iw0 + pc;
                    f32x4 v = {0.f, 0.f, 0.f, 0.f};
                    if ((unsigned)ih < (unsigned)s.H && (unsigned)iw < (unsigned)s.W)
                        v = *(const f32x4*)(img + ((size_t)ih * s.W + iw) * s.C + cb * g.CB + c4 * 4);
                    *(f32x4*)(patch + pr * g.row + pc * g.px + c4 * 4) = v;
                }
            } else {
                const int per_row = g.patch_cols * s.C, pieces = g.patch_rows * per_row, wc = s.W * s.C;
                for (int i = tid; i < pieces; i += kThreads) {
                    const int pr = i / per_row, e = i % per_row;
                    const int ih = ih0 + pr, ie = iw0 * s.C + e;
                    float v = 0.f;
                    if ((unsigned)ih < (unsigned)s.H && (unsigned)ie < (unsigned)wc) v = img[(size_t)ih * wc + ie];
                    patch[pr * g.row + e] = v;
                }
            }
            __syncthreads();
            const float* bp = b_src;
            const int rows = works ? s.R : 0;
            for (int r = 0; r < rows; ++r)
                for (int t = 0; t < g.sub; ++t) {
                    const float* ap = a_src + r * g.row + t * g.px;
                    for (int c = 0; c < g.chunks; ++c) {
                        f32x4 a, b[NB];
                        if (CHAN8) a = *(const f32x4*)ap;
                        else {
                            const int left = s.S * s.C - c * 8 - 4 * half;     // elements of the window row from here on
#pragma unroll
                            for (int i = 0; i < 4; ++i) a[i] = i < left ? ap[i] : 0.f;
                        }
#pragma unroll
                        for (int j = 0; j < NB; ++j) b[j] = *(const f32x4*)(bp + j * 256);
                        ap += 8;
                        bp += NB * 256;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][i], a[i], acc[j], 0, 0, 0);
                    }
                }
            __syncthreads();      // the next block (or tile) overwrites patch and filters
        }

        // filters are the first operand: accumulator element v of lane l belongs to pixel l % 32 and filter
        // 8 * (v / 4) + 4 * (l / 32) + v % 4 of its 32
        const int p = tp * kTile + prow, q = tq * kTile + pcol;
        if (p >= s.P || q >= s.Q) continue;
        const size_t at = (((size_t)n * s.P + p) * s.Q + q) * s.K;
        auto store = [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int f = (kt * NB + j) * 32 + 8 * q4 + 4 * half;
                    if (s.K % 4 == 0 && f < s.K) {
                        f32x4 v = {acc[j][4 * q4], acc[j][4 * q4 + 1], acc[j][4 * q4 + 2], acc[j][4 * q4 + 3]};
                        v += *(const f32x4*)(bias + f);
                        if (res) v += *(const f32x4*)(res + at + f);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = act_fn<ACT>(v[i]);
                        *(f32x4*)(y + at + f) = v;
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (f + i < s.K) {
                                float v = acc[j][4 * q4 + i] + bias[f + i];
                                if (res) v += res[at + f + i];
                                y[at + f + i] = act_fn<ACT>(v);
                            }
                    }
                }
        };
        if (s.act == 1) store(std::integral_constant<int, 1>{});
        else if (s.act == 2) store(std::integral_constant<int, 2>{});
        else if (s.act == 3) store(std::integral_constant<int, 3>{});
        else store(std::integral_constant<int, 0>{});
    }
}

// Channel blocks as large as two workgroups per compute unit allow (fewer barriers), else as one allows.
bool geometry(const ConvShape& s, int NB, Geom& g, size_t& lds)
{
    g.tiles_p = (s.P + kTile - 1) / kTile;
    g.tiles_q = (s.Q + kTile - 1) / kTile;
    g.ktiles = (s.K + 32 * NB - 1) / (32 * NB);
    const long long pixel_tiles = (long long)s.N * g.tiles_p * g.tiles_q;
    if (pixel_tiles * g.ktiles > 0x7FFFFFFFll) return false;
    g.pixel_tiles = (int)pixel_tiles;
    const long long rows = (long long)(kTile - 1) * s.stride + s.R, cols = (long long)(kTile - 1) * s.stride + s.S;
    if (rows > 4096 || cols > 4096 || s.R > 4096 || s.S > 4096 || s.C > (1 << 20)) return false;
    g.patch_rows = (int)rows;
    g.patch_cols = (int)cols;
    auto fits = [&](int cb, size_t limit) {
        g.CB = cb;
        g.cblocks = s.C / cb;
        long long row;
        if (s.C % 8 == 0) {
            g.px = cb + 4;
            g.sub = s.S;
            g.chunks = cb / 8;
            row = cols * g.px;
        } else {
            g.px = s.C;
            g.sub = 1;
            g.chunks = (s.S * s.C + 7) / 8;
            row = (cols * s.C + 8 + 3) / 4 * 4;
        }
        const long long floats = (long long)s.R * g.sub * g.chunks * NB * 256 + rows * row;
        if (floats * 4 > (long long)limit) return false;
        g.row = (int)row;
        lds = (size_t)floats * 4;
        return true;
    };
    for (const size_t limit : {kLdsTwo, kLdsOne}) {
        if (s.C % 8) { if (fits(s.C, limit)) return true; continue; }
        for (int cb = 64; cb >= 8; cb /= 2)
            if (s.C % cb == 0 && fits(cb, limit)) return true;
    }
    return false;
}

// Tiles of 32 filters instead of 64, for launches whose tiles of 64 leave compute units idle.  The channel blocks, and with them the
// order of the sums, stay those of 64: a request's bits do not depend on how many run beside it.
constexpr int kTiles64 = 256;
void halve_tiles(const ConvShape& s, Geom& g, size_t& lds)
{
    lds -= (size_t)s.R * g.sub * g.chunks * 256 * sizeof(float);
    g.ktiles = (s.K + 31) / 32;
}

template <int NB, bool CHAN8>
hipError_t launch(const float* x, const float* w, const float* bias, const float* res, float* y, const ConvShape& s, const Geom& g,
                  size_t lds, hipStream_t stream)
{
    static const hipError_t configured =
        hipFuncSetAttribute((const void*)conv_f32_kernel<NB, CHAN8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsOne);
    if (configured != hipSuccess) return configured;
    const int total = g.pixel_tiles * g.ktiles;
    // with one channel block a workgroup keeps its filters from tile to tile; otherwise one tile each
    const int grid = g.cblocks == 1 && total > 512 ? 512 : total;
    hipLaunchKernelGGL((conv_f32_kernel<NB, CHAN8>), dim3(grid), dim3(kThreads), lds, stream, x, w, bias, res, y, s, g);
    return hipGetLastError();
}

}  // namespace

bool conv_f32_supported(const ConvShape& s)
{
    // An output of one pixel, most of whose window lies on the padding: the plain kernel leaves that out.  us, plain kernel / tiles:
    // 1 x 1 map, 512 -> 512, 3x3, pad 1, one image 74 / 137, 512 images 276 / 2312.  With a whole window the tiles are ahead or
    // close: 3 x 3 map without padding, 512 -> 512, 683 / 135 and 2300 / 2217; 1x1, 256 -> 256, 39 / 20 and 75 / 107.
    if (s.P * s.Q == 1) {
        const int rows = (s.R < s.H + s.pad ? s.R : s.H + s.pad) - s.pad, cols = (s.S < s.W + s.pad ? s.S : s.W + s.pad) - s.pad;
        if (2 * rows * cols <= s.R * s.S) return false;
    }
    Geom g;
    size_t lds;
    return geometry(s, s.K > 32 ? 2 : 1, g, lds);
}

hipError_t conv_f32(const void* x, const void* w, const float* bias, const void* res, void* y, const ConvShape& s,
                    hipStream_t stream)
{
    Geom g;
    size_t lds = 0;
    int nb = s.K > 32 ? 2 : 1;
    if (!geometry(s, nb, g, lds)) return hipErrorInvalidValue;
    if (g.pixel_tiles == 0) return hipSuccess;
    if (nb == 2 && (long long)g.pixel_tiles * g.ktiles <= kTiles64) {
        halve_tiles(s, g, lds);
        nb = 1;
    }
    const float *xf = (const float*)x, *wf = (const float*)w, *rf = (const float*)res;
    const bool c8 = s.C % 8 == 0;
    if (nb == 2) return c8 ? launch<2, true>(xf, wf, bias, rf, (float*)y, s, g, lds, stream) : launch<2, false>(xf, wf, bias, rf, (float*)y, s, g, lds, stream);
    return c8 ? launch<1, true>(xf, wf, bias, rf, (float*)y, s, g, lds, stream) : launch<1, false>(xf, wf, bias, rf, (float*)y, s, g, lds, stream);
}

}  // namespace k
}  // namespace coe
