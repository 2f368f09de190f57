// bf16 convolution for few input channels (the 7x7/2, C=3 stem) on the gfx950 matrix cores, optionally fused with
// the 3x3/2 max pool that follows it.
//
// With C=3 the reduction run that is contiguous in memory is one window row: S*C elements (21 for 7x7x3).  A workgroup
// stages the input patch of a 16x16 tile of conv outputs in LDS once, and every lane builds its matrix-core operand
// straight from that patch: the reduction is cut into 8-element chunks (ceil(S*C/8) per window row, zero weights where a
// chunk overhangs the row), and one v_mfma_f32_32x32x16_bf16 consumes two chunks (lanes 0-31 one, lanes 32-63 the next).
// The filters are repacked into the same chunk order in LDS once per workgroup, which then loops over many tiles.
// The patch is fetched row by row with 2-byte buffer loads through a per-row descriptor, so both image edges and
// rows outside the image read as zero without any per-element bounds arithmetic.
// Epilogue in fp32: + bias, activation, one round-to-nearest-even to bf16.
//
// Fused pool: the stem output is 1.6 MB per 224x224 image and the pool reads it straight back to keep a quarter of
// it.  In the fused form a 16x16 conv tile starts at (14t-1, 14u-1), its rounded outputs go to LDS, and the workgroup
// writes the 7x7 pooled pixels whose 3x3 windows lie inside the tile.  Rounding is monotonic, so the max of the rounded
// values equals what a separate pool kernel would produce from the stored conv output.
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
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;       // eight wavefronts per workgroup, two workgroups per compute unit (LDS): every phase of a
                                // tile (patch staging, products, epilogue, pool) is latency-bound, more waves overlap them;
                                // measured 17 % faster than four
constexpr int kThreads = 64 * kWaves;
constexpr int kRowsPerWave = 256 / kWaves;
constexpr int kMB = kRowsPerWave / 32;      // 32-row blocks per wavefront
constexpr int kTile = 16;        // conv-output tile is kTile x kTile pixels = 256 GEMM rows, 32 per wavefront
constexpr int kPoolTile = 7;     // pooled pixels per tile side in the fused form (3x3/2 windows inside 16 rows)
constexpr int kOutPad = 8;       // elements of padding per LDS row of the conv-output tile
constexpr int kMaxRowsPerWave = 48 / kWaves;   // patch rows one wavefront fetches (patch_rows <= 48)
constexpr int kMaxDwordsPerLane = 1;  // aligned dwords one lane fetches per patch row (patch_cols + 1 <= 128 elements)

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));   // round to nearest even
}
__device__ __forceinline__ float act_fn(float v, int act)
{
    if (act == 1) return v > 0.f ? v : 0.f;
    if (act == 2) return 0.5f * v * erfcf(-v * 0.70710678118654752440f);
    return v;
}
template <typename F> __device__ __forceinline__ void with_activation(int act, F&& body)
{
    if (act == 1) body(std::integral_constant<int, 1>{});
    else if (act == 2) body(std::integral_constant<int, 2>{});
    else if (act == 3) body(std::integral_constant<int, 3>{});
    else body(std::integral_constant<int, 0>{});
}

struct StemGeom {
    int tiles_p, tiles_q, total_tiles;
    int patch_rows, patch_cols;   // patch_cols = elements of one patch row that are loaded ((tile-1)*stride+S)*C
    int patch_stride;             // elements per LDS patch row (even, covers the furthest chunk read)
    int cpr;                      // 8-element chunks per window row
    int ksteps;                   // matrix-core steps = ceil(R*cpr / 2)
    int wstride;                  // elements per LDS filter row
    int PP, PQ;                   // pooled output size (fused form)
    int staged;                   // outputs go through LDS, which then holds them beside filters and patch (not fused)
};

// CPR_, R_: chunks per window row and window rows when known at compile time (the 7x7x3 stem: 3, 7), else 0: the
// reduction loop is then unrolled with constant offsets instead of running a counted loop with a carried (row, chunk).
template <int NB, bool POOL, int CPR_, int R_>
__global__ __launch_bounds__(kThreads, 4) void conv_smallc_bf16_kernel(const uint16_t* __restrict__ x,
                                                                     const uint16_t* __restrict__ w,
                                                                     const float* __restrict__ bias,
                                                                     uint16_t* __restrict__ y, ConvShape s, StemGeom g,
                                                                     const int32_t* __restrict__ rows)
{
    constexpr int K = 32 * NB;
    constexpr int OUT_STRIDE = K + kOutPad;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t* wpack = smem;                               // [K][wstride]
    uint16_t* patch = smem + K * g.wstride;               // [patch_rows][patch_stride]
    uint16_t* otile = patch + g.patch_rows * g.patch_stride;   // [256][OUT_STRIDE], fused form or staged stores (16-byte aligned)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int SC = s.S * s.C;
    const int WC = s.W * s.C;

    // filters into chunk order; zero where a chunk overhangs its window row or the step count is padded
    for (int idx = tid; idx < K * g.ksteps * 16; idx += kThreads) {
        int kk = idx / (g.ksteps * 16), e = idx % (g.ksteps * 16);
        int chunk = e >> 3, i = e & 7;
        int r = chunk / g.cpr, sc = (chunk % g.cpr) * 8 + i;
        uint16_t v = 0;
        if (r < s.R && sc < SC) v = w[((size_t)kk * s.R + r) * SC + sc];
        wpack[kk * g.wstride + e] = v;
    }
    for (int idx = tid; idx < g.patch_rows * g.patch_stride; idx += kThreads) patch[idx] = 0;
    __syncthreads();

    const int half = lane >> 5, l32 = lane & 31;
    const int tile_step = POOL ? 2 * kPoolTile : kTile;   // conv rows/cols between tile origins
    const int tile_org = POOL ? -1 : 0;

    // The patch of the NEXT tile is fetched into registers while the current tile is computed: patch rows round-robin
    // over wavefronts, lanes along the row, one aligned dword (two elements) per lane and load.  A patch row starts at
    // element g_base of its image row, which may be odd: the loads start at the even element below it and the staging
    // step shifts by one element where needed (neighbour lane's dword + one v_alignbit), so that the LDS copy starts
    // exactly at g_base and the operand reads stay 4-byte aligned.  W*C is even, so no dword straddles a row's end.
    uint32_t pre[kMaxRowsPerWave][kMaxDwordsPerLane];
    int pre_shift = 0;
    auto prefetch = [&](int tile) {
        const int n = tile / (g.tiles_p * g.tiles_q);
        const int tp = (tile / g.tiles_q) % g.tiles_p, tq = tile % g.tiles_q;
        const int ih_base = (tp * tile_step + tile_org) * s.stride - s.pad;
        const int g_base = ((tq * tile_step + tile_org) * s.stride - s.pad) * s.C;   // may be negative
        const int e0 = g_base & ~1;                                                  // even element at or below g_base
        pre_shift = g_base - e0;
        // one descriptor per image; a dword outside its row (left or right of the image) or in a row outside the image
        // gets an offset beyond the descriptor's range and reads as zero
        // (with a row table, image n of the launch is image rows[n] of the array at x: request arranging's gather of
        // the inputs happens here instead of in a copy of its own)
        const int n_src = rows ? __builtin_amdgcn_readfirstlane(rows[n]) : n;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x + (size_t)n_src * s.H * WC), 0, s.H * WC * 2, 0x00020000);
#pragma unroll
        for (int j = 0; j < kMaxDwordsPerLane; ++j) {
            const int e = e0 + 2 * (lane + 64 * j);
            const bool col_ok = (unsigned)e < (unsigned)WC;                          // WC is even: e + 1 < WC as well
#pragma unroll
            for (int i = 0; i < kMaxRowsPerWave; ++i) {
                const int pr = wid + i * (kThreads / 64);
                const int ih = ih_base + pr;
                const bool ok = col_ok && pr < g.patch_rows && (unsigned)ih < (unsigned)s.H;
                pre[i][j] = __builtin_amdgcn_raw_buffer_load_b32(rs, ok ? (ih * WC + e) * 2 : (int)0x80000000, 0, 0);
            }
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int i = 0; i < kMaxRowsPerWave; ++i) {
            const int pr = wid + i * (kThreads / 64);
            if (pr < g.patch_rows) {
#pragma unroll
                for (int j = 0; j < kMaxDwordsPerLane; ++j) {
                    uint32_t v = pre[i][j];
                    if (pre_shift) {
                        // the dword one position further along the row: the next lane's, or lane 0's of the next load
                        uint32_t nb = __shfl_down(v, 1);
                        if (j + 1 < kMaxDwordsPerLane) {
                            const uint32_t first_of_next = __builtin_amdgcn_readfirstlane(pre[i][j + 1 < kMaxDwordsPerLane ? j + 1 : j]);
                            if (lane == 63) nb = first_of_next;
                        }
                        v = __builtin_amdgcn_alignbit(nb, v, 16);
                    }
                    const int col = 2 * (lane + 64 * j);
                    if (col + 1 >= g.patch_cols) v &= 0xFFFFu;            // nothing beyond the patch reaches LDS
                    if (col < g.patch_cols) *(uint32_t*)(patch + pr * g.patch_stride + col) = v;
                }
            }
        }
    };

    if ((int)blockIdx.x < g.total_tiles) prefetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < g.total_tiles; tile += gridDim.x) {
        const int n = tile / (g.tiles_p * g.tiles_q);
        const int tp = (tile / g.tiles_q) % g.tiles_p, tq = tile % g.tiles_q;
        const int p0 = tp * tile_step + tile_org, q0 = tq * tile_step + tile_org;     // conv-output origin of the tile
        commit();
        __syncthreads();
        if (tile + (int)gridDim.x < g.total_tiles) prefetch(tile + gridDim.x);

        f32x16 acc[kMB][NB];
#pragma unroll
        for (int i = 0; i < kMB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

        int a_off[kMB];
#pragma unroll
        for (int i = 0; i < kMB; ++i) {
            int ml = wid * kRowsPerWave + i * 32 + l32;
            a_off[i] = (ml / kTile) * s.stride * g.patch_stride + (ml % kTile) * s.stride * s.C;
        }
        auto kstep = [&](int koff, int chunk) {
            bf16x8 af[kMB], bfr[NB];
#pragma unroll
            for (int i = 0; i < kMB; ++i) {
                const uint32_t* p32 = (const uint32_t*)(patch + a_off[i] + koff);      // 4-byte aligned by construction
                uint4 v = make_uint4(p32[0], p32[1], p32[2], p32[3]);
                af[i] = __builtin_bit_cast(bf16x8, v);
            }
#pragma unroll
            for (int jn = 0; jn < NB; ++jn)
                bfr[jn] = *(const bf16x8*)(wpack + (jn * 32 + l32) * g.wstride + chunk * 8);
            // filter fragment first: a lane then holds 4 consecutive output channels of one pixel per accumulator quad
#pragma unroll
            for (int i = 0; i < kMB; ++i)
#pragma unroll
                for (int jn = 0; jn < NB; ++jn)
                    acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[jn], af[i], acc[i][jn], 0, 0, 0);
        };
        if constexpr (CPR_ > 0) {
            constexpr int KSTEPS = (R_ * CPR_ + 1) / 2;
#pragma unroll
            for (int j = 0; j < KSTEPS; ++j) {
                // chunk 2j (lanes 0-31) and 2j+1 (lanes 32-63): window row and chunk inside it are constants; a padded
                // last chunk reads the last window row again (its filters are zero, any finite data will do)
                const int c0 = 2 * j, c1 = 2 * j + 1;
                const int r0 = c0 / CPR_ < R_ ? c0 / CPR_ : R_ - 1, r1 = c1 / CPR_ < R_ ? c1 / CPR_ : R_ - 1;
                const int off0 = r0 * g.patch_stride + (c0 % CPR_) * 8, off1 = r1 * g.patch_stride + (c1 % CPR_) * 8;
                kstep(half ? off1 : off0, 2 * j + half);
            }
        } else {
            int kr = half / g.cpr, kpart = half % g.cpr;          // window row and chunk inside it of this lane's chunk
            for (int j = 0; j < g.ksteps; ++j) {
                const int r = kr < s.R ? kr : s.R - 1;             // padded step: filters are zero, any finite data will do
                kstep(r * g.patch_stride + kpart * 8, 2 * j + half);
                kpart += 2;                                        // next step: two chunks on, without a division
                while (kpart >= g.cpr) { kpart -= g.cpr; ++kr; }
            }
        }

        // (dispatched once on the activation: a per-element test compiles into hundreds of branches)
        with_activation(s.act, [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
        // accumulator element v of lane l: pixel l%32 of the 32-pixel block, filter 8*(v/4) + 4*(l/32) + v%4
#pragma unroll
        for (int i = 0; i < kMB; ++i) {
            const int ml = wid * kRowsPerWave + i * 32 + l32;
            const int p = p0 + ml / kTile, q = q0 + ml % kTile;
            const bool inside = (unsigned)p < (unsigned)s.P && (unsigned)q < (unsigned)s.Q;
#pragma unroll
            for (int jn = 0; jn < NB; ++jn)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int ch = jn * 32 + 8 * gq + half * 4;
                    const float4 bv = *(const float4*)(bias + ch);
                    float v[4] = {acc[i][jn][4 * gq + 0] + bv.x, acc[i][jn][4 * gq + 1] + bv.y, acc[i][jn][4 * gq + 2] + bv.z,
                                  acc[i][jn][4 * gq + 3] + bv.w};
                    if constexpr (ACT == 3) {
                        silu_for_bf16(v);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = act_fn(v[e], ACT);
                    }
                    uint2 o;
                    o.x = pack_bf16(v[0], v[1]);
                    o.y = pack_bf16(v[2], v[3]);
                    if (POOL) {
                        // outside the conv output: -inf (or 0 after ReLU, see the pool below) never wins the max
                        if (!inside) o = ACT == 1 ? make_uint2(0u, 0u) : make_uint2(0xFF80FF80u, 0xFF80FF80u);
                        *(uint2*)(otile + ml * OUT_STRIDE + ch) = o;
                    } else if (g.staged) {
                        *(uint2*)(otile + ml * OUT_STRIDE + ch) = o;
                    } else if (inside) {
                        *(uint2*)(y + (((size_t)n * s.P + p) * s.Q + q) * K + ch) = o;
                    }
                }
        }
        });
        if (!POOL && g.staged) {
            // whole rows of channels, 16 bytes per lane, out of the wavefront's own rows (its LDS operations keep their order)
            static_assert(kMB == 1, "32 pixels per wavefront");
#pragma unroll
            for (int k = 0; k < K / 16; ++k) {
                const int idx = lane + 64 * k, ml = wid * kRowsPerWave + idx / (K / 8), c8 = idx % (K / 8);
                const int p = p0 + ml / kTile, q = q0 + ml % kTile;
                const uint4 v = *(const uint4*)(otile + ml * OUT_STRIDE + c8 * 8);
                if ((unsigned)p < (unsigned)s.P && (unsigned)q < (unsigned)s.Q) *(uint4*)(y + (((size_t)n * s.P + p) * s.Q + q) * K + c8 * 8) = v;
            }
        }
        if (POOL) {
            __syncthreads();
            // 7x7 pooled pixels x K/8 channel groups; window of pooled (a, b) = tile rows 2a..2a+2, cols 2b..2b+2
            for (int item = tid; item < kPoolTile * kPoolTile * (K / 8); item += kThreads) {
                const int c8 = item % (K / 8), pix = item / (K / 8);
                const int a = pix / kPoolTile, b = pix % kPoolTile;
                const int pi = tp * kPoolTile + a, pj = tq * kPoolTile + b;
                if (pi >= g.PP || pj >= g.PQ) continue;
                if (s.act == 1) {
                    // after ReLU every value is >= +0, and non-negative bf16 order like their bit patterns: the max is
                    // a packed 16-bit integer max, two channels per instruction (tile pixels outside the conv output
                    // hold 0 here, which never beats a real value)
                    u16x2 m[4] = {u16x2{0, 0}, u16x2{0, 0}, u16x2{0, 0}, u16x2{0, 0}};
#pragma unroll
                    for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                        for (int dc = 0; dc < 3; ++dc) {
                            const uint4 v = *(const uint4*)(otile + ((2 * a + dr) * kTile + 2 * b + dc) * OUT_STRIDE + c8 * 8);
                            m[0] = __builtin_elementwise_max(m[0], __builtin_bit_cast(u16x2, v.x));
                            m[1] = __builtin_elementwise_max(m[1], __builtin_bit_cast(u16x2, v.y));
                            m[2] = __builtin_elementwise_max(m[2], __builtin_bit_cast(u16x2, v.z));
                            m[3] = __builtin_elementwise_max(m[3], __builtin_bit_cast(u16x2, v.w));
                        }
                    uint4 o;
                    o.x = __builtin_bit_cast(uint32_t, m[0]); o.y = __builtin_bit_cast(uint32_t, m[1]);
                    o.z = __builtin_bit_cast(uint32_t, m[2]); o.w = __builtin_bit_cast(uint32_t, m[3]);
                    *(uint4*)(y + (((size_t)n * g.PP + pi) * g.PQ + pj) * K + c8 * 8) = o;
                    continue;
                }
                float best[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
#pragma unroll
                for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                    for (int dc = 0; dc < 3; ++dc) {
                        const uint4 v = *(const uint4*)(otile + ((2 * a + dr) * kTile + 2 * b + dc) * OUT_STRIDE + c8 * 8);
                        const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            best[2 * e] = fmaxf(best[2 * e], __uint_as_float(wds[e] << 16));
                            best[2 * e + 1] = fmaxf(best[2 * e + 1], __uint_as_float(wds[e] & 0xFFFF0000u));
                        }
                    }
                uint4 o;
                o.x = (__float_as_uint(best[0]) >> 16) | (__float_as_uint(best[1]) & 0xFFFF0000u);
                o.y = (__float_as_uint(best[2]) >> 16) | (__float_as_uint(best[3]) & 0xFFFF0000u);
                o.z = (__float_as_uint(best[4]) >> 16) | (__float_as_uint(best[5]) & 0xFFFF0000u);
                o.w = (__float_as_uint(best[6]) >> 16) | (__float_as_uint(best[7]) & 0xFFFF0000u);
                *(uint4*)(y + (((size_t)n * g.PP + pi) * g.PQ + pj) * K + c8 * 8) = o;
            }
        }
        __syncthreads();      // patch (and the conv-output tile) are rewritten by the next tile
    }
}

// ---------------------------------------------------------------------------------------------------------------
// The 7x7/2 stem on three channels with ReLU and the fused 3x3/2 pool, as every ResNet-shaped expert begins: no tiles in
// LDS and no barriers.  A wavefront walks down a strip of 32 conv columns (15 pooled ones at most) and keeps in registers
//   * the operands of four pairs of input rows, (2i + 1, 2i + 2) for i = p - 2 .. p + 1, which are what conv row p needs
//     (its window rows are 2p - 3 .. 2p + 3; the last row of the last pair is left out).  A window row is the 21 elements of
//     columns 2q - 3 .. 2q + 3 in three chunks of 8, as in conv_smallc_bf16_kernel: the sums run in its order and give its bits.
//     A window begins at an odd element, so a lane loads a chunk straight from the image as the five dwords around it, 16 + 4
//     bytes, and one byte permutation per dword moves it into place and puts zeros for what lies left or right of the image
//     or behind the window.  The next pair is loaded into the registers of the pair that has just been used for the last
//     time, a whole conv row before it is needed;
//   * the running maximum of a pooled row's conv rows, after the bias.
// The filters are packed into LDS in fragment order once per workgroup and read again for every conv row.  (In registers,
// as far as they fit, they gain nothing: 1.39 ms per 4096 images with one to four of the eleven steps resident; with five and
// six the compiler spills: 1.68 and 2.12 ms.)
// Lanes 0-15 of a half hold the odd conv columns 2b - 1, lanes 16-31 the even ones 2b (b = pooled column), so that the
// horizontal maximum is one row swap and one shift within 16 lanes, after which all lanes hold results; swapping halves
// then gives a lane 8 consecutive channels to store.  ReLU and rounding are monotonic: they come after the vertical maximum
// (fp32), the horizontal one compares non-negative bf16 as integers.
// Bound by the matrix cores and the vector instructions between them: 44 of 32 cycles per strip and pooled row beside about
// 220 of 4 cycles, which the second wavefront of the SIMD overlaps in part.  Groups with filters of their own share a launch.
// Measured, 224 x 224: 4096 images 2.60 ms with 16 x 16 tiles in LDS (conv_smallc_bf16_kernel), 1.42 here (0.7 for the matrix
// instructions alone at their full rate, 0.6 for the bytes; 1.39 with windows read from an even element on, without the fifth dword);
// 29 images in 15 groups 15 launches of 17 us, now one of 22.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kStripPooled = 15;      // pooled columns per strip: 2 * 15 + 1 conv columns of 32
constexpr int kStripWaves = 4;
constexpr int kStripSlots = 2048;     // wavefronts the chip holds at two per SIMD
constexpr int kStemSteps = 11;
constexpr int kStemResident = 2;      // steps whose filter fragments stay in registers: a conv row begins without waiting for LDS

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct StripGeom {
    int PP, PQ;                       // pooled size
    int strips, strip_cols;           // strips per image, pooled columns of a strip
    int segs, seg_rows;               // segments of a strip, pooled rows of a segment
};
// Groups with filters of their own: a workgroup belongs to one of them
struct StripGroups {
    int n;
    int first_wg[kMaxGroups + 1];     // first workgroup of each group
    int out[kMaxGroups + 1];          // first image of each group in the output
    int in[kMaxGroups];               // first image (or row table entry) of each group in the input
    const void* weights[kMaxGroups];
    int64_t off_w, off_b;             // bytes from there to the filters and the bias
};

__global__ __launch_bounds__(64 * kStripWaves, 2) void conv_stem_strip_kernel(const uint16_t* __restrict__ x,
                                                                              uint16_t* __restrict__ y, ConvShape s, StripGeom g,
                                                                              StripGroups gr, const int32_t* __restrict__ rows)
{
    constexpr int kFrags = 2 * kStemSteps;
    __shared__ __attribute__((aligned(16))) uint16_t wpack[kFrags * 512];     // [step][filter block][lane][8]
    __shared__ float4 lbias[32];                               // the bias; minus infinity, for a conv row that does not exist
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    int grp = 0;
    while (grp + 1 < gr.n && (int)blockIdx.x >= gr.first_wg[grp + 1]) ++grp;
    const int wg = blockIdx.x - gr.first_wg[grp], wgs = gr.first_wg[grp + 1] - gr.first_wg[grp];
    const int tasks = (gr.out[grp + 1] - gr.out[grp]) * g.segs * g.strips;
    const uint16_t* const w = (const uint16_t*)((const char*)gr.weights[grp] + gr.off_w);
    const float* const bias = (const float*)((const char*)gr.weights[grp] + gr.off_b);

    // chunk c of window row r is elements 8c .. 8c + 7 of its 21 (zero behind them); lanes 0-31 of step j take chunk 2j,
    // lanes 32-63 chunk 2j + 1, counted over all rows
    constexpr int kChunks = kFrags * 64, kPerThread = (kChunks + 64 * kStripWaves - 1) / (64 * kStripWaves);
    uint32_t packed[kPerThread][4];                            // (all loads in flight at once)
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
        const int idx = tid + t * 64 * kStripWaves, l = idx & 63, f = idx >> 6;
        const int k = (f & 1) * 32 + (l & 31), chunk = (f >> 1) * 2 + (l >> 5);
        const int r = chunk / 3, e0 = chunk % 3 * 8;
        const bool row_ok = idx < kChunks && r < 7;
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const bool ok = row_ok && e0 + i < 21;
            const uint32_t loaded = w[ok ? (k * 7 + r) * 21 + e0 + i : 0];
            v[i] = ok ? loaded : 0u;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) packed[t][i] = v[2 * i] | v[2 * i + 1] << 16;
    }
#pragma unroll
    for (int t = 0; t < kPerThread; ++t)
        if (tid + t * 64 * kStripWaves < kChunks) *(u32x4*)(wpack + (tid + t * 64 * kStripWaves) * 8) = u32x4{packed[t][0], packed[t][1], packed[t][2], packed[t][3]};
    if (tid < 16) lbias[tid] = *(const float4*)(bias + 4 * tid);
    else if (tid < 32) lbias[tid] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    __syncthreads();
    bf16x8 fil[kStemResident][2];
#pragma unroll
    for (int j = 0; j < kStemResident; ++j)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) fil[j][nb] = *(const bf16x8*)(wpack + ((j * 2 + nb) * 64 + lane) * 8);

    const int H = s.H, WC = s.W * 3, row_bytes = WC * 2;
    const int col = lane & 15, even = (lane >> 4) & 1;
    // step ks of a pair: chunks (0 | 1) of its first row, (2 of the first | 0 of the second), (1 | 2) of the second
    for (int task = wg * kStripWaves + wid; task < tasks; task += wgs * kStripWaves) {
        const int strip = task % g.strips, seg = task / g.strips % g.segs, image = task / g.strips / g.segs;
        const int n = gr.out[grp] + image;
        const int b0 = strip * g.strip_cols, cols = g.PQ - b0 < g.strip_cols ? g.PQ - b0 : g.strip_cols;
        const int a0 = seg * g.seg_rows, a_end = a0 + g.seg_rows < g.PP ? a0 + g.seg_rows : g.PP;
        const int q = 2 * (b0 + col) - 1 + even;
        const uint32_t col_mask = (unsigned)q < (unsigned)s.Q ? ~0u : 0u;       // a column that does not exist is 0: never more than the maximum after ReLU
        const int e_q = 6 * q - 9, e_end = e_q + 21 < WC ? e_q + 21 : WC;           // the window's elements of an image row
        const int e_of[3] = {e_q + 8 * half, half ? e_q : e_q + 16, e_q + 8 + 8 * half};
        // selectors of the byte permutations: the upper half of one dword and the lower half of the next, or zeros
        u32x4 pick[3];
#pragma unroll
        for (int ks = 0; ks < 3; ++ks)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int e = e_of[ks] + 2 * d;
                pick[ks][d] = (e >= 0 && e < e_end ? 0x0302u : 0x0C0Cu) | (e + 1 >= 0 && e + 1 < e_end ? 0x05040000u : 0x0C0C0000u);
            }
        const int n_src = rows ? __builtin_amdgcn_readfirstlane(rows[gr.in[grp] + image]) : gr.in[grp] + image;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x + (size_t)n_src * H * WC), 0, H * row_bytes, 0x00020000);
        // the dword that holds the element before a chunk and its first one
        const int off[3] = {e_of[0] * 2 - 2, e_of[1] * 2 - 2 + half * row_bytes, e_of[2] * 2 - 2 + row_bytes};

        u32x4 in[4][3];                                        // [pair][step]; as loaded without the fifth dwords
        struct Fifth { uint32_t d[3]; };
        // Offsets before the image (as unsigned) and behind it read as zero, and what a lane reads beyond a row's ends is
        // not picked; only a chunk that begins left of the image's first row and reaches into it needs the other form.
        auto load_pair = [&](u32x4 (&to)[3], Fifth& fifth, int i) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                to[ks] = __builtin_amdgcn_raw_buffer_load_b128(rs, off[ks] + (2 * i + 1) * row_bytes, 0, 0);
                fifth.d[ks] = __builtin_amdgcn_raw_buffer_load_b32(rs, off[ks] + (2 * i + 1) * row_bytes + 16, 0, 0);
            }
        };
        auto load_first_pair = [&](u32x4 (&to)[3], Fifth& fifth) __attribute__((always_inline)) {     // rows -1 and 0
#pragma unroll
            for (int ks = 0; ks < 3; ++ks) {
                const bool row = ks == 2 || (ks == 1 && half);
#pragma unroll
                for (int d = 0; d < 5; ++d) {
                    const int e = e_of[ks] - 1 + 2 * d;
                    const uint32_t v = __builtin_amdgcn_raw_buffer_load_b32(rs, row && (unsigned)e < (unsigned)WC ? e * 2 : (int)0x80000000, 0, 0);
                    if (d < 4) to[ks][d] = v;
                    else fifth.d[ks] = v;
                }
            }
        };
        auto place_pair = [&](u32x4 (&v)[3], const Fifth& fifth) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < 3; ++ks)
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    v[ks][d] = __builtin_amdgcn_perm(d < 3 ? v[ks][d < 3 ? d + 1 : 3] : fifth.d[ks], v[ks][d], pick[ks][d]);
        };
        Fifth fifth[2];                                        // of the pair that is on its way and of the one before it
        f32x16 acc[2];
        // conv row p, its pairs in slots base .. base + 3; the next pair goes to slot base
        auto conv_row = [&](auto base_c, int p) __attribute__((always_inline)) {
            constexpr int base = decltype(base_c)::value;
            acc[0] = f32x16{};
            acc[1] = f32x16{};
            int fil_at = lane * 8;
            asm volatile("" : "+v"(fil_at));                   // (not kept across conv rows)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                u32x4(&pair)[3] = in[(base + j) & 3];
                if (j == 3) place_pair(pair, fifth[(base + 1) & 1]);
#pragma unroll
                for (int ks = 0; ks < 3; ++ks) {
                    if (j == 3 && ks == 2) continue;           // the eighth row
                    u32x4 v = pair[ks];
                    if (j == 3 && ks == 1) v = half ? u32x4{0u, 0u, 0u, 0u} : v;
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) {
                        const int step = 3 * j + ks;
                        const bf16x8 f = step < kStemResident ? fil[step < kStemResident ? step : 0][nb]
                                                              : *(const bf16x8*)(wpack + (step * 2 + nb) * 512 + fil_at);
                        acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, __builtin_bit_cast(bf16x8, v), acc[nb], 0, 0, 0);
                    }
                }
                if (j == 0) load_pair(pair, fifth[base & 1], p + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        float top[2][16];                                      // running maximum of the pooled row
        // f(nb, element, conv output with its bias)
        auto each = [&](int p, auto&& f) __attribute__((always_inline)) {
            int at = half + ((unsigned)p < (unsigned)s.P ? 0 : 16);
            asm volatile("" : "+v"(at));                       // (read again each time: 32 registers less)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const float4 bv = lbias[at + nb * 8 + gq * 2];
                    f(nb, gq * 4 + 0, acc[nb][gq * 4 + 0] + bv.x);
                    f(nb, gq * 4 + 1, acc[nb][gq * 4 + 1] + bv.y);
                    f(nb, gq * 4 + 2, acc[nb][gq * 4 + 2] + bv.z);
                    f(nb, gq * 4 + 3, acc[nb][gq * 4 + 3] + bv.w);
                }
        };
        uint16_t* y_at = y + ((size_t)(n * (size_t)g.PP + a0) * g.PQ + b0 + col) * 64 + 8 * (2 * half + even);
        // pooled row a from conv rows 2a - 1 (in `top`), 2a and 2a + 1
        auto pooled_row = [&](auto base_c, int a) __attribute__((always_inline)) {
            constexpr int base = decltype(base_c)::value;
            conv_row(std::integral_constant<int, base>{}, 2 * a);
            each(2 * a, [&](int nb, int v, float t) __attribute__((always_inline)) { top[nb][v] = fmaxf(top[nb][v], t); });
            conv_row(std::integral_constant<int, (base + 1) & 3>{}, 2 * a + 1);
            u16x2 m[2][4][2];                                  // [filter block][quad][channel pair]
            float out[2][16];
            each(2 * a + 1, [&](int nb, int v, float t) __attribute__((always_inline)) {
                out[nb][v] = fmaxf(fmaxf(top[nb][v], t), 0.f);
                top[nb][v] = t;
            });
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    const uint32_t o = pack_bf16(out[nb][v], out[nb][v + 1]) & col_mask;
                    m[nb][v / 4][v % 4 / 2] = __builtin_bit_cast(u16x2, o);
                }
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                uint32_t r[2][2];                              // [quad pair][channel pair]
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        // odd columns of both quads, then even columns of both
                        const auto sw = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, m[nb][2 * h][d]),
                                                                         __builtin_bit_cast(uint32_t, m[nb][2 * h + 1][d]), false, false);
                        const uint32_t right = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sw[0], 0x101, 0xF, 0xF, true);   // row_shl:1
                        const u16x2 c = __builtin_elementwise_max(__builtin_bit_cast(u16x2, (uint32_t)sw[0]), __builtin_bit_cast(u16x2, (uint32_t)sw[1]));
                        r[h][d] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(c, __builtin_bit_cast(u16x2, right)));
                    }
                const auto s0 = __builtin_amdgcn_permlane32_swap(r[0][0], r[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(r[0][1], r[1][1], false, false);
                if (col < cols) *(u32x4*)(y_at + nb * 32) = u32x4{(uint32_t)s0[0], (uint32_t)s1[0], (uint32_t)s0[1], (uint32_t)s1[1]};
            }
            y_at += (size_t)g.PQ * 64;
        };

        const int p0 = 2 * a0 - 1;
        Fifth first[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) load_pair(in[j], first[j], p0 - 2 + j);
        load_pair(in[3], fifth[1], p0 + 1);
        if (p0 == -1) load_first_pair(in[2], first[2]);
        if (p0 == 1) load_first_pair(in[0], first[0]);
#pragma unroll
        for (int j = 0; j < 3; ++j) place_pair(in[j], first[j]);
        conv_row(std::integral_constant<int, 0>{}, p0);
        each(p0, [&](int nb, int v, float t) __attribute__((always_inline)) { top[nb][v] = t; });
        for (int a = a0;;) {
            pooled_row(std::integral_constant<int, 1>{}, a);
            if (++a == a_end) break;
            pooled_row(std::integral_constant<int, 3>{}, a);
            if (++a == a_end) break;
        }
    }
}

// the shapes of conv_stem_strip_kernel (for any number of images: a request's bits do not depend on what runs beside it)
bool strip_supported(const ConvShape& s)
{
    return s.C == 3 && s.K == 64 && s.R == 7 && s.S == 7 && s.stride == 2 && s.pad == 3 && s.act == 1 && s.W % 2 == 0 && s.P >= 2 &&
           s.Q >= 2 && (long long)s.H * s.W * s.C * 2 < 0x3FFFFFFFll;
}

// Launches the strips of all groups of gr (n, out, in, weights and offsets set).  Segments: what matters is the number of conv rows
// of the wavefront that has the most; a segment has two per pooled row, one above, and the time of about three until its first
// loads are there.  All workgroups are resident at once.
hipError_t launch_strip(const void* x, void* y, const ConvShape& s, StripGroups& gr, hipStream_t stream, const int32_t* rows)
{
    StripGeom g{};
    g.PP = (s.P + 2 - 3) / 2 + 1;
    g.PQ = (s.Q + 2 - 3) / 2 + 1;
    g.strips = (g.PQ + kStripPooled - 1) / kStripPooled;
    g.strip_cols = (g.PQ + g.strips - 1) / g.strips;
    long long best = 0, best_each = 0;
    for (int r = 1; r <= g.PP; ++r) {
        const int segs = (g.PP + r - 1) / r;
        const long long per_image = (long long)g.strips * segs;
        if ((long long)s.N * per_image > 0x3FFFFFFFll) continue;
        // strips a wavefront takes, so that the workgroups of all groups fit the chip
        long long each = ((long long)s.N * per_image + kStripSlots - 1) / kStripSlots, wgs;
        do {
            wgs = 0;
            for (int i = 0; i < gr.n; ++i) wgs += ((gr.out[i + 1] - gr.out[i]) * per_image + kStripWaves * each - 1) / (kStripWaves * each);
        } while (wgs > kStripSlots / kStripWaves && ++each);
        const long long cost = each * (2 * r + 4);
        if (best == 0 || cost < best) { best = cost; best_each = each; g.segs = segs; g.seg_rows = r; }
    }
    if (best == 0) return hipErrorInvalidValue;
    gr.first_wg[0] = 0;
    for (int i = 0; i < gr.n; ++i)
        gr.first_wg[i + 1] = gr.first_wg[i] + (int)(((long long)(gr.out[i + 1] - gr.out[i]) * g.strips * g.segs + kStripWaves * best_each - 1) /
                                                    (kStripWaves * best_each));
    if (gr.first_wg[gr.n] == 0) return hipSuccess;
    hipLaunchKernelGGL(conv_stem_strip_kernel, dim3(gr.first_wg[gr.n]), dim3(64 * kStripWaves), 0, stream, (const uint16_t*)x, (uint16_t*)y,
                       s, g, gr, rows);
    return hipGetLastError();
}

bool geometry(const ConvShape& s, bool pool, StemGeom& g, size_t& smem)
{
    if (s.K != 32 && s.K != 64) return false;
    if (s.C <= 0 || s.C % 32 == 0) return false;
    if ((s.stride * s.C) % 2) return false;                        // chunk reads must stay 4-byte aligned
    int SC = s.S * s.C;
    g.cpr = (SC + 7) / 8;
    g.ksteps = (s.R * g.cpr + 1) / 2;
    g.wstride = g.ksteps * 16 + 8;
    g.patch_rows = (kTile - 1) * s.stride + s.R;
    g.patch_cols = ((kTile - 1) * s.stride + s.S) * s.C;
    int furthest = (kTile - 1) * s.stride * s.C + g.cpr * 8;       // one past the last element any chunk read touches
    int ps = g.patch_cols > furthest ? g.patch_cols : furthest;
    g.patch_stride = (ps + 7) / 8 * 8 + 8;                         // multiple of 8: the regions after it stay 16-byte aligned
    // The 32 lanes of an operand read cover two rows of the conv tile, 16 pixels each, stride * C elements apart inside a row:
    // dword 3 l for lane l of a row with the 7x7x3 stem's 6 elements per pixel.  Two tile rows are stride * patch_stride
    // elements apart; when that is a multiple of 32 dwords both rows hit the same 16 banks.  Shift it to 16 dwords mod 32:
    // the second row's banks (3 l + 16 mod 32) then fall between the first row's.
    for (int extra = 0; extra < 64; extra += 8)
        if ((s.stride * (g.patch_stride + extra) / 2) % 32 == 16) { g.patch_stride += extra; break; }
    if ((long long)s.H * s.W * s.C * 2 >= 0x7FFFFFFFll) return false;    // byte offsets inside one image are 31-bit
    if (g.patch_rows > kMaxRowsPerWave * (kThreads / 64) || g.patch_cols + 1 > kMaxDwordsPerLane * 128) return false;
    if ((s.W * s.C) % 2) return false;                             // aligned dwords must not straddle the end of an image row
    g.PP = (s.P + 2 - 3) / 2 + 1;
    g.PQ = (s.Q + 2 - 3) / 2 + 1;
    if (pool) {
        if (s.P < 2 || s.Q < 2) return false;
        g.tiles_p = (g.PP + kPoolTile - 1) / kPoolTile;
        g.tiles_q = (g.PQ + kPoolTile - 1) / kPoolTile;
    } else {
        g.tiles_p = (s.P + kTile - 1) / kTile;
        g.tiles_q = (s.Q + kTile - 1) / kTile;
    }
    long long total = (long long)s.N * g.tiles_p * g.tiles_q;
    if (total > 0x7FFFFFFFll) return false;
    g.total_tiles = (int)total;
    smem = sizeof(uint16_t) * ((size_t)s.K * g.wstride + (size_t)g.patch_rows * g.patch_stride);
    const size_t otile = sizeof(uint16_t) * (size_t)kTile * kTile * (s.K + kOutPad);
    // Whole lines of the output through LDS instead of 8-byte pieces out of the accumulators, as long as two workgroups share a compute
    // unit.  With that and its reduction unrolled the 6x6/2 stem (3 -> 64 channels, SiLU, 224 x 224) takes 188 us instead of 262 for 250
    // images (the output alone is 80 us of HBM traffic), 66 instead of 88 for 64, 15.0 instead of 18.5 for one; about a third of
    // that is the shorter SiLU.  3x3/2 on 112 x 112 without activation, 100 images: 34 / 29 us.
    g.staged = !pool && smem + otile <= 80 * 1024;
    if (pool || g.staged) smem += otile;
    return smem <= 96 * 1024;
}

template <int NB, bool POOL, int CPR_, int R_>
hipError_t launch(const void* x, const void* w, const float* bias, void* y, const ConvShape& s, const StemGeom& g, size_t smem,
                  hipStream_t stream, const int32_t* rows)
{
    static bool configured = false;
    if (!configured) {   // more than the default 64 KiB of LDS per workgroup needs an explicit opt-in
        hipError_t e = hipFuncSetAttribute((const void*)conv_smallc_bf16_kernel<NB, POOL, CPR_, R_>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
        if (e != hipSuccess) return e;
        configured = true;
    }
    // Workgroups that take tiles in turn: with staged stores of 64 channels the 512 that the chip holds (registers and LDS: two per
    // compute unit), so that all start at once.  us with 1024 / 512: 7x7/2 (3 -> 64, 224 x 224) 16 images 31 / 25, 44 images 57 / 38, 64
    // images 67 / 50, 250 images 171 / 168; 6x6/2 with SiLU 64 images 58 / 51.  Of 32 channels the chip holds more: 7x7/2, 224 x 224,
    // 64 images 37 / 36, 250 images 104 / 110.
    const int most = g.staged && NB == 2 ? 512 : 1024;
    const int grid = g.total_tiles < most ? g.total_tiles : most;
    hipLaunchKernelGGL((conv_smallc_bf16_kernel<NB, POOL, CPR_, R_>), dim3(grid), dim3(kThreads), smem, stream, (const uint16_t*)x,
                       (const uint16_t*)w, bias, (uint16_t*)y, s, g, rows);
    return hipGetLastError();
}

}  // namespace

bool conv_smallc_supported(const ConvShape& s, bool has_res, bool fused_pool)
{
    StemGeom g;
    size_t smem;
    return !has_res && geometry(s, fused_pool, g, smem);
}

hipError_t conv_smallc(const void* x, const void* w, const float* bias, void* y, const ConvShape& s, bool fused_pool,
                       hipStream_t stream, const int32_t* rows)
{
    StemGeom g;
    size_t smem = 0;
    if (!geometry(s, fused_pool, g, smem)) return hipErrorInvalidValue;
    if (g.total_tiles == 0) return hipSuccess;
    if (s.K == 64) {
        if (fused_pool && strip_supported(s)) {
            StripGroups gr{};
            gr.n = 1;
            gr.out[1] = s.N;
            gr.weights[0] = w;
            gr.off_b = (const char*)bias - (const char*)w;
            return launch_strip(x, y, s, gr, stream, rows);
        }
        if (fused_pool && g.cpr == 3 && s.R == 7)         // reduction loop unrolled with constant offsets
            return launch<2, true, 3, 7>(x, w, bias, y, s, g, smem, stream, rows);
        if (!fused_pool && g.cpr == 3 && s.R == 6) return launch<2, false, 3, 6>(x, w, bias, y, s, g, smem, stream, rows);
        return fused_pool ? launch<2, true, 0, 0>(x, w, bias, y, s, g, smem, stream, rows)
                          : launch<2, false, 0, 0>(x, w, bias, y, s, g, smem, stream, rows);
    }
    return fused_pool ? launch<1, true, 0, 0>(x, w, bias, y, s, g, smem, stream, rows)
                      : launch<1, false, 0, 0>(x, w, bias, y, s, g, smem, stream, rows);
}

bool conv_smallc_groupable(const ConvShape& s, bool fused_pool)
{
    return fused_pool && strip_supported(s);
}

hipError_t conv_smallc_grouped(const void* x, const int32_t* first_in, const GroupTable& groups, size_t off_w, size_t off_b, void* y,
                               const ConvShape& s, bool fused_pool, hipStream_t stream, const int32_t* rows)
{
    if (!conv_smallc_groupable(s, fused_pool) || groups.n <= 0 || groups.n > kMaxGroups || groups.first_row[0] != 0 ||
        groups.first_row[groups.n] != s.N || off_w > 0x7FFFFFFFull || off_b > 0x7FFFFFFFull)
        return hipErrorInvalidValue;
    StripGroups gr{};
    gr.n = groups.n;
    for (int i = 0; i < groups.n; ++i) {
        if (groups.first_row[i + 1] < groups.first_row[i] || !groups.weights[i]) return hipErrorInvalidValue;
        gr.out[i + 1] = groups.first_row[i + 1];
        gr.in[i] = first_in[i];
        gr.weights[i] = groups.weights[i];
    }
    gr.off_w = (int64_t)off_w;
    gr.off_b = (int64_t)off_b;
    return launch_strip(x, y, s, gr, stream, rows);
}

}  // namespace k
}  // namespace coe
