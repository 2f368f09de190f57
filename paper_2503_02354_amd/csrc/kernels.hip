// gfx950 kernels: request arranging (regroup), plain convolution, max pool, routing head.
// Wavefronts are 64 lanes wide throughout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace coe {
namespace k {

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round to nearest even; NaN becomes a quiet NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = f32_to_bf16(v); }
};

__device__ __forceinline__ float apply_act(float v, int act)
{
    if (act == 1) return v > 0.f ? v : 0.f;
    if (act == 2) return 0.5f * v * erfcf(-v * 0.70710678118654752440f);
    if (act == 3) return v / (1.f + expf(-v));
    return v;
}

// -------------------------------------------------------------------------------------------------------------
// regroup, index part: a stable counting sort of the request indices by expert id
// -------------------------------------------------------------------------------------------------------------
// A workgroup owns a contiguous range of the keys and every wavefront a contiguous eighth of it, so the order inside a
// group is: earlier workgroups, earlier wavefronts, earlier 64-key trips, lower lanes.  Two launches: every workgroup
// writes the histogram of its range; then every workgroup adds up the columns of all histograms for itself (its own
// group starts), counts its wavefronts' keys again and places them.  One launch when a single workgroup holds all keys.
// What bounds it is latency: 0.4 MB of keys are read twice.  The former three launches spent 92 of 103 us in a scan by one
// workgroup that walked 391 histograms of 256 keys one load after the other (100,003 keys, 370 experts); wide ranges
// leave 49 histograms and all workgroups walk them at once with eight loads in flight.  That call: 96.4 -> 12.0 us, launches
// included.
constexpr int kPlaceThreads = 512;
constexpr int kPlaceWaves = kPlaceThreads / kWave;
constexpr int kPlaceRange = 2048;        // keys of a workgroup at least: 256 per wavefront, four trips
constexpr int kPlaceMaxBlocks = 128;     // every workgroup reads every histogram: their number is bounded, ranges grow instead

// Pass 1: histogram of a workgroup's range.
__global__ __launch_bounds__(kPlaceThreads) void regroup_count_kernel(const int32_t* __restrict__ cur, int32_t n, int32_t E,
                                                                      int32_t range, int32_t* __restrict__ blockhist)
{
    extern __shared__ int32_t hist[];
    for (int e = threadIdx.x; e < E; e += kPlaceThreads) hist[e] = 0;
    __syncthreads();
    const uint32_t lo = blockIdx.x * range, hi = min((uint32_t)n, lo + range);     // unsigned: ranges end up to 2^24 beyond n
    for (uint32_t i = lo + threadIdx.x; i < hi; i += kPlaceThreads) {
        const int key = cur[i];
        if (key >= 0 && key < E) atomicAdd(&hist[key], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kPlaceThreads) blockhist[(size_t)blockIdx.x * E + e] = hist[e];
}

// inclusive prefix sum across one wavefront
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        int t = __shfl_up(v, d, kWave);
        if (lane >= d) v += t;
    }
    return v;
}

// Pass 2: group starts (written out by workgroup 0) and stable placement of the workgroup's range.  heads, if not null:
// heads[e] = the first request of group e or -1.  host, if not null: pinned host memory that receives the counts and, behind them,
// the heads.
__global__ __launch_bounds__(kPlaceThreads) void regroup_place_kernel(const int32_t* __restrict__ cur, int32_t n, int32_t E,
                                                                      int32_t range, int32_t key_bits,
                                                                      const int32_t* __restrict__ blockhist,
                                                                      int32_t* __restrict__ cnt, int32_t* __restrict__ off,
                                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                                      int32_t* __restrict__ heads, int32_t* __restrict__ host)
{
    extern __shared__ int32_t lds[];
    __shared__ int32_t wave_tot[kPlaceWaves];
    int32_t* const wcount = lds;                       // [waves][E]: keys of every wavefront, then where its next one goes
    int32_t* const total = lds + kPlaceWaves * E;      // [E]: keys of all workgroups, then the group's start
    int32_t* const before = total + E;                 // [E]: keys of earlier workgroups
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
    const int nblocks = gridDim.x, block = blockIdx.x;
    for (int j = tid; j < (kPlaceWaves + 2) * E; j += kPlaceThreads) lds[j] = 0;
    __syncthreads();

    const int per_wave = range / kPlaceWaves;          // a multiple of the wavefront size
    const uint32_t lo = (uint32_t)block * range + wid * per_wave, hi = min((uint32_t)n, lo + per_wave);
    int32_t* const mine = wcount + wid * E;
    for (uint32_t i = lo + lane; i < hi; i += kWave) {
        const int key = cur[i];
        if (key >= 0 && key < E) atomicAdd(&mine[key], 1);
    }
    if (nblocks > 1) {
        // column sums: as many threads per expert as fit, each over every so many-th histogram
        const int cols = E < kPlaceThreads ? E : kPlaceThreads, parts = kPlaceThreads / cols;
        const int part = tid / cols;
        if (part < parts)
            for (int e = tid % cols; e < E; e += cols) {
                int t = 0, b4 = 0;
#pragma unroll 8
                for (int b = part; b < nblocks; b += parts) {
                    const int v = blockhist[(size_t)b * E + e];
                    t += v;
                    b4 += b < block ? v : 0;
                }
                if (t) atomicAdd(&total[e], t);
                if (b4) atomicAdd(&before[e], b4);
            }
    }
    __syncthreads();
    if (nblocks == 1) {
        for (int e = tid; e < E; e += kPlaceThreads) {
            int t = 0;
#pragma unroll
            for (int w = 0; w < kPlaceWaves; ++w) t += wcount[w * E + e];
            total[e] = t;
        }
        __syncthreads();
    }
    // exclusive scan of the totals: consecutive experts per thread
    const int per = (E + kPlaceThreads - 1) / kPlaceThreads;
    int sum = 0;
    for (int j = 0; j < per; ++j) {
        const int e = tid * per + j;
        if (e < E) sum += total[e];
    }
    const int incl = wave_inclusive_scan(sum);
    if (lane == kWave - 1) wave_tot[wid] = incl;
    __syncthreads();
    int start = incl - sum, all = 0;
#pragma unroll
    for (int w = 0; w < kPlaceWaves; ++w) {
        if (w < wid) start += wave_tot[w];
        all += wave_tot[w];
    }
    for (int j = 0; j < per; ++j) {
        const int e = tid * per + j;
        if (e >= E) break;
        const int t = total[e];
        if (block == 0) {
            cnt[e] = t;
            off[e] = start;
            if (host) host[e] = t;
            if (heads && t == 0) {
                heads[e] = -1;
                if (host) host[E + e] = -1;
            }
        }
        total[e] = start;
        int at = start + before[e];
#pragma unroll
        for (int w = 0; w < kPlaceWaves; ++w) {
            const int c = wcount[w * E + e];
            wcount[w * E + e] = at;
            at += c;
        }
        start += t;
    }
    if (block == 0 && tid == 0) off[E] = all;
    __syncthreads();

    // a wavefront places 64 keys a trip: the lanes with the same key find each other by one ballot per key bit, the lowest
    // of them moves the wavefront's position for that key on
    const unsigned long long lt_mask = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
    for (uint32_t base = lo; base < hi; base += kWave) {
        const uint32_t i = base + lane;
        int key = i < hi ? cur[i] : -1;
        const bool live = key >= 0 && key < E;
        unsigned long long peers = __ballot(live);
        for (int b = 0; b < key_bits; ++b) {
            const bool bit = (key >> b) & 1;
            const unsigned long long set = __ballot(bit);
            peers &= bit ? set : ~set;
        }
        if (live) {
            const int pos = mine[key] + __popcll(peers & lt_mask);
            perm[pos] = i;
            inv[i] = pos;
            if (heads && pos == total[key]) {
                heads[key] = i;
                if (host) host[E + key] = i;
            }
        } else if (i < hi) {
            inv[i] = -1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (live && (peers & lt_mask) == 0) mine[key] += __popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// -------------------------------------------------------------------------------------------------------------
// a submit and a collect in one launch each
// -------------------------------------------------------------------------------------------------------------
// What bounds them is the number of queue entries: each of the copies and fills that they replace is a launch of its own of 3 to 5 us,
// whatever it moves, and a copy to pageable host memory ends in a wait.  Passes, with the counts that
// the regroup leaves in host memory and those that the host knows: one request through a ResNet-18-shaped tree 393 -> 323 us, 29 831 ->
// 753, 256 fp32 requests 1368 -> 1310.
constexpr int kMoveThreads = 256;

// images (vecs 16-byte words, none if they travel by a copy), first experts (null: expert 0), depth 0, path -1, logits 0
__global__ __launch_bounds__(kMoveThreads) void submit_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t vecs,
                                                              const int32_t* __restrict__ first, int32_t* __restrict__ cur,
                                                              int32_t* __restrict__ depth, size_t n, int32_t* __restrict__ path,
                                                              size_t path_words, float* __restrict__ logits, size_t logit_words)
{
    const size_t at = (size_t)blockIdx.x * kMoveThreads + threadIdx.x, step = (size_t)gridDim.x * kMoveThreads;
    for (size_t i = at; i < n; i += step) {
        cur[i] = first ? first[i] : 0;
        depth[i] = 0;
    }
    for (size_t i = at; i < path_words; i += step) path[i] = -1;
    for (size_t i = at; i < logit_words; i += step) logits[i] = 0.f;
    size_t i = at;
    for (; i + 3 * step < vecs; i += 4 * step) {              // four loads in flight
        const uint4 a = src[i], b = src[i + step], c = src[i + 2 * step], d = src[i + 3 * step];
        dst[i] = a; dst[i + step] = b; dst[i + 2 * step] = c; dst[i + 3 * step] = d;
    }
    for (; i < vecs; i += step) dst[i] = src[i];
}

// three arrays of 4-byte words one behind the other, into pinned host memory
__global__ __launch_bounds__(kMoveThreads) void collect_kernel(const uint32_t* __restrict__ a, size_t na, const uint32_t* __restrict__ b,
                                                               size_t nb, const uint32_t* __restrict__ c, size_t nc,
                                                               uint32_t* __restrict__ out)
{
    const size_t step = (size_t)gridDim.x * kMoveThreads;
    for (size_t i = (size_t)blockIdx.x * kMoveThreads + threadIdx.x; i < na + nb + nc; i += step)
        out[i] = i < na ? a[i] : i < na + nb ? b[i - na] : c[i - na - nb];
}

// -------------------------------------------------------------------------------------------------------------
// regroup, activation part: coalesced row gather, 16 bytes per lane
// -------------------------------------------------------------------------------------------------------------
constexpr int kGatherThreads = 256;
template <typename V>
__global__ __launch_bounds__(kGatherThreads) void gather_rows_kernel(const V* __restrict__ src,
                                                                     const int32_t* __restrict__ perm,
                                                                     size_t row_vecs, V* __restrict__ dst)
{
    int row = blockIdx.x;
    const V* s = src + (size_t)perm[row] * row_vecs;
    V* d = dst + (size_t)row * row_vecs;
    for (size_t j = (size_t)blockIdx.y * kGatherThreads + threadIdx.x; j < row_vecs; j += (size_t)gridDim.y * kGatherThreads)
        d[j] = s[j];
}

// -------------------------------------------------------------------------------------------------------------
// plain convolution: one thread per output element, channels fastest
// -------------------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void conv_direct_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                          const float* __restrict__ bias, const T* __restrict__ res,
                                                          T* __restrict__ y, ConvShape s)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)s.N * s.P * s.Q * s.K;
    if (idx >= total) return;
    int k = (int)(idx % s.K);
    size_t m = idx / s.K;
    int q = (int)(m % s.Q);
    int p = (int)((m / s.Q) % s.P);
    int n = (int)(m / ((size_t)s.Q * s.P));
    float acc = 0.f;
    for (int r = 0; r < s.R; ++r) {
        int ih = p * s.stride - s.pad + r;
        if (ih < 0 || ih >= s.H) continue;
        for (int t = 0; t < s.S; ++t) {
            int iw = q * s.stride - s.pad + t;
            if (iw < 0 || iw >= s.W) continue;
            const T* xp = x + (((size_t)n * s.H + ih) * s.W + iw) * s.C;
            const T* wp = w + (((size_t)k * s.R + r) * s.S + t) * s.C;
            for (int c = 0; c < s.C; ++c) acc = fmaf(Elem<T>::load(xp + c), Elem<T>::load(wp + c), acc);
        }
    }
    float v = acc + bias[k];
    if (res) v += Elem<T>::load(res + idx);
    Elem<T>::store(y + idx, apply_act(v, s.act));
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_kernel(const T* __restrict__ x, T* __restrict__ y, int N, int H, int W,
                                                      int C, int R, int S, int stride, int pad, int P, int Q)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)N * P * Q * C;
    if (idx >= total) return;
    int c = (int)(idx % C);
    size_t m = idx / C;
    int q = (int)(m % Q);
    int p = (int)((m / Q) % P);
    int n = (int)(m / ((size_t)Q * P));
    float best = -INFINITY;
    for (int r = 0; r < R; ++r) {
        int ih = p * stride - pad + r;
        if (ih < 0 || ih >= H) continue;
        for (int t = 0; t < S; ++t) {
            int iw = q * stride - pad + t;
            if (iw < 0 || iw >= W) continue;
            best = fmaxf(best, Elem<T>::load(x + (((size_t)n * H + ih) * W + iw) * C + c));
        }
    }
    Elem<T>::store(y + idx, best);
}

// bf16 max pool, 8 channels (16 bytes) per lane.  bf16 order equals the order of the fp32 values, so the max is taken
// on the widened values and the winning pattern is stored unchanged.
__global__ __launch_bounds__(256) void maxpool_bf16x8_kernel(const uint4* __restrict__ x, uint4* __restrict__ y, int N, int H,
                                                             int W, int C8, int R, int S, int stride, int pad, int P, int Q)
{
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)N * P * Q * C8;
    if (idx >= total) return;
    int c8 = (int)(idx % C8);
    size_t m = idx / C8;
    int q = (int)(m % Q);
    int p = (int)((m / Q) % P);
    int n = (int)(m / ((size_t)Q * P));
    float best[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) best[i] = -INFINITY;
    for (int r = 0; r < R; ++r) {
        int ih = p * stride - pad + r;
        if (ih < 0 || ih >= H) continue;
        for (int t = 0; t < S; ++t) {
            int iw = q * stride - pad + t;
            if (iw < 0 || iw >= W) continue;
            uint4 v = x[(((size_t)n * H + ih) * W + iw) * C8 + c8];
            uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                best[2 * i] = fmaxf(best[2 * i], __uint_as_float(wds[i] << 16));
                best[2 * i + 1] = fmaxf(best[2 * i + 1], __uint_as_float(wds[i] & 0xFFFF0000u));
            }
        }
    }
    uint4 o;
    o.x = (__float_as_uint(best[0]) >> 16) | (__float_as_uint(best[1]) & 0xFFFF0000u);
    o.y = (__float_as_uint(best[2]) >> 16) | (__float_as_uint(best[3]) & 0xFFFF0000u);
    o.z = (__float_as_uint(best[4]) >> 16) | (__float_as_uint(best[5]) & 0xFFFF0000u);
    o.w = (__float_as_uint(best[6]) >> 16) | (__float_as_uint(best[7]) & 0xFFFF0000u);
    y[idx] = o;
}

// The same with stride 1 on maps that fit LDS: a workgroup holds CH chunks of 8 channels of one image, takes the maximum along
// rows, then along columns, so a map is read once.  The kernel above reads it R * S times through the caches, which is what bounds its
// long launches; a short launch of this one is bound by what a single workgroup does one after the other (plane_pays).
// us, kernel above / this one: 5x5 on 14 x 14 x 256, 256 images 54 / 29, 64 images 21 / 14, one 8.0 / 11.0; on 20 x 20 x 96, 256 images
// 46 / 26, one 8.0 / 11.1; on 7 x 7 x 512, 256 images 29 / 19, one 7.5 / 5.0; 9x9 on 14 x 14 x 256, 256 images 133 / 41, one 19 / 15.
constexpr int kPlaneThreads = 256;
constexpr size_t kPlaneLds = 64 * 1024;
__device__ __forceinline__ void max_bf16x8(float (&best)[8], const uint4& v)
{
    const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        best[2 * i] = fmaxf(best[2 * i], __uint_as_float(wds[i] << 16));
        best[2 * i + 1] = fmaxf(best[2 * i + 1], __uint_as_float(wds[i] & 0xFFFF0000u));
    }
}
__device__ __forceinline__ uint4 upper_halves(const float (&v)[8])
{
    uint4 o;
    o.x = (__float_as_uint(v[0]) >> 16) | (__float_as_uint(v[1]) & 0xFFFF0000u);
    o.y = (__float_as_uint(v[2]) >> 16) | (__float_as_uint(v[3]) & 0xFFFF0000u);
    o.z = (__float_as_uint(v[4]) >> 16) | (__float_as_uint(v[5]) & 0xFFFF0000u);
    o.w = (__float_as_uint(v[6]) >> 16) | (__float_as_uint(v[7]) & 0xFFFF0000u);
    return o;
}
template <int CH>
__global__ __launch_bounds__(kPlaneThreads) void maxpool_plane_kernel(const uint4* __restrict__ x, uint4* __restrict__ y, int H, int W, int C8,
                                                                      int R, int S, int pad, int P, int Q)
{
    extern __shared__ uint4 plane[];                           // [H][W][CH] | [H][Q][CH]
    uint4* const rows = plane + H * W * CH;
    const int groups = C8 / CH, n = blockIdx.x / groups, c0 = (blockIdx.x % groups) * CH;
    const uint4* const xp = x + (size_t)n * H * W * C8 + c0;
    uint4* const yp = y + (size_t)n * P * Q * C8 + c0;
    for (int i = threadIdx.x; i < H * W * CH; i += kPlaneThreads) plane[i] = xp[(size_t)(i / CH) * C8 + i % CH];
    __syncthreads();
    for (int i = threadIdx.x; i < H * Q * CH; i += kPlaneThreads) {
        const int c = i % CH, q = i / CH % Q, h = i / CH / Q;
        const int lo = max(q - pad, 0), hi = min(q - pad + S, W);
        float best[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
        for (int w = lo; w < hi; ++w) max_bf16x8(best, plane[(h * W + w) * CH + c]);
        rows[i] = upper_halves(best);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < P * Q * CH; i += kPlaneThreads) {
        const int c = i % CH, q = i / CH % Q, p = i / CH / Q;
        const int lo = max(p - pad, 0), hi = min(p - pad + R, H);
        float best[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) best[e] = -INFINITY;
        for (int h = lo; h < hi; ++h) max_bf16x8(best, rows[(h * Q + q) * CH + c]);
        yp[(size_t)(i / CH) * C8 + c] = upper_halves(best);
    }
}

// -------------------------------------------------------------------------------------------------------------
// routing head: global average pool, FC, argmax over the routed classes, successor lookup
// -------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

constexpr int kHeadThreads = 256;

// logits of one request are in LDS: write them out, take the argmax over the routed classes (lowest index wins
// ties), look the successor up, append the expert to the request's path
__device__ __forceinline__ void route_tail(const float* logit, int ncls, int slot, int d, const RouteArgs& r)
{
    for (int j = threadIdx.x; j < r.logits_stride; j += kHeadThreads)
        r.logits[(size_t)slot * r.logits_stride + j] = j < ncls ? logit[j] : 0.f;
    if (threadIdx.x == 0 && r.cur) {
        int nxt = -1;
        if (r.n_route > 0) {
            int best = 0;
            for (int j = 1; j < r.n_route; ++j)
                if (logit[j] > logit[best]) best = j;      // strict: the lowest index wins ties
            nxt = r.succ[best];
        }
        if (d < r.max_stages) r.path[(size_t)slot * r.max_stages + d] = r.expert;
        r.depth[slot] = d + 1;
        r.cur[slot] = nxt;
    }
}

// 16-byte loads in the pooling phase: bf16 tensors whose channel count is a multiple of 8 with C/8 dividing the block
template <typename T> __host__ __device__ inline bool head_vector_path(int C)
{
    return sizeof(T) == 2 && C >= 64 && C % 8 == 0 && kHeadThreads % (C / 8) == 0;
}

// The same for fp32: C a multiple of 4 with C/4 dividing the block.  One 4-byte load at a time kept a workgroup waiting for
// memory: 256 requests of 64 x 64 images with 64 channels, two stages in four launches of 279 us; that pass 2.40 -> 1.43 ms.
template <typename T> __host__ __device__ inline bool head_vector4_path(int C)
{
    return sizeof(T) == 4 && C >= 16 && C % 4 == 0 && kHeadThreads % (C / 4) == 0;
}
// position groups of the pooling phase, whose partial sums meet in LDS
template <typename T> __host__ __device__ inline int head_groups(int C)
{
    if (head_vector_path<T>(C)) return kHeadThreads / (C / 8);
    if (head_vector4_path<T>(C)) return kHeadThreads / (C / 4);
    return C < kHeadThreads ? kHeadThreads / C : 1;
}
// LDS, in floats: feat[C], then the partial sums; the logits after them, on the fp32 path over those of the later position
// groups (nobody reads them any more)
template <typename T> __host__ __device__ inline size_t head_logit_at(int C)
{
    const int before = head_vector4_path<T>(C) ? (C < kHeadThreads ? kHeadThreads / C : 1) : head_groups<T>(C);
    return (size_t)C + (size_t)before * C;
}
template <typename T> size_t head_lds_bytes(int C, int ncls)
{
    const size_t sums = (size_t)C + (size_t)head_groups<T>(C) * C, logits = head_logit_at<T>(C) + (size_t)ncls;
    return sizeof(float) * (sums > logits ? sums : logits);
}

template <typename T>
__global__ __launch_bounds__(kHeadThreads) void head_gap_fc_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                                   const float* __restrict__ b, int HW, int C, int ncls,
                                                                   RouteArgs r, GroupTable gt, GroupRoutes gr, uint32_t off_w,
                                                                   uint32_t off_b)
{
    extern __shared__ float smem[];          // feat[C] | part[groups][C] | logit[ncls]
    int row = blockIdx.x;
    if (gt.n > 0) {
        // grouped launch: this request's group decides the FC weights and the routing rule
        int g = 0;
        while (g + 1 < gt.n && row >= gt.first_row[g + 1]) ++g;
        const char* base = (const char*)gt.weights[g];
        w = (const T*)(base + off_w);
        b = (const float*)(base + off_b);
        r.expert = gr.expert[g];
        r.succ = r.succ + gr.succ_off[g];
        r.n_route = gr.n_route[g];
        if (r.slot) r.slot = r.slot + (gr.slot_off[g] - gt.first_row[g]);
    }
    const T* xp = x + (size_t)row * HW * C;
    const int groups = head_groups<T>(C);
    float* feat = smem;
    float* part = smem + C;
    float* logit = smem + head_logit_at<T>(C);
    // the request's place in the store is on its way during phase 1
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    constexpr int kWaves = kHeadThreads / kWave;
    const int slot = r.slot ? r.slot[row] : row;
    const int depth = threadIdx.x == 0 && r.cur ? r.depth[slot] : 0;
    // and so are the weights of phase 2 where its first round takes all classes: an expert's come from memory (one request through
    // ResNet-18 shapes, 7.1 us a launch without, 6.7 with; weights that are in the cache gain nothing); of 1000 classes they would be a part
    uint4 first_w[4];
    const bool ahead = head_vector_path<T>(C) && ncls <= 4 * kWaves;
    if (ahead) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = wid + u * kWaves;
            first_w[u] = j < ncls && lane < C / 8 ? *(const uint4*)((const uint16_t*)w + (size_t)j * C + lane * 8) : make_uint4(0, 0, 0, 0);
        }
    }
    // phase 1: per-channel sums, lanes run along channels (contiguous in NHWC)
    if (head_vector_path<T>(C)) {
        // bf16, C a multiple of 8 with C/8 dividing the block: 16-byte loads, 8 channels per thread, the positions
        // dealt round-robin to 256 / (C/8) thread groups whose partial sums meet in LDS
        const int cpb = C / 8, G = kHeadThreads / cpb;
        const int chunk = threadIdx.x % cpb, pg = threadIdx.x / cpb;
        // Loads in flight, not their number, bound a workgroup: us a launch, a load at a time / sixteen, 196 positions of 256 channels, one
        // request 8.0 / 6.7, 3136 of 64 channels 18.7 / 10.3, 49 of 2048 channels 30.6 / 26.9.  What is left after whole rounds is loaded only
        // where there is a position (a load for every place, 3136 of 64 channels: 12.1); the others add a zero, which changes no sum.
        constexpr int kFlight = 16;
        const uint16_t* const at = (const uint16_t*)xp + chunk * 8;
        float a8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto add = [&](const uint4& v) {
            const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a8[2 * e] += __uint_as_float(wds[e] << 16);
                a8[2 * e + 1] += __uint_as_float(wds[e] & 0xFFFF0000u);
            }
        };
        int i = pg;
        for (; i + (kFlight - 1) * G < HW; i += kFlight * G) {
            uint4 v[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) v[u] = *(const uint4*)(at + (size_t)(i + u * G) * C);
#pragma unroll
            for (int u = 0; u < kFlight; ++u) add(v[u]);
        }
        auto rest = [&](auto most_c) {
            constexpr int most = decltype(most_c)::value;
            uint4 v[most];
#pragma unroll
            for (int u = 0; u < most; ++u) {
                v[u] = make_uint4(0, 0, 0, 0);
                if (i + u * G < HW) v[u] = *(const uint4*)(at + (size_t)(i + u * G) * C);
            }
#pragma unroll
            for (int u = 0; u < most; ++u) add(v[u]);
        };
        if (HW % (kFlight * G) <= 2 * G) rest(std::integral_constant<int, 2>{});
        else rest(std::integral_constant<int, kFlight - 1>{});
#pragma unroll
        for (int e = 0; e < 8; ++e) part[pg * C + chunk * 8 + e] = a8[e];
        __syncthreads();
        for (int c2 = threadIdx.x; c2 < C; c2 += kHeadThreads) {
            float a = 0.f;
            for (int g2 = 0; g2 < G; ++g2) a += part[g2 * C + c2];
            feat[c2] = a / (float)HW;
        }
    } else if (head_vector4_path<T>(C)) {
        // sixteen 16-byte loads in flight per thread: one workgroup streams a whole image
        constexpr int kFlight = 16;
        const int cpb = C / 4, G = groups;
        const int chunk = threadIdx.x % cpb, pg = threadIdx.x / cpb;
        const float* const at = (const float*)xp + chunk * 4;
        float4 a4 = make_float4(0.f, 0.f, 0.f, 0.f);
        int i = pg;
        for (; i + (kFlight - 1) * G < HW; i += kFlight * G) {
            float4 v[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) v[u] = *(const float4*)(at + (size_t)(i + u * G) * C);
#pragma unroll
            for (int u = 0; u < kFlight; ++u) { a4.x += v[u].x; a4.y += v[u].y; a4.z += v[u].z; a4.w += v[u].w; }
        }
        for (; i < HW; i += G) {
            const float4 v = *(const float4*)(at + (size_t)i * C);
            a4.x += v.x; a4.y += v.y; a4.z += v.z; a4.w += v.w;
        }
        *(float4*)(part + pg * C + chunk * 4) = a4;
        __syncthreads();
        for (int c2 = threadIdx.x; c2 < C; c2 += kHeadThreads) {
            float a = 0.f;
            for (int g2 = 0; g2 < G; ++g2) a += part[g2 * C + c2];
            feat[c2] = a / (float)HW;
        }
    } else if (groups > 1) {
        int g = threadIdx.x / C, c = threadIdx.x % C;
        if (g < groups) {
            float a = 0.f;
            for (int i = g; i < HW; i += groups) a += Elem<T>::load(xp + (size_t)i * C + c);
            part[g * C + c] = a;
        }
        __syncthreads();
        for (int c2 = threadIdx.x; c2 < C; c2 += kHeadThreads) {
            float a = 0.f;
            for (int g2 = 0; g2 < groups; ++g2) a += part[g2 * C + c2];
            feat[c2] = a / (float)HW;
        }
    } else {
        for (int c = threadIdx.x; c < C; c += kHeadThreads) {
            float a = 0.f;
            for (int i = 0; i < HW; ++i) a += Elem<T>::load(xp + (size_t)i * C + c);
            feat[c] = a / (float)HW;
        }
    }
    __syncthreads();
    // phase 2: one wavefront per class, lanes along the feature dimension, wavefront reduction
    if (head_vector_path<T>(C)) {
        // 16-byte weight loads, four classes per wavefront in flight: with one 2-byte load per multiply-add the loop is
        // a chain of ~C/64 * classes/4 global-load latencies per wavefront (200 us for a 2048 x 64 head)
        const uint16_t* wq = (const uint16_t*)w;
        const int cpb = C / 8;
        for (int j0 = wid; j0 < ncls; j0 += 4 * kWaves) {
            float a[4] = {0.f, 0.f, 0.f, 0.f};
            for (int ch = lane; ch < cpb; ch += kWave) {
                uint4 wv[4];
                if (ahead && ch == lane) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) wv[u] = first_w[u];
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = j0 + u * kWaves;
                        wv[u] = j < ncls ? *(const uint4*)(wq + (size_t)j * C + ch * 8) : make_uint4(0, 0, 0, 0);
                    }
                }
                const float4 f0 = *(const float4*)(feat + ch * 8), f1 = *(const float4*)(feat + ch * 8 + 4);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = fmaf(f0.x, __uint_as_float(wv[u].x << 16), a[u]);
                    a[u] = fmaf(f0.y, __uint_as_float(wv[u].x & 0xFFFF0000u), a[u]);
                    a[u] = fmaf(f0.z, __uint_as_float(wv[u].y << 16), a[u]);
                    a[u] = fmaf(f0.w, __uint_as_float(wv[u].y & 0xFFFF0000u), a[u]);
                    a[u] = fmaf(f1.x, __uint_as_float(wv[u].z << 16), a[u]);
                    a[u] = fmaf(f1.y, __uint_as_float(wv[u].z & 0xFFFF0000u), a[u]);
                    a[u] = fmaf(f1.z, __uint_as_float(wv[u].w << 16), a[u]);
                    a[u] = fmaf(f1.w, __uint_as_float(wv[u].w & 0xFFFF0000u), a[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = j0 + u * kWaves;
                const float t = wave_sum(a[u]);
                if (lane == 0 && j < ncls) logit[j] = t + b[j];
            }
        }
    } else {
        for (int j = wid; j < ncls; j += kHeadThreads / kWave) {
            float a = 0.f;
            for (int c = lane; c < C; c += kWave) a = fmaf(feat[c], Elem<T>::load(w + (size_t)j * C + c), a);
            a = wave_sum(a);
            if (lane == 0) logit[j] = a + b[j];
        }
    }
    __syncthreads();
    // phase 3: write logits, pick the route
    route_tail(logit, ncls, slot, depth, r);
}

// class-token head: layer norm of token 0 (rounded to bf16 like every stored activation), FC, routing
__global__ __launch_bounds__(kHeadThreads) void head_cls_kernel(const uint16_t* __restrict__ x, const float* __restrict__ gamma,
                                                                const float* __restrict__ beta, const uint16_t* __restrict__ w,
                                                                const float* __restrict__ b, int T, int D, int ncls, RouteArgs r,
                                                                GroupTable gt, GroupRoutes gr, uint4 off)
{
    extern __shared__ float smem[];          // feat[D] | red[8] | logit[ncls]
    float* feat = smem;
    float* red = smem + D;
    float* logit = red + 8;
    const int row = blockIdx.x;
    if (gt.n > 0) {
        // grouped launch: this request's group decides the weights and the routing rule
        int g = 0;
        while (g + 1 < gt.n && row >= gt.first_row[g + 1]) ++g;
        const char* base = (const char*)gt.weights[g];
        gamma = (const float*)(base + off.x);
        beta = (const float*)(base + off.y);
        w = (const uint16_t*)(base + off.z);
        b = (const float*)(base + off.w);
        r.expert = gr.expert[g];
        r.succ = r.succ + gr.succ_off[g];
        r.n_route = gr.n_route[g];
        if (r.slot) r.slot = r.slot + (gr.slot_off[g] - gt.first_row[g]);
    }
    const uint16_t* xp = x + (size_t)row * T * D;     // token 0
    const int slot = r.slot ? r.slot[row] : row;              // on its way during the work
    const int depth = threadIdx.x == 0 && r.cur ? r.depth[slot] : 0;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    float sum = 0.f;
    for (int c = threadIdx.x; c < D; c += kHeadThreads) { float v = bf16_to_f32(xp[c]); feat[c] = v; sum += v; }
    sum = wave_sum(sum);
    if (lane == 0) red[wid] = sum;
    __syncthreads();
    const float mean = (red[0] + red[1] + red[2] + red[3]) / (float)D;
    float sq = 0.f;
    for (int c = threadIdx.x; c < D; c += kHeadThreads) { float d = feat[c] - mean; sq += d * d; }
    sq = wave_sum(sq);
    if (lane == 0) red[4 + wid] = sq;
    __syncthreads();
    const float rstd = rsqrtf((red[4] + red[5] + red[6] + red[7]) / (float)D + 1e-6f);
    for (int c = threadIdx.x; c < D; c += kHeadThreads)
        feat[c] = bf16_to_f32(f32_to_bf16((feat[c] - mean) * rstd * gamma[c] + beta[c]));
    __syncthreads();
    for (int j = wid; j < ncls; j += kHeadThreads / kWave) {
        float a = 0.f;
        for (int c = lane; c < D; c += kWave) a = fmaf(feat[c], bf16_to_f32(w[(size_t)j * D + c]), a);
        a = wave_sum(a);
        if (lane == 0) logit[j] = a + b[j];
    }
    __syncthreads();
    route_tail(logit, ncls, slot, depth, r);
}

// -------------------------------------------------------------------------------------------------------------
// detector-shaped experts: channel concatenation, nearest-neighbour upsampling, detection read-out
// -------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void concat_kernel(const uint4* __restrict__ a, const uint4* __restrict__ b, uint4* __restrict__ out,
                                                     size_t rows, int A8, int B8)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C8 = A8 + B8;
    if (idx >= rows * C8) return;
    const size_t r = idx / C8;
    const int c = (int)(idx % C8);
    out[idx] = c < A8 ? a[r * A8 + c] : b[r * B8 + (c - A8)];
}

__global__ __launch_bounds__(256) void upsample2_kernel(const uint4* __restrict__ x, uint4* __restrict__ out, int N, int H, int W, int C8)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t total = (size_t)N * 4 * H * W * C8;
    if (idx >= total) return;
    const int c = (int)(idx % C8);
    size_t m = idx / C8;
    const int w = (int)(m % (2 * W)); m /= 2 * W;
    const int h = (int)(m % (2 * H));
    const int n = (int)(m / (2 * H));
    out[idx] = x[(((size_t)n * H + h / 2) * W + w / 2) * C8 + c];
}

__device__ __forceinline__ float sigmoid_f(float v) { return 1.f / (1.f + expf(-v)); }

// one workgroup per request.  A box is box_len = 5 + classes consecutive elements; thread t owns element t % box_len of
// boxes t / box_len, + per_iter, ... (per_iter = boxes the workgroup covers at once), so consecutive threads read consecutive
// elements and a thread's class never changes: it keeps its best score in a register.  The per_iter partial maxima of a
// class meet in LDS at the end.  Scores are products of two sigmoids, hence positive, and the maximum does not depend on
// the order it is taken in.
constexpr int kDetMaxClasses = 251;            // box_len <= kHeadThreads
__global__ __launch_bounds__(kHeadThreads) void head_det_kernel(const uint16_t* __restrict__ m0, int hw0, const uint16_t* __restrict__ m1,
                                                                int hw1, int anchors, int ncls, RouteArgs r)
{
    __shared__ float part[kHeadThreads];
    __shared__ float logit[kHeadThreads];
    const int row = blockIdx.x;
    const int slot = r.slot ? r.slot[row] : row;              // on its way during the work
    const int depth = threadIdx.x == 0 && r.cur ? r.depth[slot] : 0;
    const int box_len = 5 + ncls, stride = anchors * box_len;
    const int per_iter = kHeadThreads / box_len;
    const int j = threadIdx.x % box_len, b0 = threadIdx.x / box_len;
    float best = 0.f;
    if (b0 < per_iter && j >= 5) {
        for (int map = 0; map < 2; ++map) {
            const uint16_t* mp = map == 0 ? m0 : m1;
            const int hw = map == 0 ? hw0 : hw1;
            if (!mp) continue;
            const uint16_t* base = mp + (size_t)row * hw * stride;
            const int nbox = hw * anchors;                           // boxes of one position are consecutive
            // four boxes per trip: eight loads in flight per thread (a launch may hold only a few workgroups per compute unit)
            int bx = b0;
            for (; bx + 3 * per_iter < nbox; bx += 4 * per_iter) {
                uint16_t o[4], v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint16_t* box = base + (size_t)(bx + u * per_iter) * box_len;
                    o[u] = box[4];
                    v[u] = box[j];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) best = fmaxf(best, sigmoid_f(bf16_to_f32(o[u])) * sigmoid_f(bf16_to_f32(v[u])));
            }
            for (; bx < nbox; bx += per_iter) {
                const uint16_t* box = base + (size_t)bx * box_len;
                best = fmaxf(best, sigmoid_f(bf16_to_f32(box[4])) * sigmoid_f(bf16_to_f32(box[j])));
            }
        }
    }
    part[threadIdx.x] = best;
    __syncthreads();
    for (int c = threadIdx.x; c < ncls; c += kHeadThreads) {
        float m = 0.f;
        for (int b = 0; b < per_iter; ++b) m = fmaxf(m, part[b * box_len + 5 + c]);
        logit[c] = m;
    }
    __syncthreads();
    route_tail(logit, ncls, slot, depth, r);
}

}  // namespace

// -------------------------------------------------------------------------------------------------------------
// launchers
// -------------------------------------------------------------------------------------------------------------
hipError_t regroup_index(const int32_t* cur, int32_t n, int32_t E, int32_t* cnt, int32_t* off, int32_t* perm,
                         int32_t* inv, int32_t* blockhist, int32_t* heads, int32_t* host, hipStream_t stream)
{
    if (n < 0 || E <= 0 || E > kRegroupMaxExperts) return hipErrorInvalidValue;
    const int32_t share = (int32_t)(((long long)n + kPlaceMaxBlocks - 1) / kPlaceMaxBlocks);
    const int32_t range = share <= kPlaceRange ? kPlaceRange : (share + kPlaceThreads - 1) / kPlaceThreads * kPlaceThreads;
    const int32_t nblocks = n <= range ? 1 : (int32_t)(((long long)n + range - 1) / range);
    int32_t key_bits = 0;
    while ((1 << key_bits) < E) ++key_bits;
    if (nblocks > 1)
        hipLaunchKernelGGL(regroup_count_kernel, dim3(nblocks), dim3(kPlaceThreads), sizeof(int32_t) * E, stream, cur, n, E, range,
                           blockhist);
    const size_t lds = sizeof(int32_t) * (size_t)E * (kPlaceWaves + 2);
    static const hipError_t configured = hipFuncSetAttribute((const void*)regroup_place_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                             (int)(sizeof(int32_t) * kRegroupMaxExperts * (kPlaceWaves + 2)));
    if (configured != hipSuccess) return configured;
    hipLaunchKernelGGL(regroup_place_kernel, dim3(nblocks), dim3(kPlaceThreads), lds, stream, cur, n, E, range, key_bits, blockhist,
                       cnt, off, perm, inv, heads, host);
    return hipGetLastError();
}

// -------------------------------------------------------------------------------------------------------------
// regroup for callers that cannot allocate: the per-workgroup histograms live in a static device array instead of a
// buffer the caller or a context owns.  Every GPU the library runs on holds its own copy of the array (4 MiB) until the
// process ends; in host code the array's name is only a handle for hipGetSymbolAddress, the address a kernel can use is
// looked up once per device and kept.
// -------------------------------------------------------------------------------------------------------------
static __device__ __align__(256) int32_t scratch[kRegroupStaticInts];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
int32_t* g_scratch_ptr[kMaxDevices] = {nullptr};
}  // namespace

hipError_t regroup_index_static(const int32_t* cur, int32_t n, int32_t E, int32_t* cnt, int32_t* off, int32_t* perm,
                                int32_t* inv, hipStream_t stream)
{
    if (n < 0 || E <= 0 || E > kRegroupMaxExperts) return hipErrorInvalidValue;
    const long long nblocks = ((long long)n + kRegroupTile - 1) / kRegroupTile;
    if (nblocks * E > (long long)kRegroupStaticInts) return hipErrorInvalidValue;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int32_t* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));      // this device's copy of the array
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            g_scratch_ptr[dev] = (int32_t*)p;
        }
        ptr = g_scratch_ptr[dev];
    }
    // every histogram entry the placement reads is written by the count kernel of the same call: nothing has to start at zero
    return regroup_index(cur, n, E, cnt, off, perm, inv, ptr, nullptr, nullptr, stream);
}

hipError_t submit_store(const void* src, void* dst, size_t bytes, const int32_t* first, int32_t* cur, int32_t* depth, size_t n,
                        int32_t* path, size_t path_words, float* logits, size_t logit_words, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    if (bytes % 16 || (bytes && (((uintptr_t)src | (uintptr_t)dst) & 15))) return hipErrorInvalidValue;
    const size_t words = std::max(std::max(bytes / 16, n), std::max(path_words, logit_words));
    const size_t blocks = std::min<size_t>((words + kMoveThreads - 1) / kMoveThreads, 2048);
    hipLaunchKernelGGL(submit_kernel, dim3((unsigned)blocks), dim3(kMoveThreads), 0, stream, (const uint4*)src, (uint4*)dst, bytes / 16,
                       first, cur, depth, n, path, path_words, logits, logit_words);
    return hipGetLastError();
}

hipError_t collect_words(const void* a, size_t na, const void* b, size_t nb, const void* c, size_t nc, void* out, hipStream_t stream)
{
    const size_t words = na + nb + nc;
    if (words == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((words + kMoveThreads - 1) / kMoveThreads, 1024);
    hipLaunchKernelGGL(collect_kernel, dim3((unsigned)blocks), dim3(kMoveThreads), 0, stream, (const uint32_t*)a, na, (const uint32_t*)b, nb,
                       (const uint32_t*)c, nc, (uint32_t*)out);
    return hipGetLastError();
}

hipError_t gather_rows(const void* src, const int32_t* perm, int32_t n_rows, size_t row_bytes, void* dst,
                       hipStream_t stream)
{
    if (n_rows <= 0) return hipSuccess;
    if (row_bytes % 4) return hipErrorInvalidValue;
    if (row_bytes % 16 == 0) {
        size_t vecs = row_bytes / 16;
        int gy = (int)((vecs + kGatherThreads * 8 - 1) / (kGatherThreads * 8));
        if (gy < 1) gy = 1;
        if (gy > 64) gy = 64;
        hipLaunchKernelGGL(gather_rows_kernel<uint4>, dim3(n_rows, gy), dim3(kGatherThreads), 0, stream,
                           (const uint4*)src, perm, vecs, (uint4*)dst);
    } else {
        size_t vecs = row_bytes / 4;
        int gy = (int)((vecs + kGatherThreads * 8 - 1) / (kGatherThreads * 8));
        if (gy < 1) gy = 1;
        if (gy > 64) gy = 64;
        hipLaunchKernelGGL(gather_rows_kernel<uint32_t>, dim3(n_rows, gy), dim3(kGatherThreads), 0, stream,
                           (const uint32_t*)src, perm, vecs, (uint32_t*)dst);
    }
    return hipGetLastError();
}

bool all_finite(const float* v, size_t n)
{
    uint32_t largest = 0;                     // exponent bits
    for (size_t i = 0; i < n; ++i) {
        uint32_t bits;
        std::memcpy(&bits, v + i, sizeof bits);
        largest = std::max(largest, bits & 0x7F800000u);
    }
    return largest != 0x7F800000u;
}

hipError_t conv_direct(int dtype, const void* x, const void* w, const float* bias, const void* res, void* y,
                       const ConvShape& s, bool finite_filters, hipStream_t stream)
{
    size_t total = (size_t)s.N * s.P * s.Q * s.K;
    if (total == 0) return hipSuccess;
    if (dtype == 0 && finite_filters && conv_f32_supported(s)) return conv_f32(x, w, bias, res, y, s, stream);
    size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (dtype == 1)
        hipLaunchKernelGGL(conv_direct_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint16_t*)x,
                           (const uint16_t*)w, bias, (const uint16_t*)res, (uint16_t*)y, s);
    else
        hipLaunchKernelGGL(conv_direct_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, (const float*)x,
                           (const float*)w, bias, (const float*)res, (float*)y, s);
    return hipGetLastError();
}

// Both kernels' times in us, fitted to launches of 1 to 1024 images with 5x5 to 13x13 windows on maps of 4 x 4 to 22 x 22: what a launch
// of any size takes, and what each 16 bytes of its output (`vecs` in all) add.  A workgroup of the plane kernel goes over its
// CH chunks 256 at a time, three times.  Below 5x5 the kernel for all pools is taken throughout (3x3 on 14 x 14 x 64, 64 images: 9.6, plane 11.1).
static bool plane_pays(size_t vecs, int32_t H, int32_t W, int32_t R, int32_t S, int ch)
{
    if (R * S < 25) return false;
    const double r = std::min(R, H), s = std::min(S, W), turns = (double)H * W * ch / kPlaneThreads;
    const double plane = 2.5 + turns * (0.4 + 0.095 * (r + s)) + (double)vecs * (6.0 + 0.8 * (r + s)) * 1e-6;
    const double general = 2.6 + 0.21 * r * s + (double)vecs * 1.15 * r * s * 1e-6;
    return plane <= general;
}

hipError_t maxpool(int dtype, const void* x, void* y, int32_t N, int32_t H, int32_t W, int32_t C, int32_t R, int32_t S,
                   int32_t stride, int32_t pad, int32_t P, int32_t Q, hipStream_t stream)
{
    size_t total = (size_t)N * P * Q * C;
    if (total == 0) return hipSuccess;
    if (dtype == 1 && C % 32 == 0 && stride == 1) {
        // eight chunks of 8 channels are whole lines; four where eight do not fit
        const size_t chunk = ((size_t)H * W + (size_t)H * Q) * sizeof(uint4);
        const int ch = C % 64 == 0 && 8 * chunk <= kPlaneLds ? 8 : 4 * chunk <= kPlaneLds ? 4 : 0;
        const size_t blocks = ch ? (size_t)N * (C / 8 / ch) : 0;
        if (ch && blocks <= 0x7FFFFFFFull && plane_pays(total / 8, H, W, R, S, ch)) {
            if (ch == 8)
                hipLaunchKernelGGL(maxpool_plane_kernel<8>, dim3((unsigned)blocks), dim3(kPlaneThreads), 8 * chunk, stream, (const uint4*)x,
                                   (uint4*)y, H, W, C / 8, R, S, pad, P, Q);
            else
                hipLaunchKernelGGL(maxpool_plane_kernel<4>, dim3((unsigned)blocks), dim3(kPlaneThreads), 4 * chunk, stream, (const uint4*)x,
                                   (uint4*)y, H, W, C / 8, R, S, pad, P, Q);
            return hipGetLastError();
        }
    }
    if (dtype == 1 && C % 8 == 0) {
        size_t blocks8 = (total / 8 + 255) / 256;
        if (blocks8 > 0x7FFFFFFFull) return hipErrorInvalidValue;
        hipLaunchKernelGGL(maxpool_bf16x8_kernel, dim3((unsigned)blocks8), dim3(256), 0, stream, (const uint4*)x, (uint4*)y, N,
                           H, W, C / 8, R, S, stride, pad, P, Q);
        return hipGetLastError();
    }
    size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (dtype == 1)
        hipLaunchKernelGGL(maxpool_kernel<uint16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint16_t*)x,
                           (uint16_t*)y, N, H, W, C, R, S, stride, pad, P, Q);
    else
        hipLaunchKernelGGL(maxpool_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, (const float*)x, (float*)y,
                           N, H, W, C, R, S, stride, pad, P, Q);
    return hipGetLastError();
}

hipError_t head_gap_fc(int dtype, const void* x, const void* w, const float* b, int32_t N, int32_t HW, int32_t C,
                       int32_t ncls, const RouteArgs& r, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    const size_t smem = dtype == 1 ? head_lds_bytes<uint16_t>(C, ncls) : head_lds_bytes<float>(C, ncls);
    if (smem > 60 * 1024) return hipErrorInvalidValue;
    const GroupTable gt{};
    const GroupRoutes gr{};
    if (dtype == 1)
        hipLaunchKernelGGL(head_gap_fc_kernel<uint16_t>, dim3(N), dim3(kHeadThreads), smem, stream, (const uint16_t*)x,
                           (const uint16_t*)w, b, HW, C, ncls, r, gt, gr, 0u, 0u);
    else
        hipLaunchKernelGGL(head_gap_fc_kernel<float>, dim3(N), dim3(kHeadThreads), smem, stream, (const float*)x,
                           (const float*)w, b, HW, C, ncls, r, gt, gr, 0u, 0u);
    return hipGetLastError();
}

hipError_t head_gap_fc_grouped(int dtype, const void* x, const GroupTable& groups, size_t off_w, size_t off_b, int32_t N,
                               int32_t HW, int32_t C, int32_t ncls, const RouteArgs& r, const GroupRoutes& routes,
                               hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    if (groups.n <= 0 || groups.n > kMaxGroups || groups.first_row[0] != 0 || groups.first_row[groups.n] != N ||
        off_w > 0x7FFFFFFFull || off_b > 0x7FFFFFFFull)
        return hipErrorInvalidValue;
    const size_t smem = dtype == 1 ? head_lds_bytes<uint16_t>(C, ncls) : head_lds_bytes<float>(C, ncls);
    if (smem > 60 * 1024) return hipErrorInvalidValue;
    if (dtype == 1)
        hipLaunchKernelGGL(head_gap_fc_kernel<uint16_t>, dim3(N), dim3(kHeadThreads), smem, stream, (const uint16_t*)x,
                           (const uint16_t*)nullptr, (const float*)nullptr, HW, C, ncls, r, groups, routes, (uint32_t)off_w,
                           (uint32_t)off_b);
    else
        hipLaunchKernelGGL(head_gap_fc_kernel<float>, dim3(N), dim3(kHeadThreads), smem, stream, (const float*)x,
                           (const float*)nullptr, (const float*)nullptr, HW, C, ncls, r, groups, routes, (uint32_t)off_w,
                           (uint32_t)off_b);
    return hipGetLastError();
}

hipError_t concat_channels(const void* a, const void* b, void* out, int64_t rows, int32_t Ca, int32_t Cb, hipStream_t stream)
{
    if (Ca <= 0 || Cb <= 0 || Ca % 8 || Cb % 8 || rows < 0) return hipErrorInvalidValue;
    const size_t total = (size_t)rows * ((Ca + Cb) / 8);
    if (total == 0) return hipSuccess;
    const size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(concat_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4*)a, (const uint4*)b, (uint4*)out,
                       (size_t)rows, Ca / 8, Cb / 8);
    return hipGetLastError();
}

hipError_t upsample2(const void* x, void* out, int32_t N, int32_t H, int32_t W, int32_t C, hipStream_t stream)
{
    if (C <= 0 || C % 8 || H <= 0 || W <= 0 || N < 0) return hipErrorInvalidValue;
    const size_t total = (size_t)N * 4 * H * W * (C / 8);
    if (total == 0) return hipSuccess;
    const size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(upsample2_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4*)x, (uint4*)out, N, H, W, C / 8);
    return hipGetLastError();
}

hipError_t head_det(const void* m0, int32_t hw0, const void* m1, int32_t hw1, int32_t N, int32_t anchors, int32_t ncls,
                    const RouteArgs& r, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    if (!m0 || hw0 <= 0 || anchors <= 0 || ncls <= 0 || ncls > kDetMaxClasses || (m1 && hw1 <= 0)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(head_det_kernel, dim3(N), dim3(kHeadThreads), 0, stream, (const uint16_t*)m0, hw0, (const uint16_t*)m1, hw1,
                       anchors, ncls, r);
    return hipGetLastError();
}

hipError_t head_cls(const void* x, const float* gamma, const float* beta, const void* w, const float* b, int32_t N, int32_t T,
                    int32_t D, int32_t ncls, const RouteArgs& r, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    size_t smem = sizeof(float) * ((size_t)D + 8 + (size_t)ncls);
    if (smem > 60 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(head_cls_kernel, dim3(N), dim3(kHeadThreads), smem, stream, (const uint16_t*)x, gamma, beta,
                       (const uint16_t*)w, b, T, D, ncls, r, GroupTable{}, GroupRoutes{}, make_uint4(0, 0, 0, 0));
    return hipGetLastError();
}

hipError_t head_cls_grouped(const void* x, const GroupTable& groups, const size_t off[4], int32_t N, int32_t T, int32_t D, int32_t ncls,
                            const RouteArgs& r, const GroupRoutes& routes, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    if (groups.n <= 0 || groups.n > kMaxGroups || groups.first_row[0] != 0 || groups.first_row[groups.n] != N) return hipErrorInvalidValue;
    for (int i = 0; i < 4; ++i)
        if (off[i] > 0x7FFFFFFFull) return hipErrorInvalidValue;
    size_t smem = sizeof(float) * ((size_t)D + 8 + (size_t)ncls);
    if (smem > 60 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(head_cls_kernel, dim3(N), dim3(kHeadThreads), smem, stream, (const uint16_t*)x, (const float*)nullptr,
                       (const float*)nullptr, (const uint16_t*)nullptr, (const float*)nullptr, T, D, ncls, r, groups, routes,
                       make_uint4((uint32_t)off[0], (uint32_t)off[1], (uint32_t)off[2], (uint32_t)off[3]));
    return hipGetLastError();
}

}  // namespace k
}  // namespace coe
