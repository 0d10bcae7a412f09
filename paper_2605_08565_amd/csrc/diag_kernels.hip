// Diagnostics of the paper's appendix: the clipping-only part of the block SSE ("Clipping only
// MSE" figure) and the histograms of quantised entries and of chosen scales.  Both read what
// mxq_quantize wrote; neither is on the hot path.
#include "mxq_device.hpp"
#include "mxq_launch.hpp"

namespace mxq {

// A lane's 8 consecutive elements and the scale bytes of their blocks, as loaded.
template <int DT, int B>
struct ClipChunk {
    u32x4 a, b;                                     // b: fp32 only
    uint32_t sb;                                    // block k's byte in bits 8k .. 8k + 7
};

// `c` counts complete chunks.
template <int DT, int B>
__device__ __forceinline__ ClipChunk<DT, B> load_clip(const void* __restrict__ x, const uint8_t* __restrict__ scales, int64_t c)
{
    ClipChunk<DT, B> r{};
    const u32x4* xv = static_cast<const u32x4*>(x);
    if constexpr (DT == kBF16) {
        r.a = xv[c];
    } else {
        r.a = xv[2 * c];
        r.b = xv[2 * c + 1];
    }
    if constexpr (B == 2) r.sb = reinterpret_cast<const uint32_t*>(scales)[c];
    else if constexpr (B == 4) r.sb = reinterpret_cast<const uint16_t*>(scales)[c];
    else r.sb = scales[c / (B / 8)];
    return r;
}

// Clipping-only SSEs of the lane's blocks.  An element clips when fl32(|v| / S) > 6, which for the
// short significands of S is the same as |v| > 6 * S (6 * S is exact); its residual is
// v - (+-6) * S, one FMA because the product is exact.
template <int B>
__device__ __forceinline__ void clip_sums(float (&v)[8], uint32_t sb, int fmt, float T, float (&sse)[4])
{
    constexpr int NBLK = (B < 8) ? 8 / B : 1;
    constexpr int EPB = (B < 8) ? B : 8;
    if (T != 1.0f) {                                // uniform
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = v[i] / T;
    }
    float sq[8];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        const float S = scale_byte_value(fmt, (sb >> (8 * k)) & 0xFFu);
        const float lim = 6.0f * S;
#pragma unroll
        for (int i = 0; i < EPB; ++i) {
            const int j = k * EPB + i;
            const float q = u2f(0x40C00000u | (f2u(v[j]) & 0x80000000u));      // +-6
            const float e = __builtin_fmaf(-q, S, v[j]);
            const float s = e * e;
            sq[j] = (__builtin_fabsf(v[j]) > lim && S > 0.0f) ? s : 0.0f;
        }
    }
    block_sse<B>(sq, sse);
}

template <int DT, int B>
__device__ __forceinline__ void store_clip(const ClipChunk<DT, B>& r, int64_t c, int fmt, float T, float* __restrict__ out)
{
    constexpr int LANES = (B < 8) ? 1 : B / 8;
    float v[8], sse[4];
    if constexpr (DT == kBF16) {
        v[0] = u2f(r.a.x << 16); v[1] = u2f(r.a.x & 0xFFFF0000u);
        v[2] = u2f(r.a.y << 16); v[3] = u2f(r.a.y & 0xFFFF0000u);
        v[4] = u2f(r.a.z << 16); v[5] = u2f(r.a.z & 0xFFFF0000u);
        v[6] = u2f(r.a.w << 16); v[7] = u2f(r.a.w & 0xFFFF0000u);
    } else {
        v[0] = u2f(r.a.x); v[1] = u2f(r.a.y); v[2] = u2f(r.a.z); v[3] = u2f(r.a.w);
        v[4] = u2f(r.b.x); v[5] = u2f(r.b.y); v[6] = u2f(r.b.z); v[7] = u2f(r.b.w);
    }
    clip_sums<B>(v, r.sb, fmt, T, sse);
    if constexpr (B == 2) reinterpret_cast<f32x4*>(out)[c] = f32x4{sse[0], sse[1], sse[2], sse[3]};
    else if constexpr (B == 4) reinterpret_cast<f32x2*>(out)[c] = f32x2{sse[0], sse[1]};
    else out[c / LANES] = sse[0];                   // the same value from every lane of the block
}

// n not a multiple of 8 (b = 2 or 4): the last elements, by one lane.
template <int DT, int B>
__device__ __forceinline__ void clip_tail(const void* __restrict__ x, const uint8_t* __restrict__ scales, int64_t n, int fmt, float T,
                                          float* __restrict__ out)
{
    const int64_t first = n >> 3 << 3;
    const int count = (int)(n - first);
    if (count == 0) return;
    float v[8], sse[4];
    load_partial<DT>(x, first, count, v);
    uint32_t sb = 0u;
    for (int k = 0; k < count / B; ++k) sb |= (uint32_t)scales[first / B + k] << (8 * k);
    clip_sums<B>(v, sb, fmt, T, sse);
    for (int k = 0; k < count / B; ++k) out[first / B + k] = sse[k];
}

// One lane = 8 consecutive elements; a workgroup takes ITEMS times 256 chunks and ends, all its loads first (ITEMS > 0), or
// goes through the tensor with the next chunk's loads under way (ITEMS = 0).
template <int DT, int B, int ITEMS>
__global__ void __launch_bounds__(kThreads)
clip_sse_kernel(const void* __restrict__ x, const uint8_t* __restrict__ scales, int64_t n, int fmt,
                float T, float* __restrict__ out)
{
    const int64_t n_full = n >> 3;
    if constexpr (ITEMS > 0) {
        const int64_t c0 = (int64_t)blockIdx.x * (kThreads * ITEMS) + threadIdx.x;
        ClipChunk<DT, B> r[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) r[i] = load_clip<DT, B>(x, scales, min(c0 + i * kThreads, n_full - 1));
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (c0 + i * kThreads < n_full) store_clip<DT, B>(r[i], c0 + i * kThreads, fmt, T, out);
    } else {
        const int64_t stride = (int64_t)gridDim.x * kThreads;
        int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
        if (c - threadIdx.x < n_full) {                              // uniform
            ClipChunk<DT, B> r = load_clip<DT, B>(x, scales, min(c, n_full - 1));
            for (; c - threadIdx.x < n_full; c += stride) {          // uniform
                const ClipChunk<DT, B> now = r;
                if (c - threadIdx.x + stride < n_full) r = load_clip<DT, B>(x, scales, min(c + stride, n_full - 1));
                if (c < n_full) store_clip<DT, B>(now, c, fmt, T, out);
            }
        }
    }
    if constexpr (B < 8) {
        if (blockIdx.x == 0 && threadIdx.x == 0) clip_tail<DT, B>(x, scales, n, fmt, T, out);
    }
}

// Three chunks per lane all at once from 33.5 M elements on, the loop below.  (Ordinary loads: what the quantise pass left in
// the caches is read there.)  Loop without the next chunk under way -> as it is, three inputs in turn, b = 16: bf16 4096 x 4096
// 9.2 -> 8.1 us, 4096 x 14336 29.7 -> 26.9, 8192 x 4096 b = 8 16.5 -> 15.4, 4096 x 4096 b = 2 14.0 -> 13.4; fp32 2048 x 4096 7.5 -> 7.4, 8192 x
// 4096 b = 32 26.7 -> 26.2.  Non-temporal loads: 8.2, 25.9, 16.4, 15.3; 8.6, 27.7.  Four chunks from 4096 slices on: 4096 x 4096 8.9.
constexpr int kClipItems = 3;
constexpr int64_t kClipFrom = 16384 * kThreads, kClipMost = 1 << 24;   // chunks, workgroups

template <int DT>
static void launch_clip_dt(const void* x, const uint8_t* scales, int64_t n, int block, int fmt, float T,
                           float* out, hipStream_t stream, unsigned grid, bool large)
{
#define MXQ_CLIP(BB)                                                                                  \
    hipLaunchKernelGGL((large ? clip_sse_kernel<DT, BB, kClipItems> : clip_sse_kernel<DT, BB, 0>), dim3(grid), dim3(kThreads), 0, stream, x, scales, n, fmt, T, out)
    switch (block) {
        case 2: MXQ_CLIP(2); break;
        case 4: MXQ_CLIP(4); break;
        case 8: MXQ_CLIP(8); break;
        case 16: MXQ_CLIP(16); break;
        case 32: MXQ_CLIP(32); break;
        case 64: MXQ_CLIP(64); break;
        default: MXQ_CLIP(128); break;
    }
#undef MXQ_CLIP
}

hipError_t launch_clip_sse(const void* x, const uint8_t* scales, int64_t n, int dtype, int block,
                           int scale_fmt, float T, float* out, hipStream_t stream)
{
    const int64_t chunks = n / 8, tile = (int64_t)kThreads * kClipItems;
    const bool large = chunks >= kClipFrom && chunks / tile < kClipMost;
    const unsigned grid = large ? (unsigned)((chunks + tile - 1) / tile) : (unsigned)stream_grid(chunks);
    if (dtype == kBF16) launch_clip_dt<kBF16>(x, scales, n, block, scale_fmt, T, out, stream, grid, large);
    else launch_clip_dt<kF32>(x, scales, n, block, scale_fmt, T, out, stream, grid, large);
    return hipGetLastError();
}

// Histograms.  Both arrays are read with 128-bit loads.
//
// Element magnitudes: the low three bits of the 32 nibbles in a 128-bit vector are transposed
// into three 32-bit planes (plane p holds bit p of every nibble: the four dwords' bit-p masks
// 0x11111111 << p are shifted to interleave), and each of the 8 magnitudes is one boolean
// function of the three planes followed by a population count that adds into a per-lane
// register counter: about 40 vector instructions per 32 elements.
//
// Scale bytes: a per-workgroup LDS histogram with one copy per lane of a wavefront (64 copies,
// word [code][lane]: 64 KiB), so that the lanes of one LDS atomic never meet on a word, however
// popular a code is, and fall on the banks like any 64-lane access.
//
// Codes and scales are counted by different workgroups of one launch, so that neither waits for the other's clearing,
// counting and closing.  Partial results meet in 64-bit atomics on the caller's arrays, which a small kernel clears
// first; where one workgroup does for an array it stores its counts, and where one does for each there is no clearing.
// What bounds it up to some 10 M elements is the chain of a launch, a load, the counting and the closing atomics, which come to
// one address at 5 to 10 ns each: so a workgroup takes at least 64 KiB of codes or 32 KiB of scales.  One workgroup after the
// other for both arrays, 256 of them -> as it is (128 / 16, 32 / 8 KiB): 4096 x 4096 b = 16 10.7 -> 8.8 us (9.9, 10.0), b = 4 11.2 -> 9.0
// (11.9, 10.6), b = 2 12.3 -> 10.3 (12.8, 11.4); 1024 x 1024 b = 16 8.0 -> 7.2 (8.7, 6.7); 64 x 1024 7.6 -> 4.9; 4096 x 14336 b = 16 14.0
// -> 13.1 (13.4, 13.6).  The bytes before the first 16-byte boundary and those after the last complete vector are
// counted serially by one thread.
__global__ void hist_clear_kernel(unsigned long long* elem_hist, unsigned long long* scale_hist)
{
    const uint32_t t = threadIdx.x;
    if (t < 8u) elem_hist[t] = 0ull;
    scale_hist[t] = 0ull;
}

constexpr int kHistThreads = 1024;
constexpr int kHistCopies = 64;
constexpr int64_t kHistCodes = 64 << 10, kHistScales = 32 << 10;       // bytes a workgroup takes at least
constexpr int64_t kHistMaxGrid = 256;                                  // for each array
static_assert(kHistThreads == 4 * 256 && kHistCopies == 64, "the closing reduction maps four threads to a code");

// cnt[k] += number of nibbles of the four dwords whose low three bits equal k
__device__ __forceinline__ void count_magnitudes(const u32x4 w, uint32_t (&cnt)[8])
{
    constexpr uint32_t M0 = 0x11111111u, M1 = 0x22222222u, M2 = 0x44444444u;
    const uint32_t p0 = (w.x & M0) | ((w.y & M0) << 1) | ((w.z & M0) << 2) | ((w.w & M0) << 3);
    const uint32_t p1 = ((w.x & M1) >> 1) | (w.y & M1) | ((w.z & M1) << 1) | ((w.w & M1) << 2);
    const uint32_t p2 = ((w.x & M2) >> 2) | ((w.y & M2) >> 1) | (w.z & M2) | ((w.w & M2) << 1);
    cnt[0] += (uint32_t)__builtin_popcount(~p2 & ~p1 & ~p0);
    cnt[1] += (uint32_t)__builtin_popcount(~p2 & ~p1 & p0);
    cnt[2] += (uint32_t)__builtin_popcount(~p2 & p1 & ~p0);
    cnt[3] += (uint32_t)__builtin_popcount(~p2 & p1 & p0);
    cnt[4] += (uint32_t)__builtin_popcount(p2 & ~p1 & ~p0);
    cnt[5] += (uint32_t)__builtin_popcount(p2 & ~p1 & p0);
    cnt[6] += (uint32_t)__builtin_popcount(p2 & p1 & ~p0);
    cnt[7] += (uint32_t)__builtin_popcount(p2 & p1 & p0);
}

// An array of bytes: `head` bytes, `vec` aligned 16-byte vectors, the rest.
struct ByteArray {
    const uint8_t* bytes;
    int64_t count, head, vec;
    __device__ __forceinline__ ByteArray(const uint8_t* p, int64_t n) : bytes(p), count(n)
    {
        head = min(n, (int64_t)((16u - (uint32_t)(reinterpret_cast<uintptr_t>(p) & 15u)) & 15u));
        vec = (n - head) >> 4;
    }
    __device__ __forceinline__ const u32x4* vectors() const { return reinterpret_cast<const u32x4*>(bytes + head); }
    template <class F>
    __device__ __forceinline__ void outside(F f) const              // the bytes outside the vectors
    {
        for (int64_t b = 0; b < head; ++b) f(bytes[b]);
        for (int64_t b = head + (vec << 4); b < count; ++b) f(bytes[b]);
    }
};

// Workgroup `group` of `groups` that count the scales.
__device__ __forceinline__ void count_scales(const ByteArray a, uint32_t group, uint32_t groups, uint32_t* sh_scale,
                                             unsigned long long* __restrict__ scale_hist)
{
    const u32x4* sv = a.vectors();
    const int64_t stride = (int64_t)groups * kHistThreads, t0 = (int64_t)group * kHistThreads + threadIdx.x;
    u32x4 r[2] = {};
    if (a.vec > 0) {                                                 // in flight while the LDS is cleared
#pragma unroll
        for (int u = 0; u < 2; ++u) r[u] = __builtin_nontemporal_load(sv + min(t0 + u * stride, a.vec - 1));
    }
    for (uint32_t i = threadIdx.x; i < (uint32_t)(kHistCopies * 64); i += kHistThreads) reinterpret_cast<u32x4*>(sh_scale)[i] = u32x4{};
    __syncthreads();

    uint32_t* mine = sh_scale + (threadIdx.x & (kHistCopies - 1));        // word of code c: mine[c * 64]
    for (int64_t i = t0; i < a.vec; i += 2 * stride) {               // two loads in flight per lane
        if (i != t0) {
#pragma unroll
            for (int u = 0; u < 2; ++u) r[u] = __builtin_nontemporal_load(sv + min(i + u * stride, a.vec - 1));
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (i + u * stride >= a.vec) continue;
            const uint32_t d[4] = {r[u].x, r[u].y, r[u].z, r[u].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                atomicAdd(&mine[(d[j] & 0xFFu) * kHistCopies], 1u);
                atomicAdd(&mine[((d[j] >> 8) & 0xFFu) * kHistCopies], 1u);
                atomicAdd(&mine[((d[j] >> 16) & 0xFFu) * kHistCopies], 1u);
                atomicAdd(&mine[(d[j] >> 24) * kHistCopies], 1u);
            }
        }
    }
    if (t0 == 0) a.outside([&](uint8_t b) { atomicAdd(&mine[(uint32_t)b * kHistCopies], 1u); });
    __syncthreads();
    // four threads per code, 16 copies each, every lane of a wavefront from a bank of its own
    const uint32_t code = threadIdx.x >> 2, part = threadIdx.x & 3u;
    uint32_t c = 0u;
#pragma unroll
    for (uint32_t i = 0; i < kHistCopies / 4; ++i)
        c += sh_scale[code * kHistCopies + part * (kHistCopies / 4) + ((i + code) & (kHistCopies / 4 - 1))];
    c += dpp_u<kDppXor1>(c);
    c += dpp_u<kDppXor2>(c);
    if (part == 0u) {
        if (groups == 1u) scale_hist[code] = c;                      // uniform
        else if (c) atomicAdd(&scale_hist[code], (unsigned long long)c);
    }
}

// Workgroup `group` of `groups` that count the codes.
__device__ __forceinline__ void count_codes(const ByteArray a, uint32_t group, uint32_t groups, uint32_t* sh_elem,
                                            unsigned long long* __restrict__ elem_hist)
{
    const u32x4* cv = a.vectors();
    const int64_t stride = (int64_t)groups * kHistThreads, t0 = (int64_t)group * kHistThreads + threadIdx.x;
    if (threadIdx.x < 8) sh_elem[threadIdx.x] = 0u;
    uint32_t cnt[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    for (int64_t i = t0; i < a.vec; i += 4 * stride) {               // four loads in flight per lane
        u32x4 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = __builtin_nontemporal_load(cv + min(i + u * stride, a.vec - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * stride < a.vec) count_magnitudes(r[u], cnt);
    }
    if (t0 == 0) {
        a.outside([&](uint8_t b) {
            cnt[b & 7u] += 1u;
            cnt[(b >> 4) & 7u] += 1u;
        });
    }
    __syncthreads();
    // the 16 lanes of a DPP row add up in registers; one lane per row adds into the LDS
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        uint32_t c = cnt[k];
        c += dpp_u<kDppXor1>(c);
        c += dpp_u<kDppXor2>(c);
        c += dpp_u<kDppHalfMirror>(c);
        c += dpp_u<kDppMirror>(c);
        if ((threadIdx.x & 15) == 0 && c) atomicAdd(&sh_elem[k], c);
    }
    __syncthreads();
    if (threadIdx.x < 8) {
        const uint32_t c = sh_elem[threadIdx.x];
        if (groups == 1u) elem_hist[threadIdx.x] = c;                // uniform
        else if (c) atomicAdd(&elem_hist[threadIdx.x], (unsigned long long)c);
    }
}

// The first `scale_groups` workgroups count the scales, the others the codes.
__global__ void __launch_bounds__(kHistThreads)
histogram_kernel(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales, int64_t n,
                 int64_t n_blocks, uint32_t scale_groups, unsigned long long* __restrict__ elem_hist,
                 unsigned long long* __restrict__ scale_hist)
{
    __shared__ __align__(16) uint32_t shared[kHistCopies * 256];
    if (blockIdx.x < scale_groups) count_scales(ByteArray(scales, n_blocks), blockIdx.x, scale_groups, shared, scale_hist);
    else count_codes(ByteArray(codes, n >> 1), blockIdx.x - scale_groups, gridDim.x - scale_groups, shared, elem_hist);
}

// Workgroups for `bytes` bytes of an array: one for every `least`, but a lane's and a workgroup's counters are 32-bit (at
// most 2^31 elements, two to a byte of codes).
static int64_t hist_groups(int64_t bytes, int64_t least)
{
    const int64_t groups = (bytes + least - 1) / least, needed = (bytes >> 30) + 1;
    return groups < needed ? needed : groups < kHistMaxGrid ? (groups < 1 ? 1 : groups) : needed < kHistMaxGrid ? kHistMaxGrid : needed;
}

hipError_t launch_histogram(const uint8_t* codes, const uint8_t* scales, int64_t n, int block,
                            unsigned long long* elem_hist, unsigned long long* scale_hist,
                            hipStream_t stream)
{
    const int64_t scale_groups = hist_groups(n / block, kHistScales), code_groups = hist_groups(n >> 1, kHistCodes);
    if (n == 0 || scale_groups > 1 || code_groups > 1) {
        hipLaunchKernelGGL(hist_clear_kernel, dim3(1), dim3(256), 0, stream, elem_hist, scale_hist);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || n == 0) return e;
    }
    hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)(scale_groups + code_groups)), dim3(kHistThreads), 0, stream,
                       codes, scales, n, n / block, (uint32_t)scale_groups, elem_hist, scale_hist);
    return hipGetLastError();
}

}  // namespace mxq
