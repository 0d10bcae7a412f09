// De-quantisation (Section 2, paragraph after Eq. 2: the codes times the block scale) and the tensor
// abs-max of hierarchical scaling (first stage of the two-stage process, Section 2).
#include "mxq_device.hpp"
#include "mxq_launch.hpp"

#include <mutex>

namespace mxq {

using bf16x2 = __bf16 __attribute__((ext_vector_type(2)));

// Two fp32 -> two bf16 (round to nearest even, v_cvt_pk_bf16_f32), first value in the low half.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// bf16 output: one lane = 8 consecutive elements = one dword of codes = one 128-bit store; a
// block of b >= 8 elements spans b/8 lanes that all read the same scale byte, a block of b < 8
// lies inside the lane.
//
// A workgroup does ITEMS chunks per lane and ends: all their loads are in flight before the first is
// converted, and no wavefront waits for a load in a loop with one in flight.  One chunk per lane where
// all workgroups of the tensor are resident at once (the shortest path through the kernel), else four:
// 4096 x 14336, b = 16, against a loop over single chunks in 2048 workgroups: bf16 28.2 -> 25.9 us
// (5.8 TB/s), fp32 56.5 -> 47.3 us (5.7 TB/s); two chunks 26.7 / 48.5 us, eight 26.9 / 50.0 us, one 31.0
// us.  16 x 4096 in a graph: one chunk 2.4 us, four 2.9 us.
// bf16 with b < 8, whose scales are half as many bytes as its codes or as many, takes three chunks a lane
// once four no longer leave all workgroups resident.  b = 2, loop -> four chunks with non-temporal scale
// loads -> as it is: 4096 x 4096 10.9 -> 11.4 -> 9.4 us (three chunks 10.5), 5000 x 4096 12.7 -> 14.1 ->
// 12.3 (four 13.4), 8192 x 4096 19.2 -> 20.2 -> 18.2 (19.6), 14336 x 4096 31.5 -> 31.7 -> 28.8 (30.1);
// b = 4 10.4 -> 10.3 -> 9.7, 11.9 -> 12.7 -> 10.9 (12.1), 18.4 -> 18.1 -> 16.8 (17.5), 29.4 -> 29.0 -> 27.3
// (27.8).  (With eight such tensors in turn, none of it found in the Infinity Cache, b = 2 stays up to 6 %
// behind the loop between 14 and 17 M elements.)
constexpr int kDqItems = 4, kDqItemsLarge = 3;
constexpr int64_t kDqResident = 256 * 8;                            // workgroups
template <int B, int ITEMS>
__global__ void __launch_bounds__(kThreads)
dequant_bf16_kernel(const uint32_t* __restrict__ codes, const uint8_t* __restrict__ scales, uint64_t n,
                    int fmt, float T_arg, const float* __restrict__ t_dev, uint16_t* __restrict__ out)
{
    const float T = t_dev ? *t_dev : T_arg;                         // per-tensor scale by value or from device memory
    constexpr int NBLK = (B < 8) ? 8 / B : 1;
    constexpr uint32_t LANES = (B < 8) ? 1 : B / 8;
    constexpr int EPB = (B < 8) ? B : 8;
    const uint64_t c0 = (uint64_t)blockIdx.x * (kThreads * ITEMS);
    const uint64_t n_full = n >> 3;
    const uint32_t valid = (c0 < n_full) ? (uint32_t)min((uint64_t)(kThreads * ITEMS), n_full - c0) : 0u;   // complete chunks here
    if (valid != 0u) {
        const uint32_t* cp = codes + c0;
        u32x4* op = reinterpret_cast<u32x4*>(out) + c0;
        const uint8_t* sp = scales + ((B >= 8) ? c0 / LANES : c0 * NBLK);
        uint32_t packed[ITEMS], sb[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t c = min((uint32_t)threadIdx.x + (uint32_t)i * kThreads, valid - 1u);
            packed[i] = __builtin_nontemporal_load(cp + c);
            if constexpr (NBLK == 4) sb[i] = reinterpret_cast<const uint32_t*>(sp)[c];
            else if constexpr (NBLK == 2) sb[i] = reinterpret_cast<const uint16_t*>(sp)[c];
            else sb[i] = sp[c / LANES];
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t c = (uint32_t)threadIdx.x + (uint32_t)i * kThreads;
            float r[8], S[NBLK];
#pragma unroll
            for (int k = 0; k < NBLK; ++k) S[k] = scale_byte_value(fmt, (sb[i] >> (8 * k)) & 0xFFu);
            e2m1_unpack8(packed[i], 1.0f, r);
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = (r[j] * S[j / EPB]) * T;
            u32x4 o;
            o.x = pack_bf16x2(r[0], r[1]);
            o.y = pack_bf16x2(r[2], r[3]);
            o.z = pack_bf16x2(r[4], r[5]);
            o.w = pack_bf16x2(r[6], r[7]);
            if (c < valid) __builtin_nontemporal_store(o, op + c);
        }
    }
    if constexpr (B < 8) {                                          // n not a multiple of 8: the last few, two by two
        const uint64_t first = n_full << 3;
        const uint32_t pair = threadIdx.x;
        if (blockIdx.x == gridDim.x - 1u && first + 2u * pair < n) {
            const uint64_t at = first + 2u * pair;
            float a, b;
            e2m1_unpack2<0>((uint32_t)reinterpret_cast<const uint8_t*>(codes)[at >> 1], 1.0f, a, b);
            const float S = scale_byte_value(fmt, scales[at / B]);
            out[at] = (uint16_t)(pack_bf16x2((a * S) * T, 0.0f) & 0xFFFFu);
            out[at + 1u] = (uint16_t)(pack_bf16x2((b * S) * T, 0.0f) & 0xFFFFu);
        }
    }
}

// fp32 output: one lane = 4 consecutive elements = 16 bits of codes = one 128-bit store, so a
// store instruction of a wavefront covers 1 KiB without gaps (with 8 elements per lane its two
// stores would each leave every other 16 bytes untouched).  n is even, so at most 2 elements are
// left behind the complete quads.
template <int B, int ITEMS>
__global__ void __launch_bounds__(kThreads)
dequant_f32_kernel(const uint16_t* __restrict__ codes, const uint8_t* __restrict__ scales, uint64_t n, int fmt, float T_arg, const float* __restrict__ t_dev, float* __restrict__ out)
{
    const float T = t_dev ? *t_dev : T_arg;
    constexpr int EPB = (B < 4) ? B : 4;
    constexpr uint32_t LANES = (B < 4) ? 1 : B / 4;
    const uint64_t q0 = (uint64_t)blockIdx.x * (kThreads * ITEMS);
    const uint64_t n_full = n >> 2;
    const uint32_t valid = (q0 < n_full) ? (uint32_t)min((uint64_t)(kThreads * ITEMS), n_full - q0) : 0u;   // complete quads here
    if (valid != 0u) {
        const uint16_t* cp = codes + q0;
        u32x4* op = reinterpret_cast<u32x4*>(out) + q0;
        const uint8_t* sp = scales + ((B >= 4) ? q0 / LANES : q0 * 2u);
        uint32_t packed[ITEMS], sb[ITEMS];
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t q = min((uint32_t)threadIdx.x + (uint32_t)i * kThreads, valid - 1u);
            packed[i] = __builtin_nontemporal_load(cp + q);
            if constexpr (B == 2) sb[i] = *reinterpret_cast<const uint16_t*>(sp + q * 2u);
            else sb[i] = sp[q / LANES];
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t q = (uint32_t)threadIdx.x + (uint32_t)i * kThreads;
            float r[4], S[4 / EPB];
#pragma unroll
            for (int k = 0; k < 4 / EPB; ++k) S[k] = scale_byte_value(fmt, (sb[i] >> (8 * k)) & 0xFFu);
            e2m1_unpack2<0>(packed[i], 1.0f, r[0], r[1]);
            e2m1_unpack2<1>(packed[i], 1.0f, r[2], r[3]);
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = (r[j] * S[j / EPB]) * T;
            const u32x4 o = {f2u(r[0]), f2u(r[1]), f2u(r[2]), f2u(r[3])};
            if (q < valid) __builtin_nontemporal_store(o, op + q);
        }
    }
    if constexpr (B < 4) {
        const uint64_t at = n_full << 2;
        if (at < n && blockIdx.x == gridDim.x - 1u && threadIdx.x == 0u) {
            float a, b;
            e2m1_unpack2<0>((uint32_t)reinterpret_cast<const uint8_t*>(codes)[at >> 1], 1.0f, a, b);
            const float S = scale_byte_value(fmt, scales[at / B]);
            out[at] = (a * S) * T;
            out[at + 1u] = (b * S) * T;
        }
    }
}

static void launch_dequant_f32(const DequantArgs& a)
{
    const bool one = a.n <= kDqResident * kThreads * 4;
    const int64_t tile = 4 * (int64_t)kThreads * (one ? 1 : kDqItems);
    const unsigned grid = (unsigned)((a.n + tile - 1) / tile);
#define MXQ_DQF(BB)                                                                                  \
    hipLaunchKernelGGL((one ? dequant_f32_kernel<BB, 1> : dequant_f32_kernel<BB, kDqItems>), dim3(grid), dim3(kThreads), 0, a.stream,    \
                       (const uint16_t*)a.codes, a.scales, (uint64_t)a.n, a.scale_fmt, a.T, a.t_dev, (float*)a.out)
    switch (a.block) {
        case 2: MXQ_DQF(2); break;
        case 4: MXQ_DQF(4); break;
        case 8: MXQ_DQF(8); break;
        case 16: MXQ_DQF(16); break;
        case 32: MXQ_DQF(32); break;
        case 64: MXQ_DQF(64); break;
        default: MXQ_DQF(128); break;
    }
#undef MXQ_DQF
}

static void launch_dequant_bf16(const DequantArgs& a)
{
    const int64_t resident = kDqResident * kThreads * 8;                 // elements, one chunk per lane
    const int items = a.n <= resident ? 1 : (a.block < 8 && a.n > resident * kDqItems) ? kDqItemsLarge : kDqItems;
    const int64_t tile = 8 * (int64_t)kThreads * items;
    const unsigned grid = (unsigned)((a.n + tile - 1) / tile);
#define MXQ_DQ(BB)                                                                                   \
    hipLaunchKernelGGL((items == 1 ? dequant_bf16_kernel<BB, 1> : items == kDqItems ? dequant_bf16_kernel<BB, kDqItems>         \
                        : dequant_bf16_kernel<BB, (BB < 8) ? kDqItemsLarge : kDqItems>), dim3(grid), dim3(kThreads), 0,         \
                       a.stream, (const uint32_t*)a.codes, a.scales, (uint64_t)a.n, a.scale_fmt, a.T, a.t_dev, (uint16_t*)a.out)
    switch (a.block) {
        case 2: MXQ_DQ(2); break;
        case 4: MXQ_DQ(4); break;
        case 8: MXQ_DQ(8); break;
        case 16: MXQ_DQ(16); break;
        case 32: MXQ_DQ(32); break;
        case 64: MXQ_DQ(64); break;
        default: MXQ_DQ(128); break;
    }
#undef MXQ_DQ
}

// A grid counts fewer than 2^32 threads of 16 to 32 elements: larger tensors (codes or output may lie in
// host memory that the GPU can address) are taken in pieces.
constexpr int64_t kDqPiece = (int64_t)1 << 35;

hipError_t launch_dequant(const DequantArgs& a)
{
    DequantArgs piece = a;
    for (int64_t done = 0; done < a.n; done += kDqPiece) {
        piece.codes = a.codes + done / 2;
        piece.scales = a.scales + done / a.block;
        piece.out = static_cast<char*>(a.out) + done * (a.dtype == kBF16 ? 2 : 4);
        piece.n = a.n - done < kDqPiece ? a.n - done : kDqPiece;
        if (a.dtype == kBF16) launch_dequant_bf16(piece);
        else launch_dequant_f32(piece);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Tensor abs-max.  |x| of finite fp32 values orders like the unsigned integer bits & 0x7fffffff,
// so the reduction is an integer max; the workgroups' partial results meet in one 32-bit atomic
// max on a device word.  Two closing schemes (and a third for tensors small enough for one workgroup,
// further down):
//   * no workspace: the word is the caller's output, which a one-thread kernel clears first (a
//     kernel, not a memset node, so the pair can be captured in a graph) -- two launches -- or
//     which the caller guarantees to hold zero (or a maximum to be continued) -- one launch; that
//     form can clear a second word on the way, the output of the caller's next call;
//   * workspace (two words: accumulator, ticket; both zero between calls): every workgroup adds
//     its maximum to the accumulator, then takes a ticket; the workgroup that draws the last
//     ticket copies the accumulator to the output and returns both words to zero -- one launch.
__global__ void absmax_clear_kernel(uint32_t* out) { *out = 0u; }

// One workgroup of 1024 threads per compute unit with four independent 128-bit loads per lane in
// flight (16 MiB over the chip); the ragged last chunk (n not a multiple of 8) is read element-wise
// by one lane.  Few, large workgroups because the closing accesses to the one word serialise at about
// 5 ns each, whatever their kind.
//
// The quantise pass of hierarchical scaling reads the tensor next, and what is still in a die's L2
// (4 MiB on each of eight) or in the Infinity Cache need not come from HBM again.  So every die reads
// here what it will read there: workgroups go to the dies in turn, the streaming kernels give slice s
// (256 chunks) to a workgroup on die s mod 8, and the eight workgroups of a team share a group of
// 512 KiB slice by slice in the same way.  Groups are walked from the last to the first, because the
// quantise pass begins at the first.  The first 64 MiB are read with ordinary loads, which stay in the
// caches, what lies behind them (and is read before them) with non-temporal ones.  Abs-max and abs-max
// quantisation (b = 16) in a graph, contiguous ascending tiles and non-temporal loads throughout -> this
// order, ordinary loads throughout -> as it is: bf16 64 MiB 30.9 -> 27.2 -> 26.6 us, 112 MiB 49.2 -> 46.0
// -> 45.2, 384 MiB 153 -> 164 -> 149; fp32 128 MiB 52.5 -> 46.7 -> 46.8.  The abs-max alone: 64 MiB 13.7 ->
// 14.8 -> 14.5, 112 MiB 21.1 -> 22.8 -> 21.8, 224 MiB 39.1 -> 41.6 -> 38.7.  With 32 MiB kept instead of 64
// it is as fast as with none (13.9, 20.9, 38.1), but the pair on re-used outputs loses 1 us at 64 MiB, up to 4 on fp32.
// (Ordinary loads also push out what others have written: eight fills of 64 MiB and eight abs-max take 30.5
// us a pair instead of 24.3, and quantising with b <= 4 into fresh buffers loses 5 to 10 %.)
constexpr int kAbsItems = 4;
constexpr int kAbsThreads = 1024;
constexpr int kAbsMaxGrid = 256;
constexpr int kAbsTile = kAbsThreads * kAbsItems;                    // vectors a workgroup has in flight
constexpr int64_t kAbsKeepVectors = (64 << 20) / 16;

// Maximum over the lane's vectors of one group (bit pattern); `left` vectors of the tensor from `base` on.
template <int DT, bool STREAM>
__device__ __forceinline__ uint32_t group_absmax(const u32x4* base, uint32_t left, uint32_t off, uint32_t step)
{
    u32x4 r[kAbsItems];
#pragma unroll
    for (int i = 0; i < kAbsItems; ++i) {
        const u32x4* p = base + min(off + (uint32_t)i * step, left - 1u);      // lanes beyond it read the last vector again
        if constexpr (STREAM) r[i] = __builtin_nontemporal_load(p);
        else r[i] = *p;
    }
    uint32_t m = 0u;
#pragma unroll
    for (int i = 0; i < kAbsItems; ++i) {
        if constexpr (DT == kBF16) {
            // two bf16 per dword: compare the high halves and the low halves separately
            const uint32_t hi = max(max(r[i].x & 0x7FFF0000u, r[i].y & 0x7FFF0000u),
                                    max(r[i].z & 0x7FFF0000u, r[i].w & 0x7FFF0000u));
            const uint32_t lo = max(max(r[i].x & 0x7FFFu, r[i].y & 0x7FFFu),
                                    max(r[i].z & 0x7FFFu, r[i].w & 0x7FFFu));
            m = max(m, max(hi, lo << 16));
        } else {
            m = max(m, max(max(r[i].x & 0x7FFFFFFFu, r[i].y & 0x7FFFFFFFu),
                           max(r[i].z & 0x7FFFFFFFu, r[i].w & 0x7FFFFFFFu)));
        }
    }
    return m;
}

// Maximum over the workgroup's share (bit pattern); valid in thread 0.  ALONE: one workgroup, tile by
// tile.  Else the grid is a multiple of 8, or less than 8 for a tensor of no more tiles than workgroups.
template <int DT, bool ALONE>
__device__ __forceinline__ uint32_t workgroup_absmax(const void* __restrict__ x, int64_t n)
{
    constexpr int64_t kVec = (DT == kBF16) ? 1 : 2;               // 128-bit vectors per chunk
    const int64_t n_vec = (n >> 3) * kVec;                         // complete vectors
    const u32x4* xv = static_cast<const u32x4*>(x);
    constexpr uint32_t kSlice = kThreads * (uint32_t)kVec;         // vectors of a slice of the streaming kernels
    constexpr int64_t kGroup = kAbsTile * (ALONE ? 1 : 8);         // vectors; powers of two, no division
    uint32_t m = 0u;
    const uint32_t members = ALONE ? 1u : min(gridDim.x, 8u), member = ALONE ? 0u : blockIdx.x & 7u;
    const uint32_t teams = ALONE ? 1u : (gridDim.x + 7u) >> 3;
    const uint32_t off = (member + threadIdx.x / kSlice * members) * kSlice + threadIdx.x % kSlice;
    const uint32_t step = members * kAbsThreads;
    int64_t g = (n_vec + kGroup - 1) / kGroup - 1 - (int64_t)(ALONE ? 0u : blockIdx.x >> 3);
    if constexpr (!ALONE) {
        // (A loop of its own: of two loads in the branches of one the compiler makes a single ordinary one.)
        for (; g >= kAbsKeepVectors / kGroup; g -= teams)                                               // uniform
            m = max(m, group_absmax<DT, true>(xv + g * kGroup, (uint32_t)min(kGroup, n_vec - g * kGroup), off, step));
    }
    for (; g >= 0; g -= teams)                                                                          // uniform
        m = max(m, group_absmax<DT, false>(xv + g * kGroup, (uint32_t)min(kGroup, n_vec - g * kGroup), off, step));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        for (int64_t i = (n >> 3) << 3; i < n; ++i) {
            uint32_t b;
            if constexpr (DT == kBF16) b = (uint32_t)static_cast<const uint16_t*>(x)[i] << 16;
            else b = static_cast<const uint32_t*>(x)[i];
            m = max(m, b & 0x7FFFFFFFu);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    __shared__ uint32_t part[kAbsThreads / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    uint32_t w = 0u;
    if (threadIdx.x == 0) {
        w = part[0];
        for (int i = 1; i < kAbsThreads / 64; ++i) w = max(w, part[i]);
    }
    return w;
}

template <int DT, bool TICKET>
__global__ void __launch_bounds__(kAbsThreads)
absmax_kernel(const void* __restrict__ x, int64_t n, uint32_t* __restrict__ out, uint32_t* __restrict__ ws,
              uint32_t* __restrict__ clear_word)
{
    if (clear_word && blockIdx.x == 0 && threadIdx.x == 0) *clear_word = 0u;      // for a LATER launch
    const uint32_t w = workgroup_absmax<DT, false>(x, n);
    if (threadIdx.x == 0) {
        if constexpr (!TICKET) {
            // The word only grows during a call, so a workgroup whose maximum does not exceed the
            // value it reads (at device scope, past the per-CU cache) has nothing to add: after
            // the first few workgroups almost none issues the atomic max.
            if (w > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, w);
        } else {
            // Read-modify-writes at device scope are performed at the one point all compute dies
            // share.  The ticket is requested only after the value returned by the max has arrived
            // (its increment depends on it), i.e. after the max was performed there; the workgroup
            // that draws the last ticket therefore exchanges out a word that already holds every
            // other workgroup's contribution.  No cache-wide fence is needed (one costs several
            // microseconds here, more than the second launch it would save).
            const uint32_t before = atomicMax(ws, w);
            const uint32_t ticket = atomicAdd(ws + 1, 1u + (before >> 31));      // bit 31 is never set
            if (ticket == gridDim.x - 1u) {
                *out = atomicExch(ws, 0u);
                atomicExch(ws + 1, 0u);
            }
        }
    }
}

// A tensor that one workgroup reads in the time a second launch costs: no word to clear, no atomic,
// no workspace -- one launch for every form but the running maximum (whose word other streams may be
// raising at the same time; it is one launch anyway).  One workgroup against several, graph replay, bf16:
// with the clearing launch 16 KiB 2.3 against 4.1 us, 128 KiB 2.9 against 4.3, 160 KiB 3.3 against 4.2; with
// the ticket 16 KiB 2.3 against 3.2 to 3.6, 128 KiB 2.9 against 3.4, 160 KiB 3.3 against 3.3 -- so the line
// lies at 160 KiB for all of them.  (A division by the number of workgroups that share a group cost every
// call of this size 0.3 us; groups are powers of two now.)
// Launched one by one from Python the second launch costs another 3.5 us of host time.
constexpr int64_t kAbsSmallBytes = 160 << 10;

template <int DT>
__global__ void __launch_bounds__(kAbsThreads)
absmax_small_kernel(const void* __restrict__ x, int64_t n, uint32_t* __restrict__ out)
{
    const uint32_t w = workgroup_absmax<DT, true>(x, n);
    if (threadIdx.x == 0) *out = w;
}

// Workgroups for `tiles` tiles: one each up to 8 (a team reads its group of 8 at once), then whole teams up
// to one workgroup per compute unit.  A ticket costs a workgroup three dependent accesses to one place, so
// with tickets it reads at least two tiles as soon as there are 64 workgroups (16 MiB: 10.3 -> 7.2 us).
static unsigned absmax_grid(int64_t tiles, bool ticket)
{
    if (tiles <= 8) return (unsigned)tiles;
    int64_t teams = tiles / 8 + (tiles % 8 != 0 ? 1 : 0);
    if (ticket && teams > 8) teams = (teams < 16) ? 8 : (teams + 1) / 2;
    return 8u * (unsigned)(teams < kAbsMaxGrid / 8 ? teams : kAbsMaxGrid / 8);
}

// `ws`: the two-word workspace of the ticket scheme, or NULL.  `accumulate` (without ws): the output
// word is not cleared first; `clear_word` (accumulate only, may be NULL) is set to zero instead.
hipError_t launch_absmax(const void* x, int64_t n, int dtype, float* out, uint32_t* ws, bool accumulate,
                         float* clear_word, hipStream_t stream)
{
    if (accumulate && n == 0) {
        if (!clear_word) return hipSuccess;
        hipLaunchKernelGGL(absmax_clear_kernel, dim3(1), dim3(1), 0, stream, (uint32_t*)clear_word);
        return hipGetLastError();
    }
    if (!accumulate && n > 0 && n * (dtype == kBF16 ? 2 : 4) <= kAbsSmallBytes) {
        const dim3 one(1), block(kAbsThreads);
        if (dtype == kBF16) hipLaunchKernelGGL(absmax_small_kernel<kBF16>, one, block, 0, stream, x, n, (uint32_t*)out);
        else hipLaunchKernelGGL(absmax_small_kernel<kF32>, one, block, 0, stream, x, n, (uint32_t*)out);
        return hipGetLastError();
    }
    if ((!ws && !accumulate) || n == 0) {
        hipLaunchKernelGGL(absmax_clear_kernel, dim3(1), dim3(1), 0, stream, (uint32_t*)out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || n == 0) return e;
    }
    const int64_t per_tile = kAbsTile * (dtype == kBF16 ? 8 : 4);                    // elements
    const dim3 grid(absmax_grid(n / per_tile + (n % per_tile != 0 ? 1 : 0), ws != nullptr)), block(kAbsThreads);
    uint32_t* o = (uint32_t*)out;
    uint32_t* cw = (uint32_t*)clear_word;
    if (dtype == kBF16) {
        if (ws) hipLaunchKernelGGL((absmax_kernel<kBF16, true>), grid, block, 0, stream, x, n, o, ws, cw);
        else hipLaunchKernelGGL((absmax_kernel<kBF16, false>), grid, block, 0, stream, x, n, o, ws, cw);
    } else {
        if (ws) hipLaunchKernelGGL((absmax_kernel<kF32, true>), grid, block, 0, stream, x, n, o, ws, cw);
        else hipLaunchKernelGGL((absmax_kernel<kF32, false>), grid, block, 0, stream, x, n, o, ws, cw);
    }
    return hipGetLastError();
}

// Workspace of the entry point that may not allocate and takes no workspace argument: the two
// words of the ticket scheme (the rest is padding to the alignment) live in the library's own
// device image, one copy per GPU, zero when the image is loaded and returned to zero by every call.
// In host code the array's name is only a handle for hipGetSymbolAddress; the address it yields for
// the current device is what kernels and launches are given.
constexpr int kStaticScratchWords = 64;
static __device__ __align__(256) uint32_t scratch[kStaticScratchWords];

constexpr int kMaxDevices = 64;
static uint32_t* g_scratch_ptr[kMaxDevices];      // device address of `scratch`, per device
static std::mutex g_scratch_mutex;

// Device address of the current device's copy of `scratch`, resolved once per device.
static hipError_t static_scratch(uint32_t** ptr)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<uint32_t*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

// The ticket scheme on the library's own workspace: no allocation, no workspace argument.
hipError_t launch_absmax_static(const void* x, int64_t n, int dtype, float* out, hipStream_t stream)
{
    uint32_t* ws = nullptr;
    const hipError_t e = static_scratch(&ws);
    if (e != hipSuccess) return e;
    return launch_absmax(x, n, dtype, out, ws, false, nullptr, stream);
}

}  // namespace mxq
