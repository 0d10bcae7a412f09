// Streaming recipes of Section 2: abs-max scale (Eq. 2; Eq. 1 for power-of-two scales),
// prevent-zero clamp (Eq. 3) and 4-over-6 (Eq. 4), one pass over the tensor.
//
// Mapping: every lane owns 8 consecutive elements (one 128-bit load for bf16, two for fp32),
// so a block of b >= 8 elements is b/8 neighbouring lanes of one DPP row and a block of
// b < 8 sits inside a lane.  Per lane the kernel emits one dword of packed codes; the first
// lane of a block emits the scale byte and the block SSE.  Loads are issued before what is processed
// meanwhile: the next chunk's in a loop, or three chunks' at once in workgroups that end (large tensors).
// HBM-bound by design: algorithmic traffic is sizeof(in) + 0.5 + 5/b bytes per element.
#include "mxq_device.hpp"
#include "mxq_launch.hpp"

#include <type_traits>

#ifndef MXQ_STREAM_ITEMS
#define MXQ_STREAM_ITEMS 1
#endif

namespace mxq {

// Eq. 2 / Eq. 3: scale codes from the block abs-max for M = 6 and (4-over-6 only) M = 4.
// `floor_code` is 1 under prevent-zero (eps_SF is code 1 in both formats), else 0.  For E4M3 one
// v_cvt_pk_fp8_f32 rounds both quotients.
template <int FMT, bool FOUR6>
__device__ __forceinline__ void absmax_codes(float amax, uint32_t floor_code, uint32_t& c6, uint32_t& c4)
{
    const float y6 = sixth_of(amax);
    const float y4 = quarter_of(amax);
    if constexpr (FMT == kE4M3) {
        const float m = ScaleFmt<kE4M3>::kMaxValue;
        int old;                                       // the conversion writes the low half; the high half is never read
        asm volatile("" : "=v"(old));
        const uint32_t both = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(fminf(y6, m), fminf(y4, m), old, false);
        c6 = max(both & 0xFFu, floor_code);
        c4 = FOUR6 ? max((both >> 8) & 0xFFu, floor_code) : 0u;
    } else {
        c6 = max(sf_encode_rne<FMT>(y6), floor_code);
        c4 = FOUR6 ? max(sf_encode_rne<FMT>(y4), floor_code) : 0u;
    }
}

// Quantise the lane's 8 values (NBLK blocks of EPB elements, one table entry each): packed nibbles and
// the 8 squared residuals.  The quotient is one truncated product with 1/S (ScalePair) or the
// two-part product (ScaleEntry).
template <int NBLK, int EPB, class Entry>
__device__ __forceinline__ void quant_lane(const float (&v)[8], const Entry (&entry)[NBLK], uint32_t& packed, float (&sq)[8],
                                           float (&S)[NBLK])
{
    float y[8];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) S[k] = entry[k].S;
    if constexpr (Entry::kOneProduct) {
        float r[NBLK];
#pragma unroll
        for (int k = 0; k < NBLK; ++k) r[k] = entry[k].r;
        quot8_truncated<NBLK>(v, r, y);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = quot(v[j], Recip{entry[j / EPB].rhi, entry[j / EPB].rlo});
    }
    packed = e2m1_pack8(y, 1.0f);
    float q[8];
    e2m1_unpack8(packed, 1.0f, q);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float e = __builtin_fmaf(-q[j], S[j / EPB], v[j]);   // q*S is exact: one rounding
        sq[j] = e * e;
    }
}

// Same under power-of-two scales 2^(code-127): v / 2^k is exact, so the conversion
// instruction applies each block's scale itself and the inverse conversion returns q * S.
template <int NBLK, int EPB>
__device__ __forceinline__ void quant_lane_pow2(const float (&v)[8], const uint32_t (&code)[NBLK],
                                                uint32_t& packed, float (&sq)[8], float (&S)[NBLK])
{
#pragma unroll
    for (int k = 0; k < NBLK; ++k) S[k] = (code[k] == 0u) ? u2f(0x00400000u) : u2f(code[k] << 23);
    packed = e2m1_pack8_scales<EPB>(v, S);
    float qS[8];
    e2m1_unpack2<0>(packed, S[0 / EPB], qS[0], qS[1]);
    e2m1_unpack2<1>(packed, S[2 / EPB], qS[2], qS[3]);
    e2m1_unpack2<2>(packed, S[4 / EPB], qS[4], qS[5]);
    e2m1_unpack2<3>(packed, S[6 / EPB], qS[6], qS[7]);
#pragma unroll
    for (int j = 0; j < 8; ++j) { const float e = v[j] - qS[j]; sq[j] = e * e; }
}

// Clipping-only part of the block SSE (appendix figure "Clipping only MSE"): the squared residuals
// of the elements that saturate, |v| > 6 S (the same decision as fl32(|v| / S) > 6, because 6 S is
// exact), others contribute +0; S = 0 clips nothing.  A saturating element quantises to +-6, so its
// squared residual is the one the block SSE already holds.
template <int B, int NBLK, int EPB>
__device__ __forceinline__ void block_clip_sse(const float (&v)[8], const float (&sq)[8], const float (&S)[NBLK],
                                               float (&clip)[4])
{
    float csq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float s = S[j / EPB];
        csq[j] = (__builtin_fabsf(v[j]) > 6.0f * s && s > 0.0f) ? sq[j] : 0.0f;
    }
    block_sse<B>(csq, clip);
}

// Everything between the load and the store for one lane's 8 values.  `tdyn` (one of kNoT,
// kFastT, kSlowT; wave-uniform) is read only when TMODE == kDynT.
template <int B, int FMT, bool FOUR6, int TMODE, bool CLIP, class Entry>
__device__ __forceinline__ void process_chunk(float (&v)[8], float T, float rT, int tdyn, bool pz,
                                              const Entry* tab, uint32_t& packed,
                                              uint32_t (&code_out)[(B < 8) ? 8 / B : 1], float (&sse_sel)[4],
                                              float (&clip_sel)[4])
{
    constexpr int NBLK = (B < 8) ? 8 / B : 1;          // blocks inside one lane
    constexpr int LANES = (B < 8) ? 1 : B / 8;         // lanes per block
    constexpr int EPB = (B < 8) ? B : 8;               // elements of one block inside a lane

    float amax[NBLK];
    if constexpr (TMODE == kDynT) {
        if (tdyn == kNoT) adjust_and_amax<kNoT, NBLK, EPB, LANES>(v, T, rT, amax);
        else if (tdyn == kFastT) adjust_and_amax<kFastT, NBLK, EPB, LANES>(v, T, rT, amax);
        else adjust_and_amax<kSlowT, NBLK, EPB, LANES>(v, T, rT, amax);
    } else {
        adjust_and_amax<TMODE, NBLK, EPB, LANES>(v, T, rT, amax);
    }

    float sq[8], S[NBLK];
    if constexpr (FMT == kE8M0) {
#pragma unroll
        for (int k = 0; k < NBLK; ++k) code_out[k] = pow2_code(amax[k]);
        quant_lane_pow2<NBLK, EPB>(v, code_out, packed, sq, S);
        block_sse<B>(sq, sse_sel);
        if constexpr (CLIP) block_clip_sse<B, NBLK, EPB>(v, sq, S, clip_sel);
    } else {
        uint32_t c4[NBLK];
        const uint32_t floor_code = pz ? 1u : 0u;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) absmax_codes<FMT, FOUR6>(amax[k], floor_code, code_out[k], c4[k]);
        Entry entry[NBLK];
#pragma unroll
        for (int k = 0; k < NBLK; ++k) entry[k] = tab[code_out[k]];
        quant_lane<NBLK, EPB>(v, entry, packed, sq, S);
        block_sse<B>(sq, sse_sel);
        if constexpr (CLIP) block_clip_sse<B, NBLK, EPB>(v, sq, S, clip_sel);
        if constexpr (FOUR6) {
            uint32_t packed4;
            float sse4[4], clip4[4];
#pragma unroll
            for (int k = 0; k < NBLK; ++k) entry[k] = tab[c4[k]];
            quant_lane<NBLK, EPB>(v, entry, packed4, sq, S);
            block_sse<B>(sq, sse4);
            if constexpr (CLIP) block_clip_sse<B, NBLK, EPB>(v, sq, S, clip4);
            // Eq. 4: M = 4 only when its SSE is strictly lower
#pragma unroll
            for (int k = 0; k < NBLK; ++k) {
                if (sse4[k] < sse_sel[k]) {
                    constexpr uint32_t m = (EPB == 8) ? 0xFFFFFFFFu : ((1u << ((4 * EPB) & 31)) - 1u);
                    const uint32_t mask = m << ((4 * EPB * k) & 31);
                    packed = (packed & ~mask) | (packed4 & mask);
                    code_out[k] = c4[k];
                    sse_sel[k] = sse4[k];
                    if constexpr (CLIP) clip_sel[k] = clip4[k];
                }
            }
        }
    }
}

template <int DT> struct RawChunk;
template <> struct RawChunk<kBF16> { u32x4 a; };
template <> struct RawChunk<kF32> { u32x4 a, b; };

// `tile` points at the workgroup's 256 chunks (wave-uniform), `tid` is the lane's chunk inside
// it and `chunks` the number of valid chunks (lanes beyond them re-read the last valid data).
// bf16: one 128-bit load per lane.  fp32: a chunk is two 128-bit vectors; so that every load
// instruction of a wavefront covers 1 KiB without gaps, lane l of wave w reads vectors
// 128w + l and 128w + 64 + l, and widen() below hands every lane its own chunk through LDS.
template <int DT>
__device__ __forceinline__ RawChunk<DT> load_raw(const u32x4* __restrict__ tile, uint32_t tid, uint32_t chunks)
{
    RawChunk<DT> r;
    if constexpr (DT == kBF16) {
        r.a = __builtin_nontemporal_load(tile + min(tid, chunks - 1u));
    } else {
        const uint32_t j = 2u * (tid & ~63u) + (tid & 63u);
        const uint32_t last = 2u * chunks - 1u;
        r.a = __builtin_nontemporal_load(tile + min(j, last));
        r.b = __builtin_nontemporal_load(tile + min(j + 64u, last));
    }
    return r;
}

// Raw registers -> the lane's 8 consecutive elements as fp32.  fp32 input: the wavefront
// writes its two 1 KiB load results to its private 2 KiB of LDS and every lane reads back
// vectors 2l and 2l + 1.  LDS operations of one wavefront execute in program order, so no
// barrier instruction is needed; the fences keep the compiler from reordering across them.
template <int DT>
__device__ __forceinline__ void widen(const RawChunk<DT>& r, float (&v)[8], u32x4* wave_lds)
{
    if constexpr (DT == kBF16) {
        v[0] = u2f(r.a.x << 16); v[1] = u2f(r.a.x & 0xFFFF0000u);
        v[2] = u2f(r.a.y << 16); v[3] = u2f(r.a.y & 0xFFFF0000u);
        v[4] = u2f(r.a.z << 16); v[5] = u2f(r.a.z & 0xFFFF0000u);
        v[6] = u2f(r.a.w << 16); v[7] = u2f(r.a.w & 0xFFFF0000u);
    } else {
        const uint32_t l = threadIdx.x & 63u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        wave_lds[l] = r.a;
        wave_lds[64u + l] = r.b;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const u32x4 a = wave_lds[2u * l], b = wave_lds[2u * l + 1u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        v[0] = u2f(a.x); v[1] = u2f(a.y); v[2] = u2f(a.z); v[3] = u2f(a.w);
        v[4] = u2f(b.x); v[5] = u2f(b.y); v[6] = u2f(b.z); v[7] = u2f(b.w);
    }
}

// Results of one lane for one tile, kept in registers until they are stored.
template <int B>
struct TileOut {
    static constexpr int NBLK = (B < 8) ? 8 / B : 1;
    uint32_t packed;
    uint32_t code[NBLK];
    float sse[4];
    float clip[4];       // clipping-only SSE; carried only by the kernels that output it
};

// The complete chunks are cut into slices of 256 chunks (one chunk per lane).  Slice indices
// are 32-bit and wave-uniform, so all tile arithmetic runs on the scalar unit and every address
// is a scalar base plus a 32-bit lane offset.
struct Slices {
    uint32_t count;        // number of slices
    uint32_t last;         // chunks in the last slice, 1 .. 256
    __device__ __forceinline__ uint32_t chunks(uint32_t s) const { return (s + 1u == count) ? last : (uint32_t)kThreads; }
    __device__ __forceinline__ uint64_t elements() const                             // in all complete chunks
    {
        return (count == 0u) ? 0u : ((uint64_t)(count - 1u) * kThreads + last) * 8u;
    }
};

// Flags of a launch (wave-uniform).
enum : int { kPreventZero = 1, kSsePastCaches = 2 };

// A block SSE is written and not read again here.  With ordinary stores it displaces other lines in the caches;
// written past them (non-temporal) it does not, but a later reader, or the next call that writes the same
// buffer, finds nothing there.  (The two asm comments keep the compiler from making one store of both.)
// Only the kernels that sse_past_caches may send there have the choice (kMayPass): it costs the others 1 % (fp32
// b = 16 1024 x 4096 5.04 -> 4.92 us, 4096 x 14336 50.4 -> 50.2; bf16 abs-max b = 16 512 x 4096 2.98 -> 2.91).
template <int DT, int B, bool FOUR6, int TMODE, bool CLIP>
constexpr bool kMayPass = DT == kBF16 && (FOUR6 || B == 2 || TMODE == kDynT || TMODE == kLeanT) && !CLIP;

template <bool MAY_PASS, class V>
__device__ __forceinline__ void store_sse(V* p, V v, int flags)
{
    if constexpr (!MAY_PASS) {
        *p = v;
    } else if (flags & kSsePastCaches) {
        asm volatile("; block SSE, past the caches");
        __builtin_nontemporal_store(v, p);
        asm volatile("; block SSE, past the caches, stored");
    } else {
        asm volatile("; block SSE");
        *p = v;
        asm volatile("; block SSE, stored");
    }
}

// Stores of one slice.
template <int B, bool MAY_PASS>
__device__ __forceinline__ void store_slice(const TileOut<B>& o, uint32_t s, Slices sl, int flags,
                                            uint32_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                            float* __restrict__ sse_out, float* __restrict__ clip_out)
{
    constexpr int NBLK = TileOut<B>::NBLK;
    constexpr int LANES = (B < 8) ? 1 : B / 8;
    const uint32_t tid = threadIdx.x;
    if (s >= sl.count) return;                                       // uniform
    const uint64_t c0 = (uint64_t)s * kThreads;                      // first chunk of the slice
    if (tid < sl.chunks(s)) {
        __builtin_nontemporal_store(o.packed, codes + c0 + tid);
        if constexpr (B >= 8) {
            if ((tid & (LANES - 1)) == 0) {
                const uint32_t blk = tid / LANES;
                (scales + c0 / LANES)[blk] = (uint8_t)o.code[0];
                if (sse_out) store_sse<MAY_PASS>((sse_out + c0 / LANES) + blk, o.sse[0], flags);
                if (clip_out) (clip_out + c0 / LANES)[blk] = o.clip[0];
            }
        } else if constexpr (NBLK == 2) {
            reinterpret_cast<uint16_t*>(scales + c0 * 2)[tid] = (uint16_t)(o.code[0] | (o.code[1] << 8));
            if (sse_out) store_sse<MAY_PASS>(reinterpret_cast<f32x2*>(sse_out + c0 * 2) + tid, f32x2{o.sse[0], o.sse[1]}, flags);
            if (clip_out) reinterpret_cast<float2*>(clip_out + c0 * 2)[tid] = make_float2(o.clip[0], o.clip[1]);
        } else {
            reinterpret_cast<uint32_t*>(scales + c0 * 4)[tid] =
                o.code[0] | (o.code[1] << 8) | (o.code[2] << 16) | (o.code[3] << 24);
            if (sse_out)
                store_sse<MAY_PASS>(reinterpret_cast<f32x4*>(sse_out + c0 * 4) + tid, f32x4{o.sse[0], o.sse[1], o.sse[2], o.sse[3]}, flags);
            if (clip_out)
                reinterpret_cast<float4*>(clip_out + c0 * 4)[tid] =
                    make_float4(o.clip[0], o.clip[1], o.clip[2], o.clip[3]);
        }
    }
}

// Where the block SSEs of a complete slice go.
enum : int { kNoSse = 0, kSseCached = 1, kSsePast = 2 };

// Stores of one slice of 256 complete chunks.  Every lane of a block stores the block's scale byte and SSE to the same
// place: without masks and branches the compiler can count the stores that lie behind a load.  They are the same values
// but for an SSE that is NaN (a block with a NaN or an infinity), of which each lane may hold another sign and payload.
template <int B, int SSE>
__device__ __forceinline__ void store_complete_slice(const TileOut<B>& o, uint32_t s, uint32_t* __restrict__ codes,
                                                     uint8_t* __restrict__ scales, float* __restrict__ sse_out)
{
    constexpr int NBLK = TileOut<B>::NBLK;
    constexpr int LANES = (B < 8) ? 1 : B / 8;
    const uint32_t tid = threadIdx.x;
    const uint64_t c0 = (uint64_t)s * kThreads;                      // first chunk of the slice
    const auto store = [](auto* p, auto v) {
        if constexpr (SSE == kSsePast) __builtin_nontemporal_store(v, p);
        else if constexpr (SSE == kSseCached) *p = v;
    };
    __builtin_nontemporal_store(o.packed, codes + c0 + tid);
    if constexpr (B >= 8) {
        (scales + c0 / LANES)[tid / LANES] = (uint8_t)o.code[0];
        store((sse_out + c0 / LANES) + tid / LANES, o.sse[0]);
    } else if constexpr (NBLK == 2) {
        reinterpret_cast<uint16_t*>(scales + c0 * 2)[tid] = (uint16_t)(o.code[0] | (o.code[1] << 8));
        store(reinterpret_cast<f32x2*>(sse_out + c0 * 2) + tid, f32x2{o.sse[0], o.sse[1]});
    } else {
        reinterpret_cast<uint32_t*>(scales + c0 * 4)[tid] = o.code[0] | (o.code[1] << 8) | (o.code[2] << 16) | (o.code[3] << 24);
        store(reinterpret_cast<f32x4*>(sse_out + c0 * 4) + tid, f32x4{o.sse[0], o.sse[1], o.sse[2], o.sse[3]});
    }
}

// Scale table of a kernel.  One truncated product does for bf16 values that nothing has divided (8 significant
// bits); fp32 values and quotients by a tensor scale have 24 and need both parts.
template <int DT, int TMODE>
using TableEntry = std::conditional_t<DT == kBF16 && TMODE == kNoT, ScalePair, ScaleEntry>;

// Whether a kernel forms its table or copies it (fill_scale_table).
template <int DT, int TMODE>
constexpr bool kFormTable = DT == kF32 || TMODE == kNoT;

// A workgroup tile is kItems consecutive slices; every lane owns one chunk of each slice.
constexpr int kItems = MXQ_STREAM_ITEMS;

template <int DT>
__device__ __forceinline__ void load_tile(RawChunk<DT> (&buf)[kItems], const void* __restrict__ x,
                                          uint32_t s0, Slices sl)
{
    constexpr uint64_t kVecPerChunk = (DT == kBF16) ? 1 : 2;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t s = s0 + (uint32_t)i;
        if (s < sl.count) {                                          // uniform
            buf[i] = load_raw<DT>(static_cast<const u32x4*>(x) + (uint64_t)s * kThreads * kVecPerChunk,
                                  (uint32_t)threadIdx.x, sl.chunks(s));
        }
    }
}

// One step of the software pipeline for the tile at slice s0 whose raw data sits in `cur`:
//   wait until `cur` has landed -> issue the stores of the PREVIOUS tile -> issue the loads of
//   the NEXT tile into `nxt` -> quantise `cur` into `out`.
// On gfx9 loads and stores share one in-order counter, so the wait at the top covers every
// memory operation still in flight; with this order all of them were issued a whole compute
// phase earlier and the wait is short.
template <int DT, int B, int FMT, bool FOUR6, int TMODE, bool CLIP, class Entry>
__device__ __forceinline__ void stream_step(RawChunk<DT> (&cur)[kItems], RawChunk<DT> (&nxt)[kItems],
                                            TileOut<B> (&out)[kItems], bool have_prev, uint32_t s_prev,
                                            const void* __restrict__ x, uint32_t s0, uint32_t stride,
                                            Slices sl, float T, float rT, int tdyn, int flags, const Entry* tab,
                                            u32x4* wave_lds, uint32_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                            float* __restrict__ sse_out, float* __restrict__ clip_out, uint32_t& largest_sse)
{
    float v[kItems][8];
    __builtin_amdgcn_s_waitcnt(0x0F70);                              // vmcnt(0)
#pragma unroll
    for (int i = 0; i < kItems; ++i) widen<DT>(cur[i], v[i], wave_lds);
    __builtin_amdgcn_sched_barrier(0);
    if (have_prev) {                                                 // uniform
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            store_slice<B, kMayPass<DT, B, FOUR6, TMODE, CLIP>>(out[i], s_prev + (uint32_t)i, sl, flags, codes, scales, sse_out, CLIP ? clip_out : nullptr);
    }
    if (s0 + stride < sl.count) load_tile<DT>(nxt, x, s0 + stride, sl);            // uniform
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        process_chunk<B, FMT, FOUR6, TMODE, CLIP>(v[i], T, rT, tdyn, (flags & kPreventZero) != 0, tab, out[i].packed, out[i].code, out[i].sse,
                                                  out[i].clip);
    if constexpr (TMODE == kLeanT) {
#pragma unroll
        for (int i = 0; i < kItems; ++i)
#pragma unroll
            for (int k = 0; k < TileOut<B>::NBLK; ++k) largest_sse = max(largest_sse, f2u(out[i].sse[k]));
    }
}

// Ragged tail: when n is not a multiple of 8 (only possible for b = 2 or 4) the last `count` < 8
// elements are handled by one lane of an extra workgroup of the same launch, reading and writing
// element-wise.  (A launch of its own, as it was, cost more than it does on any tensor that fits in a
// few microseconds: 2563 x 4110 elements, b = 2, 18.4 us against 14.9 us for 2563 x 4112.)
template <int DT, int B, int FMT, bool FOUR6, int TMODE, bool CLIP, class Entry>
__device__ __forceinline__ void stream_tail(const void* __restrict__ x, uint64_t first, uint32_t count, float T, float rT,
                                            int tdyn, bool pz, const Entry* tab, uint8_t* __restrict__ codes,
                                            uint8_t* __restrict__ scales, float* __restrict__ sse_out,
                                            float* __restrict__ clip_out)
{
    if (threadIdx.x >= 64u) return;                                  // one wavefront, its first lane stores
    TileOut<B> o;
    float v[8];
    load_partial<DT>(x, (int64_t)first, (threadIdx.x == 0) ? (int)count : 0, v);
    process_chunk<B, FMT, FOUR6, TMODE, CLIP>(v, T, rT, tdyn, pz, tab, o.packed, o.code, o.sse, o.clip);
    if (threadIdx.x != 0) return;
    for (uint32_t i = 0; i < count / 2u; ++i) codes[first / 2u + i] = (uint8_t)(o.packed >> (8u * i));
    for (uint32_t k = 0; k < (uint32_t)TileOut<B>::NBLK; ++k) {
        if (k < count / (uint32_t)B) {
            scales[first / B + k] = (uint8_t)o.code[k];
            if (sse_out) sse_out[first / B + k] = o.sse[k];
            if constexpr (CLIP) { if (clip_out) clip_out[first / B + k] = o.clip[k]; }
        }
    }
}

// The complete chunks of one workgroup, grid-stride over workgroup tiles with two register buffers
// alternating between "being processed" and "in flight"; bufA holds the first tile's loads.  With kLeanT the
// bits of the largest block SSE that the lane has seen come back (a NaN is above all others).
template <int DT, int B, int FMT, bool FOUR6, int TMODE, bool CLIP, class Entry>
__device__ __forceinline__ uint32_t stream_tiles(RawChunk<DT> (&bufA)[kItems], const void* __restrict__ x, uint32_t s0,
                                             uint32_t stride, Slices sl, float T, float rT, int tdyn, int flags, const Entry* tab,
                                             u32x4* wave_lds, uint32_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                             float* __restrict__ sse_out, float* __restrict__ clip_out)
{
    RawChunk<DT> bufB[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) bufB[i] = RawChunk<DT>{};
    TileOut<B> out[kItems];
    bool have_prev = false;
    uint32_t s_prev = s0, largest_sse = 0u;
    while (true) {
        stream_step<DT, B, FMT, FOUR6, TMODE, CLIP>(bufA, bufB, out, have_prev, s_prev, x, s0, stride, sl, T, rT, tdyn,
                                                    flags, tab, wave_lds, codes, scales, sse_out, clip_out, largest_sse);
        have_prev = true;
        s_prev = s0;
        s0 += stride;
        if (s0 >= sl.count) break;
        stream_step<DT, B, FMT, FOUR6, TMODE, CLIP>(bufB, bufA, out, true, s_prev, x, s0, stride, sl, T, rT, tdyn,
                                                    flags, tab, wave_lds, codes, scales, sse_out, clip_out, largest_sse);
        s_prev = s0;
        s0 += stride;
        if (s0 >= sl.count) break;
    }
#pragma unroll
    for (int i = 0; i < kItems; ++i)
        store_slice<B, kMayPass<DT, B, FOUR6, TMODE, CLIP>>(out[i], s_prev + (uint32_t)i, sl, flags, codes, scales, sse_out, CLIP ? clip_out : nullptr);
    return largest_sse;
}

// ---------------------------------------------------------------------------------------
// Large tensors without a per-tensor scale in device memory: a workgroup takes kOnce consecutive slices and ends.  All
// its loads are in flight before the first slice is quantised, a slice waits for its own load only, and the next
// workgroup's loads start when this one's last stores do.  Bound by HBM (4-over-6: vector issue beside it).  In the loop
// of stream_kernel a wavefront has one tile's loads in flight, and none while it waits for them and the stores before.
// Loop -> two / three / four slices: 4096 x 14336 bf16 abs-max b = 16 28.4 -> 27.3 / 26.6 / 27.6 us, 4-over-6 b = 8 31.3 -> 29.7
// / 29.4 / 30.6, b = 32 28.6 -> 26.2 / 26.0 / 26.7, b = 2 48.1 -> 46.0 / 46.2 / 46.3; fp32 b = 16 49.5 -> 46.0 / 46.2 / 47.3;
// a batch of 218 M elements, 4-over-6 b = 32 112.8 -> 103.4 / 97.8 / 96.7 (5.1 -> 5.9 TB/s).  A tensor of fewer slices has too
// few workgroups for their phases to overlap: 4096 x 4096 (8192 slices) bf16 abs-max b = 16 8.3 -> 8.9, 2563 x 4110 b = 2 12.1 ->
// 12.5; 6000 x 4096 (11719) 13.4 -> 13.5; 8192 x 4096 (16384) 4-over-6 b = 16 16.6 -> 16.5, b = 4 22.8 -> 21.4, abs-max 16.7 ->
// 16.2.  fp32 has its line there too, and T by value (four recipes and formats, b = 2 .. 128, three slices against the loop):
// 4096 slices 0.93 to 1.08 of the loop's time, 1.03 in the mean; 8192 0.92 to 1.06, 1.01; 12288 0.96 to 1.03, 0.99; 16383 0.91 to
// 0.99, 0.96.  58.7 M elements, fp32 abs-max b = 16 T = 1 51.8 -> 48.0, T by value 51.7 -> 48.4, 4-over-6 b = 8 T by value 55.8 ->
// 51.9; bf16 abs-max T by value b = 8 33.8 -> 32.1, b = 2 58.3 -> 55.1.  Behind an abs-max pass (T in device memory) the loop's order of the slices finds more in the caches: 8192 x 4096
// abs-max and quantise, b = 16, 26.2 -> 29.7.
// ---------------------------------------------------------------------------------------
constexpr int kOnce = 3;
constexpr int64_t kOnceFrom = 16384;                                 // slices
constexpr int64_t kOnceMost = (int64_t)1 << 25;                      // a grid counts fewer than 2^32 threads

// The kOnce slices from s0 on; slices beyond the last are read as the last.
template <int DT>
__device__ __forceinline__ void load_once(RawChunk<DT> (&raw)[kOnce], const void* __restrict__ x, uint32_t s0, Slices sl)
{
    constexpr uint64_t kVecPerChunk = (DT == kBF16) ? 1 : 2;
#pragma unroll
    for (int i = 0; i < kOnce; ++i) {
        const uint32_t s = min(s0 + (uint32_t)i, sl.count - 1u);     // uniform
        raw[i] = load_raw<DT>(static_cast<const u32x4*>(x) + (uint64_t)s * kThreads * kVecPerChunk, (uint32_t)threadIdx.x, sl.chunks(s));
    }
}

template <int DT, int B, int FMT, bool FOUR6, int TMODE, class Entry>
__device__ __forceinline__ void once_slices(const RawChunk<DT> (&raw)[kOnce], uint32_t s0, Slices sl, float T, float rT, int flags,
                                            const Entry* tab, u32x4* wave_lds, uint32_t* __restrict__ codes,
                                            uint8_t* __restrict__ scales, float* __restrict__ sse_out)
{
    constexpr bool kPass = kMayPass<DT, B, FOUR6, TMODE, false>;
    const auto slices = [&](auto store) {
#pragma unroll
        for (int i = 0; i < kOnce; ++i) {
            float v[8];
            widen<DT>(raw[i], v, wave_lds);
            TileOut<B> o;
            process_chunk<B, FMT, FOUR6, TMODE, false>(v, T, rT, TMODE, (flags & kPreventZero) != 0, tab, o.packed, o.code, o.sse, o.clip);
            store(o, s0 + (uint32_t)i);
            __builtin_amdgcn_sched_barrier(0);                       // one slice at a time: registers
        }
    };
    if (s0 + (uint32_t)kOnce >= sl.count)                            // uniform; the last slices of the tensor
        slices([&](const TileOut<B>& o, uint32_t s) { store_slice<B, kPass>(o, s, sl, flags, codes, scales, sse_out, nullptr); });
    else if (!sse_out)
        slices([&](const TileOut<B>& o, uint32_t s) { store_complete_slice<B, kNoSse>(o, s, codes, scales, nullptr); });
    else if (kPass && (flags & kSsePastCaches))
        slices([&](const TileOut<B>& o, uint32_t s) { store_complete_slice<B, kPass ? kSsePast : kSseCached>(o, s, codes, scales, sse_out); });
    else
        slices([&](const TileOut<B>& o, uint32_t s) { store_complete_slice<B, kSseCached>(o, s, codes, scales, sse_out); });
}

// The first `tiles` workgroups take the slices; one more, where there is one, takes the ragged tail.
template <int DT, int B, int FMT, bool FOUR6, int TMODE>
__global__ void __launch_bounds__(kThreads)
stream_once_kernel(const void* __restrict__ x, uint32_t n_slices, uint32_t last_chunks, uint32_t tail, float T, int flags,
                   uint32_t tiles, uint32_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ sse_out)
{
    static_assert(TMODE == kNoT || TMODE == kFastT, "T by value");
    using Entry = TableEntry<DT, TMODE>;
    __shared__ Entry tab[(FMT == kE8M0) ? 1 : 256];
    __shared__ u32x4 xpose[(DT == kF32) ? 2 * kThreads : 1];        // 2 KiB per wavefront, fp32 input only
    u32x4* wave_lds = xpose + ((DT == kF32) ? 2u * (threadIdx.x & ~63u) : 0u);

    const Slices sl{n_slices, last_chunks};
    const uint32_t s0 = blockIdx.x * (uint32_t)kOnce;
    RawChunk<DT> raw[kOnce];
    load_once<DT>(raw, x, s0, sl);                                   // in flight while the scale table is built
    const float rT = 1.0f / T;                                       // correctly rounded
    if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, TMODE>>(tab);
    if constexpr (B < 8) {
        if (blockIdx.x == tiles) {
            stream_tail<DT, B, FMT, FOUR6, TMODE, false>(x, sl.elements(), tail, T, rT, TMODE, (flags & kPreventZero) != 0, tab,
                                                         reinterpret_cast<uint8_t*>(codes), scales, sse_out, nullptr);
            return;
        }
    }
    once_slices<DT, B, FMT, FOUR6, TMODE>(raw, s0, sl, T, rT, flags, tab, wave_lds, codes, scales, sse_out);
}

// Main kernel.  The number of workgroups without the one for the tail is an argument: the launch's own count lies in
// another cache line of the arguments than the rest, and where the compiler asks for it before the first loads, those wait
// for it.  Count of the launch -> argument, abs-max b = 16: 512 x 4096 bf16 3.33 -> 3.08 us, fp32 3.92 -> 3.67; 1024 x 4096
// 4.06 -> 3.75, 5.32 -> 5.11; 4096 x 4096 9.25 -> 9.02, 14.6 -> 14.5.
template <int DT, int B, int FMT, bool FOUR6, int TMODE, bool CLIP>
__device__ __forceinline__ void stream_body(const void* __restrict__ x, uint32_t n_slices, uint32_t last_chunks, uint32_t tail, float T_arg,
                                            int flags, uint32_t workers, const float* __restrict__ absmax_dev,
                                            float* __restrict__ t_out, uint32_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                            float* __restrict__ sse_out, float* __restrict__ clip_out)
{
    using Entry = TableEntry<DT, TMODE>;
    __shared__ Entry tab[(FMT == kE8M0) ? 1 : 256];
    __shared__ u32x4 xpose[(DT == kF32) ? 2 * kThreads : 1];        // 2 KiB per wavefront, fp32 input only
    u32x4* wave_lds = xpose + ((DT == kF32) ? 2u * (threadIdx.x & ~63u) : 0u);

    const Slices sl{n_slices, last_chunks};
    const uint32_t stride = workers * (uint32_t)kItems;
    const uint32_t s0 = blockIdx.x * (uint32_t)kItems;
    float T = T_arg;
    int tdyn = TMODE;
    if constexpr (TMODE == kDynT) {                  // T from the abs-max left in device memory, if there is one
        if (absmax_dev) T = tensor_scale_of<FMT>(*absmax_dev);
        tdyn = (T == 1.0f) ? kNoT : (fast_division_ok(T) ? kFastT : kSlowT);
        if (t_out && blockIdx.x == 0 && threadIdx.x == 0) *t_out = T;
    }
    const float rT = 1.0f / T;                                       // correctly rounded
    if constexpr (B < 8) {
        if (tail != 0u && blockIdx.x == workers) {
            if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, TMODE>>(tab);
            stream_tail<DT, B, FMT, FOUR6, TMODE, CLIP>(x, sl.elements(), tail, T, rT, tdyn, (flags & kPreventZero) != 0, tab,
                                                        reinterpret_cast<uint8_t*>(codes), scales, sse_out, clip_out);
            return;
        }
    }
    if (s0 >= sl.count) return;                                      // whole workgroup

    RawChunk<DT> first[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) first[i] = RawChunk<DT>{};
    load_tile<DT>(first, x, s0, sl);                                 // in flight while the scale table is built
    if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, TMODE>>(tab);
    stream_tiles<DT, B, FMT, FOUR6, TMODE, CLIP>(first, x, s0, stride, sl, T, rT, tdyn, flags, tab, wave_lds, codes, scales,
                                                 sse_out, clip_out);
}

// Arguments of a launch as one: the host spends 0.05 us on each argument, 0.6 of the 3.3 us of a launch with thirteen, and small
// calls take as long as the host does.
struct StreamKernelArgs {
    const void* x;
    uint32_t n_slices, last_chunks, tail;
    float T;
    int flags;
    uint32_t workers;
    const float* absmax_dev;
    float* t_out;
    uint32_t* codes;
    uint8_t* scales;
    float* sse;
    float* clip;
};

template <int DT, int B, int FMT, bool FOUR6, int TMODE, bool CLIP>
__global__ void __launch_bounds__(kThreads)
stream_kernel(const StreamKernelArgs a)
{
    stream_body<DT, B, FMT, FOUR6, TMODE, CLIP>(a.x, a.n_slices, a.last_chunks, a.tail, a.T, a.flags, a.workers, a.absmax_dev, a.t_out,
                                                a.codes, a.scales, a.sse, a.clip);
}

// bf16 under a tensor scale, T by value or from the abs-max in device memory, for tensors of several tiles a
// workgroup: 29 vector instructions of 160 a chunk (4-over-6) go where lean_T finds the shorter sequences exact
// for this T.  Every wavefront finds that out by itself in some 45 instructions.  The other T's (four of the 128 that
// a bf16 abs-max gives) go the general way, 4-over-6 with b = 2 in a plain loop, whose registers are few, without
// prefetch.  General kernel -> this one for such a T: 2048 x 4096 4-over-6 b = 16 7.00 -> 7.24 us, b = 64 7.02 -> 7.53;
// 4096 x 4096 4-over-6 b = 16 12.1 -> 12.1, abs-max 9.9 -> 10.1; 8192 x 4096 4-over-6 b = 16 22.2 -> 21.5, abs-max 17.6
// -> 17.9; 4-over-6 b = 2 33.9 -> 36.8.  (With the first tile loaded a second time 7.60, 7.87, 12.5, 10.5, 21.8, 18.3.)
// General kernel -> this one, T from device memory, E4M3: 8192 x 4096 4-over-6 b = 16 22.1 -> 20.5 us, b = 64 22.3
// -> 20.5, b = 4 26.6 -> 24.2, b = 2 33.2 -> 32.1, abs-max b = 16 18.3 -> 17.9; 14336 x 4096 4-over-6 b = 16 35.6 -> 32.6.
// With fewer tiles a workgroup than these the test of T costs what it saves (two tiles, 2048 x 4096: 4-over-6
// b = 16, T from the device 7.3 -> 7.1 us, by value b = 4 8.6 -> 9.2, abs-max b = 16 6.2 -> 6.7).  The abs-max recipes
// with b < 16 are bound by memory, and by value, where no wavefront has to derive T, they are 1 to 2 % faster
// in the general kernel while that has the short division.
constexpr int64_t kScaledTiles = 4, kScaledTilesFour6 = 2, kScaledTilesFour6ByValue = 3;
template <int B, bool FOUR6>
static bool takes_scaled_kernel(const StreamArgs& a, int64_t slices, int64_t workers)
{
    if (a.clip || slices == 0) return false;
    if (a.absmax_dev) return slices >= (FOUR6 ? kScaledTilesFour6 : kScaledTiles) * workers;
    if (a.T == 1.0f || !lean_T_in_range(a.T)) return false;
    if (!FOUR6 && B < 16 && fast_division_ok(a.T)) return false;
    return slices >= (FOUR6 ? kScaledTilesFour6ByValue : kScaledTiles) * workers;
}

// The wavefront's chunks the general way in a plain loop: few registers, no prefetch, and no barrier with a table in memory.
template <int B, int FMT, bool FOUR6>
__device__ __forceinline__ void general_tiles(const void* __restrict__ x, uint32_t s0, uint32_t stride, Slices sl, float T, float rT,
                                              int tdyn, int flags, const ScaleEntry* tab, uint32_t* __restrict__ codes,
                                              uint8_t* __restrict__ scales, float* __restrict__ sse_out)
{
#pragma unroll 1
    for (; s0 < sl.count; s0 += stride) {                            // uniform
        RawChunk<kBF16> raw[kItems];
        load_tile<kBF16>(raw, x, s0, sl);
        float v[8];
        widen<kBF16>(raw[0], v, nullptr);
        TileOut<B> o;
        process_chunk<B, FMT, FOUR6, kDynT, false>(v, T, rT, tdyn, (flags & kPreventZero) != 0, tab, o.packed, o.code, o.sse, o.clip);
        store_slice<B, kMayPass<kBF16, B, FOUR6, kDynT, false>>(o, s0, sl, flags, codes, scales, sse_out, nullptr);
    }
}

template <int B, int FMT, bool FOUR6>
__global__ void __launch_bounds__(kThreads)
stream_scaled_kernel(const void* __restrict__ x, uint32_t n_slices, uint32_t last_chunks, uint32_t tail, float T_arg, int flags,
                     uint32_t stride, const float* __restrict__ absmax_dev, float* __restrict__ t_out,
                     uint32_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ sse_out)
{
    static_assert(FMT != kE8M0 && kItems == 1, "scales from a table, one slice per tile");
    __shared__ ScaleEntry tab[256];
    __shared__ uint32_t again;
    const Slices sl{n_slices, last_chunks};
    const uint32_t s0 = blockIdx.x;
    // The first tile's loads are in flight while T is looked at, and both parts of 1/T live in vector registers
    // (an instruction with a scalar operand costs more): not where the 64 registers that eight wavefronts a
    // SIMD leave for each do not hold them.
    constexpr bool kEarly = !(B == 2 && FOUR6);
    RawChunk<kBF16> first[kItems];
    if constexpr (kEarly) first[0] = RawChunk<kBF16>{};
    if (kEarly && s0 < stride) load_tile<kBF16>(first, x, s0, sl);
    const LeanPair pair = kLeanPairs.of[threadIdx.x & 31u];
    if constexpr (kEarly) __builtin_amdgcn_sched_barrier(0);
    float T = T_arg;
    if (absmax_dev) T = tensor_scale_of<FMT>(*absmax_dev);
    if (t_out && blockIdx.x == 0 && threadIdx.x == 0) *t_out = T;
    const float rT = 1.0f / T;                                       // correctly rounded
    const int tdyn = (T == 1.0f) ? kNoT : (fast_division_ok(T) ? kFastT : kSlowT);
    Recip r = lean_recip(T);
    uint32_t above = 0u;
    if (s0 < stride && lean_T_in_range(T) && lean_T(pair, T, rT, r, above)) {     // uniform: every wavefront finds the same
        if constexpr (!kEarly) load_tile<kBF16>(first, x, s0, sl);
        ScalePair* pairs = reinterpret_cast<ScalePair*>(tab);
        if constexpr (!kEarly) again = 0u;
        fill_scale_table<FMT>(pairs, above);
        if constexpr (kEarly) {
            asm volatile("" : "+v"(r.hi), "+v"(r.lo));
        } else {
            r.hi = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)f2u(r.hi)));
            r.lo = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)f2u(r.lo)));
        }
        const uint32_t largest_sse =
            stream_tiles<kBF16, B, FMT, FOUR6, kLeanT, false>(first, x, s0, stride, sl, r.hi, r.lo, kLeanT, flags, pairs,
                                                              (u32x4*)nullptr, codes, scales, sse_out, (float*)nullptr);
        // An element that is not finite, or is not any more after the division, leaves such an SSE, and the general way
        // may see it otherwise (div_by_T makes a NaN of an infinity, with a sign of its own): the wavefront goes that way
        // too, so that the outputs of a row do not depend on the size of its tensor.  (The whole workgroup, with a
        // barrier, takes 1 to 2 % longer on all tensors: 8192 x 4096 4-over-6 b = 16 20.1 us against 19.7, 14336 x 4096 32.5
        // against 31.7.  With b = 2 it saves the registers of a second copy of the code.)
        const bool bad = __builtin_amdgcn_ballot_w64(largest_sse >= 0x7F800000u) != 0ull;
        if constexpr (kEarly) {
            if (bad)                                                 // rare
                general_tiles<B, FMT, FOUR6>(x, s0, stride, sl, T, rT, tdyn, flags, kScaleTable<FMT, ScaleEntry>.of, codes, scales, sse_out);
            return;
        }
        if (bad) again = 1u;
        __syncthreads();
        if (again == 0u) return;                                     // uniform
    }
    fill_scale_table<FMT, kFormTable<kBF16, kDynT>>(tab);
    if constexpr (B < 8) {
        if (s0 == stride) {
            stream_tail<kBF16, B, FMT, FOUR6, kDynT, false>(x, sl.elements(), tail, T, rT, tdyn, (flags & kPreventZero) != 0, tab,
                                                            reinterpret_cast<uint8_t*>(codes), scales, sse_out, nullptr);
            return;
        }
    }
    if constexpr (kEarly)
        stream_tiles<kBF16, B, FMT, FOUR6, kDynT, false>(first, x, s0, stride, sl, T, rT, tdyn, flags, tab, (u32x4*)nullptr,
                                                         codes, scales, sse_out, (float*)nullptr);
    else
        general_tiles<B, FMT, FOUR6>(x, s0, stride, sl, T, rT, tdyn, flags, tab, codes, scales, sse_out);
}

// ---------------------------------------------------------------------------------------
// Several tensors in one launch.  A model's smaller matrices hold a few microseconds of work each,
// less than the start-up and drain of a launch; here up to kMaxBatch tensors share one grid.  The
// slices of all tensors form one index space (prefix sums in the kernel arguments); a workgroup
// resolves every tile to its tensor with a handful of scalar compares and then runs the very same
// pipeline step as the single-tensor kernel.  No per-tensor scale, no clipping output.
// ---------------------------------------------------------------------------------------
struct BatchArgs {
    const void* x[kMaxBatch];
    uint32_t* codes[kMaxBatch];
    uint8_t* scales[kMaxBatch];
    float* sse[kMaxBatch];
    uint32_t first[kMaxBatch + 1];        // first global slice (tile of kOnce slices) of tensor t; first[count] = total
    uint32_t slices[kMaxBatch];
    uint32_t last[kMaxBatch];             // chunks in tensor t's last slice, 1 .. 256
    uint32_t tail[kMaxBatch];             // elements behind the complete chunks, 0 .. 7 (b = 2, 4)
    uint32_t count;
    uint32_t workers;                     // workgroups that share the slices; those behind them, one per tensor, take the tails
};

struct TileRef {                          // one tile = one slice of one tensor
    uint32_t t, s;                        // tensor, slice inside it
    Slices sl;
};

__device__ __forceinline__ TileRef locate(const BatchArgs& a, uint32_t g)
{
    uint32_t t = 0u;
#pragma unroll
    for (int k = 1; k < kMaxBatch; ++k) t += ((uint32_t)k < a.count && g >= a.first[k]) ? 1u : 0u;
    return TileRef{t, g - a.first[t], Slices{a.first[t + 1] - a.first[t], a.last[t]}};
}

template <int DT, int B, int FMT, bool FOUR6, class Entry>
__device__ __forceinline__ void batch_step(RawChunk<DT> (&cur)[kItems], RawChunk<DT> (&nxt)[kItems],
                                           TileOut<B> (&out)[kItems], bool have_prev, TileRef prev,
                                           bool have_next, TileRef next, const BatchArgs& a, int flags,
                                           const Entry* tab, u32x4* wave_lds)
{
    static_assert(kItems == 1, "one slice per tile");
    float v[8];
    __builtin_amdgcn_s_waitcnt(0x0F70);                              // vmcnt(0)
    widen<DT>(cur[0], v, wave_lds);
    __builtin_amdgcn_sched_barrier(0);
    if (have_prev)                                                   // uniform
        store_slice<B, kMayPass<DT, B, FOUR6, kNoT, false>>(out[0], prev.s, prev.sl, flags, a.codes[prev.t], a.scales[prev.t], a.sse[prev.t], nullptr);
    if (have_next) load_tile<DT>(nxt, a.x[next.t], next.s, next.sl); // uniform
    __builtin_amdgcn_sched_barrier(0);
    process_chunk<B, FMT, FOUR6, kNoT, false>(v, 1.0f, 1.0f, kNoT, (flags & kPreventZero) != 0, tab, out[0].packed, out[0].code, out[0].sse,
                                              out[0].clip);
}

// (Resolving the descriptors of a tile one pipeline step ahead, pointers included, was measured
// and is slower: it keeps three sets of pointers alive in scalar registers.)
template <int DT, int B, int FMT, bool FOUR6>
__global__ void __launch_bounds__(kThreads)
stream_batch_kernel(const BatchArgs a, int flags)
{
    using Entry = TableEntry<DT, kNoT>;
    __shared__ Entry tab[(FMT == kE8M0) ? 1 : 256];
    __shared__ u32x4 xpose[(DT == kF32) ? 2 * kThreads : 1];
    u32x4* wave_lds = xpose + ((DT == kF32) ? 2u * (threadIdx.x & ~63u) : 0u);

    const uint32_t total = a.first[a.count];
    const uint32_t stride = a.workers;
    uint32_t g = blockIdx.x;
    if constexpr (B < 8) {
        if (g >= stride) {
            const uint32_t t = g - stride;
            if (a.tail[t] == 0u) return;
            if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, kNoT>>(tab);
            stream_tail<DT, B, FMT, FOUR6, kNoT, false>(a.x[t], Slices{a.first[t + 1] - a.first[t], a.last[t]}.elements(),
                                                        a.tail[t], 1.0f, 1.0f, kNoT, (flags & kPreventZero) != 0, tab,
                                                        reinterpret_cast<uint8_t*>(a.codes[t]), a.scales[t], a.sse[t], nullptr);
            return;
        }
    }
    if (g >= total) return;                                          // whole workgroup

    RawChunk<DT> bufA[kItems], bufB[kItems];
    bufA[0] = RawChunk<DT>{};
    bufB[0] = RawChunk<DT>{};
    TileRef cur = locate(a, g), prev = cur, next = cur;
    load_tile<DT>(bufA, a.x[cur.t], cur.s, cur.sl);
    if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, kNoT>>(tab);
    TileOut<B> out[kItems];
    bool have_prev = false;
    while (true) {
        bool have_next = g + stride < total;
        if (have_next) next = locate(a, g + stride);
        batch_step<DT, B, FMT, FOUR6>(bufA, bufB, out, have_prev, prev, have_next, next, a, flags, tab, wave_lds);
        have_prev = true;
        prev = cur;
        if (!have_next) break;
        cur = next;
        g += stride;
        have_next = g + stride < total;
        if (have_next) next = locate(a, g + stride);
        batch_step<DT, B, FMT, FOUR6>(bufB, bufA, out, true, prev, have_next, next, a, flags, tab, wave_lds);
        prev = cur;
        if (!have_next) break;
        cur = next;
        g += stride;
    }
    store_slice<B, kMayPass<DT, B, FOUR6, kNoT, false>>(out[0], prev.s, prev.sl, flags, a.codes[prev.t], a.scales[prev.t], a.sse[prev.t], nullptr);
}

// The same with kOnce consecutive slices of one tensor to a workgroup: first[] counts such tiles, and the slices of a
// tensor follow from its own count.
template <int DT, int B, int FMT, bool FOUR6>
__global__ void __launch_bounds__(kThreads)
stream_batch_once_kernel(const BatchArgs a, int flags)
{
    using Entry = TableEntry<DT, kNoT>;
    __shared__ Entry tab[(FMT == kE8M0) ? 1 : 256];
    __shared__ u32x4 xpose[(DT == kF32) ? 2 * kThreads : 1];
    u32x4* wave_lds = xpose + ((DT == kF32) ? 2u * (threadIdx.x & ~63u) : 0u);

    const uint32_t g = blockIdx.x;
    if constexpr (B < 8) {
        if (g >= a.workers) {
            const uint32_t t = g - a.workers;
            if (a.tail[t] == 0u) return;
            if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, kNoT>>(tab);
            stream_tail<DT, B, FMT, FOUR6, kNoT, false>(a.x[t], Slices{a.slices[t], a.last[t]}.elements(), a.tail[t], 1.0f, 1.0f, kNoT,
                                                        (flags & kPreventZero) != 0, tab, reinterpret_cast<uint8_t*>(a.codes[t]),
                                                        a.scales[t], a.sse[t], nullptr);
            return;
        }
    }
    uint32_t t = 0u;
#pragma unroll
    for (int k = 1; k < kMaxBatch; ++k) t += ((uint32_t)k < a.count && g >= a.first[k]) ? 1u : 0u;
    const Slices sl{a.slices[t], a.last[t]};
    const uint32_t s0 = (g - a.first[t]) * (uint32_t)kOnce;
    RawChunk<DT> raw[kOnce];
    load_once<DT>(raw, a.x[t], s0, sl);
    if constexpr (FMT != kE8M0) fill_scale_table<FMT, kFormTable<DT, kNoT>>(tab);
    once_slices<DT, B, FMT, FOUR6, kNoT>(raw, s0, sl, 1.0f, 1.0f, flags, tab, wave_lds, a.codes[t], a.scales[t], a.sse[t]);
}

// ------------------------------------------------------------------------------ dispatch

// Where the block SSEs are written past the caches: bf16, up to 15 MiB of them from an input of up to 128 MiB; with 4-over-6 or
// b = 2 from 6 MiB on; where T comes from the abs-max in device memory, from 8 MiB on (4-over-6 4).  The lines are drawn
// by the call alone and by the call with a reader of the SSEs behind it (a tensor MSE is usually next), each with four
// sets of outputs in turn and with one set re-used; a hierarchical call has its abs-max pass in front each time.  Without
// the reader it has to gain, and with it the whole must not lose.  Ordinary -> past the caches in per cent, E4M3, four
// inputs in turn, in the order alone, alone re-used, with reader, with reader re-used:
//   4-over-6 b = 16   2 MiB -3 -3 +5 +5    4 MiB -3 -3 +3 -1    6 MiB -5 -3 +3 -5    8 MiB -5 -3  0 -5   12 MiB -4 -4 -1 -3
//                    14 MiB -2 -3  0 -1   15 MiB -2 -2  0 +2   18 MiB -1  0 +2 +2   24 MiB +1 +2 +3 +3
//            b = 8    4 MiB -2 -5 +6 -3    8 MiB -5 -6 +2 -7   12 MiB -2 -2 +4 -7   18 MiB +2 +1 +8 +4
//            b = 4    6 MiB -13 -15 0 -9   8 MiB -11 -11 0 -11 12 MiB -4 -3 +5 -14  20 MiB +2 +1 +9 +2
//            b = 2    4 MiB  0  0  0 +9    8 MiB -8 -9 -2 -6   12 MiB -18 -17 -6 -7 24 MiB -2 -1 +6 +10
//            b = 32   4 MiB -3  0 +1  0    7 MiB -2 -3  0 -1    8 MiB -3 -3 +1 +1
//   abs-max  b = 16   4 MiB +1  0 +5 +2    8 MiB -4 -4 +1 -3   12 MiB -1 -2 +2 -1   14 MiB  0 -1 +3 +2
//            b = 8    4 MiB  0  0 +9 +7    8 MiB -2 -3 +5 -5   14 MiB +1  0 +5 -4
//            b = 2    8 MiB -9 -7 +1 -2   12 MiB -14 -15 0 -3
//   powers of two b = 16  4 MiB -1 -1 +4 +2   8 MiB -3 -3 +2 -2   14 MiB -1 -2 +2 +2
//   fp32     b = 16   2 MiB  0  0 +5 +6    8 MiB -1 -1 +2 +2;  b = 8  2 MiB +2 +4 +9 +11   8 MiB -1 -3 +4  0
// Batches follow their sum (4-over-6 b = 16: 8 MiB -5 -5 -1 -7, 14 MiB -3 -2 0 -1, 20 MiB 0 -2 +2 +1).
// With the abs-max pass, T from device memory:
//   abs-max  b = 4    8 MiB -7 -7 -2 -9    b = 8    4 MiB -4 -4 +3  0    8 MiB -5 -5 -1 -2
//            b = 16   2 MiB -2 -2 +3 +2    4 MiB -2 -2 +3 +2    8 MiB -1 -1 +1 +1   14 MiB -2 -2  0  0
//            b = 32   4 MiB  0 -1 +2 +3    7 MiB +1  0 +2 +2
//   4-over-6 b = 4    8 MiB -6 -5 -2 -11   b = 8    4 MiB -2 -4 +2 -2    8 MiB -5 -5  0 -2
//            b = 16   2 MiB -1 -1 +3 +4    4 MiB -2 -2  0 +2    8 MiB -3 -3 -1 -1   14 MiB -2 -2 -1 -1
//            b = 32   4 MiB -1 -1 +1  0    7 MiB -2 -2  0  0;  b = 64  2 MiB 0 0 +2 +1
template <int DT, int B, bool FOUR6>
static int sse_past_caches(int64_t n, bool behind_absmax)
{
    constexpr int64_t kMiB = 1 << 20;
    if (DT != kBF16 || n > 64 * kMiB || !(FOUR6 || B == 2 || behind_absmax)) return 0;
    const int64_t sse_bytes = n / B * 4, from = behind_absmax ? (FOUR6 ? 4 : 8) : 6;
    return (sse_bytes >= from * kMiB && sse_bytes <= 15 * kMiB) ? kSsePastCaches : 0;
}

template <int DT, int B, int FMT, bool FOUR6>
static hipError_t launch_recipe(const StreamArgs& a, int pz)
{
    const int64_t n_full = a.n / 8;
    const int count = (int)(a.n - n_full * 8);
    // reciprocal-refined division only where its exactness argument holds; with the abs-max in
    // device memory the kernel makes the same choice itself
    // the variant that also writes the clipping-only SSE exists for the run-time mode only
    const int tmode = (a.absmax_dev || a.clip) ? kDynT : (a.T == 1.0f) ? kNoT : (fast_division_ok(a.T) ? kFastT : kSlowT);
    const int64_t slices = (n_full + kThreads - 1) / kThreads;
    const uint32_t n_slices = (uint32_t)slices;
    const uint32_t last = (uint32_t)(n_full - (slices - 1) * kThreads);              // not read when there is no slice
    const uint32_t tail = (B < 8) ? (uint32_t)count : 0u;
    const int workers = (n_slices == 0u) ? 0 : stream_grid(((slices + kItems - 1) / kItems) * kThreads);
    const dim3 grid((unsigned)workers + (tail != 0u ? 1u : 0u)), block(kThreads);
    uint32_t* codes = reinterpret_cast<uint32_t*>(a.codes);
    const int flags = pz | sse_past_caches<DT, B, FOUR6>(a.n, a.absmax_dev != nullptr);
    if constexpr (DT == kBF16 && FMT != kE8M0) {
        if (takes_scaled_kernel<B, FOUR6>(a, slices, workers)) {
            hipLaunchKernelGGL((stream_scaled_kernel<B, FMT, FOUR6>), grid, block, 0, a.stream, a.x, n_slices, last, tail, a.T,
                               flags, (uint32_t)workers, a.absmax_dev, a.t_out, codes, a.scales, a.sse);
            return hipGetLastError();
        }
    }
    if (slices >= kOnceFrom && slices <= kOnceMost && (tmode == kNoT || tmode == kFastT)) {
        const uint32_t tiles = (n_slices + (uint32_t)kOnce - 1u) / (uint32_t)kOnce;
        const dim3 once(tiles + (tail != 0u ? 1u : 0u));
#define MXQ_LAUNCH_ONCE(MODE)                                                                                                  \
    hipLaunchKernelGGL((stream_once_kernel<DT, B, FMT, FOUR6, MODE>), once, block, 0, a.stream, a.x, n_slices, last, tail,     \
                       a.T, flags, tiles, codes, a.scales, a.sse)
        if (tmode == kNoT) MXQ_LAUNCH_ONCE(kNoT);
        else MXQ_LAUNCH_ONCE(kFastT);
#undef MXQ_LAUNCH_ONCE
        return hipGetLastError();
    }
    const StreamKernelArgs args{a.x, n_slices, last, tail, a.T, flags, (uint32_t)workers, a.absmax_dev, a.t_out, codes, a.scales, a.sse, a.clip};
#define MXQ_LAUNCH_STREAM(MODE, CLIP)                                                                 \
    hipLaunchKernelGGL((stream_kernel<DT, B, FMT, FOUR6, MODE, CLIP>), grid, block, 0, a.stream, args)
    if (a.clip) MXQ_LAUNCH_STREAM(kDynT, true);
    else if (tmode == kNoT) MXQ_LAUNCH_STREAM(kNoT, false);
    else if (tmode == kFastT) MXQ_LAUNCH_STREAM(kFastT, false);
    else if (tmode == kSlowT) MXQ_LAUNCH_STREAM(kSlowT, false);
    else MXQ_LAUNCH_STREAM(kDynT, false);
#undef MXQ_LAUNCH_STREAM
    return hipGetLastError();
}

template <int DT, int B, int FMT>
static hipError_t launch_fmt(const StreamArgs& a)
{
    const bool four6 = (a.recipe == 2 || a.recipe == 3);
    const int pz = (a.recipe == 1 || a.recipe == 3) ? 1 : 0;
    if constexpr (FMT == kE8M0) {
        return launch_recipe<DT, B, FMT, false>(a, 0);
    } else {
        return four6 ? launch_recipe<DT, B, FMT, true>(a, pz) : launch_recipe<DT, B, FMT, false>(a, pz);
    }
}

template <int DT, int B>
static hipError_t launch_block(const StreamArgs& a)
{
    switch (a.scale_fmt) {
        case kE8M0: return launch_fmt<DT, B, kE8M0>(a);
        case kE4M3: return launch_fmt<DT, B, kE4M3>(a);
        default: return launch_fmt<DT, B, kUE5M3>(a);
    }
}

template <int DT>
static hipError_t launch_dt(const StreamArgs& a)
{
    switch (a.block) {
        case 2: return launch_block<DT, 2>(a);
        case 4: return launch_block<DT, 4>(a);
        case 8: return launch_block<DT, 8>(a);
        case 16: return launch_block<DT, 16>(a);
        case 32: return launch_block<DT, 32>(a);
        case 64: return launch_block<DT, 64>(a);
        default: return launch_block<DT, 128>(a);
    }
}

// ------------------------------------------------------------------------------ batch dispatch

template <int DT, int B, int FMT, bool FOUR6>
static hipError_t launch_batch_recipe(const StreamArgs* t, int count, int pz, hipStream_t stream)
{
    // up to kMaxBatch tensors per launch, ragged tails (b = 2, 4) included
    for (int i0 = 0; i0 < count; i0 += kMaxBatch) {
        BatchArgs a{};
        int64_t sum = 0;
        for (int i = i0; i < count && i < i0 + kMaxBatch; ++i) sum += (t[i].n / 8 + kThreads - 1) / kThreads;
        const bool once = sum >= kOnceFrom && sum <= kOnceMost;
        const int64_t per = once ? kOnce : 1;
        uint32_t n_t = 0u;
        int64_t total = 0;
        bool tails = false;
        for (int i = i0; i < count && i < i0 + kMaxBatch; ++i) {
            const int64_t n_full = t[i].n / 8;
            const int64_t slices = (n_full + kThreads - 1) / kThreads;
            a.x[n_t] = t[i].x;
            a.codes[n_t] = reinterpret_cast<uint32_t*>(t[i].codes);
            a.scales[n_t] = t[i].scales;
            a.sse[n_t] = t[i].sse;
            a.first[n_t] = (uint32_t)total;                      // the host has bounded the sum below 2^32
            a.slices[n_t] = (uint32_t)slices;
            a.last[n_t] = (uint32_t)(n_full - (slices - 1) * kThreads);
            a.tail[n_t] = (uint32_t)(t[i].n - n_full * 8);
            tails |= a.tail[n_t] != 0u;
            total += (slices + per - 1) / per;
            ++n_t;
        }
        a.first[n_t] = (uint32_t)total;
        a.count = n_t;
        const int flags = pz | sse_past_caches<DT, B, FOUR6>(sum * kThreads * 8, false);
        const int workers = (total == 0) ? 0 : once ? (int)total : stream_grid(total * kThreads);
        a.workers = (uint32_t)workers;
        const dim3 grid((unsigned)workers + (tails ? n_t : 0u));
        if (once)
            hipLaunchKernelGGL((stream_batch_once_kernel<DT, B, FMT, FOUR6>), grid, dim3(kThreads), 0, stream, a, flags);
        else
            hipLaunchKernelGGL((stream_batch_kernel<DT, B, FMT, FOUR6>), grid, dim3(kThreads), 0, stream, a, flags);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int DT, int B>
static hipError_t launch_batch_block(const StreamArgs* t, int count, hipStream_t stream)
{
    const int recipe = t[0].recipe;
    const bool four6 = (recipe == 2 || recipe == 3);
    const int pz = (recipe == 1 || recipe == 3) ? 1 : 0;
    switch (t[0].scale_fmt) {
        case kE8M0: return launch_batch_recipe<DT, B, kE8M0, false>(t, count, 0, stream);
        case kE4M3: return four6 ? launch_batch_recipe<DT, B, kE4M3, true>(t, count, pz, stream)
                                 : launch_batch_recipe<DT, B, kE4M3, false>(t, count, pz, stream);
        default: return four6 ? launch_batch_recipe<DT, B, kUE5M3, true>(t, count, pz, stream)
                              : launch_batch_recipe<DT, B, kUE5M3, false>(t, count, pz, stream);
    }
}

template <int DT>
static hipError_t launch_batch_dt(const StreamArgs* t, int count, hipStream_t stream)
{
    switch (t[0].block) {
        case 2: return launch_batch_block<DT, 2>(t, count, stream);
        case 4: return launch_batch_block<DT, 4>(t, count, stream);
        case 8: return launch_batch_block<DT, 8>(t, count, stream);
        case 16: return launch_batch_block<DT, 16>(t, count, stream);
        case 32: return launch_batch_block<DT, 32>(t, count, stream);
        case 64: return launch_batch_block<DT, 64>(t, count, stream);
        default: return launch_batch_block<DT, 128>(t, count, stream);
    }
}

// `t[0 .. count)`: validated tensors that share dtype, block, scale format and a streaming recipe.
hipError_t launch_stream_batch(const StreamArgs* t, int count, hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    return (t[0].dtype == kBF16) ? launch_batch_dt<kBF16>(t, count, stream) : launch_batch_dt<kF32>(t, count, stream);
}

hipError_t launch_stream(const StreamArgs& a)
{
    return (a.dtype == kBF16) ? launch_dt<kBF16>(a) : launch_dt<kF32>(a);
}

}  // namespace mxq
