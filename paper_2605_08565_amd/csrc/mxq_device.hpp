// Device-side building blocks of libmxq (gfx950): number formats, exact-decision quotients,
// E2M1 rounding, wavefront reductions.  Everything here follows Section 2 of "Finer is Better
// (with the Right Scaling)" (Eq. 1-4); the places where a cheaper instruction sequence
// replaces a literal IEEE division carry the argument for why every rounding DECISION is
// unchanged.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mxq_arith.hpp"      // the division-free sequences, shared with the host-side proof

namespace mxq {

constexpr int kE8M0 = 0, kE4M3 = 1, kUE5M3 = 2;
constexpr int kBF16 = 0, kF32 = 1;

// ---------------------------------------------------------------------------------------
// 8-bit floating-point scale formats (Background; eps under Eq. 3).
// ---------------------------------------------------------------------------------------
template <int FMT> struct ScaleFmt;
template <> struct ScaleFmt<kE4M3> {
    static constexpr int kBias = 7;              // eps = 2^(1-7-3) = 2^-9
    static constexpr int kMaxCode = 0x7E;        // 1.75 * 2^8 = 448
    static constexpr float kMaxValue = 448.0f;
};
template <> struct ScaleFmt<kUE5M3> {
    static constexpr int kBias = 15;             // eps = 2^-17
    static constexpr int kMaxCode = 0xFE;        // 1.75 * 2^16
    static constexpr float kMaxValue = 114688.0f;
};

template <int FMT>
__device__ __forceinline__ float sf_decode(uint32_t code) { return sf_decode_bias<ScaleFmt<FMT>::kBias>(code); }

// Round_SF of Eq. 2: round-to-nearest-even of y >= 0 into the format, clipped to the largest
// finite value.  For E4M3 the gfx950 conversion v_cvt_pk_fp8_f32 does the rounding (OCP E4M3,
// nearest even, sub-normals included) in one instruction; it turns values beyond 448 into NaN
// rather than clipping, hence the clamp in front of it.  UE5M3 rounds on the bit pattern.
template <int FMT>
__device__ __forceinline__ uint32_t sf_encode_rne(float y)
{
    y = fminf(y, ScaleFmt<FMT>::kMaxValue);
    if constexpr (FMT == kE4M3) {
        return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(y, y, 0, false) & 0xFFu;
    } else {
        return sf_encode_bits<ScaleFmt<FMT>::kBias>(y);
    }
}

// Value of any scale byte of any format (NaN for bytes that are not finite numbers); used where
// the format is a run-time argument (de-quantise, diagnostics).
__device__ __forceinline__ float scale_byte_value(int fmt, uint32_t code)
{
    const float nan = u2f(0x7FC00000u);
    if (fmt == kE8M0) {
        if (code == 255u) return nan;
        return (code == 0u) ? u2f(0x00400000u) : u2f(code << 23);      // 2^-127 is sub-normal
    }
    if (fmt == kE4M3) return (code > (uint32_t)ScaleFmt<kE4M3>::kMaxCode) ? nan : sf_decode<kE4M3>(code);
    return (code > (uint32_t)ScaleFmt<kUE5M3>::kMaxCode) ? nan : sf_decode<kUE5M3>(code);
}

// Per-tensor scale of hierarchical scaling from the tensor abs-max: the same function as the
// host helper of the C ABI, so both give the same bits.
template <int FMT>
__device__ __forceinline__ float tensor_scale_of(float absmax)
{
    float sf_max;
    if constexpr (FMT == kE8M0) sf_max = u2f(254u << 23);
    else sf_max = ScaleFmt<FMT>::kMaxValue;
    return tensor_scale_from(absmax, sf_max);
}

// Entry of every scale byte, put once per workgroup into LDS, one entry per thread.  Code 0 has S = 0 and a zero
// "reciprocal", so that every quotient is a signed 0.
struct __align__(16) ScaleEntry {          // for quot(): reciprocal in two parts, as make_recip() has them
    static constexpr bool kOneProduct = false;
    float S, rhi, rlo, pad;
    static constexpr ScaleEntry of(float S)
    {
        float hi = 1.0f / S;
        if ((double)hi * S > 1.0) hi = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, hi) - 1u);      // exact product
        return ScaleEntry{S, hi, (float)(1.0 - (double)hi * S) * hi, 0.0f};
    }
};
struct __align__(8) ScalePair {            // for quot_truncated(): the float nearest to 1/S
    static constexpr bool kOneProduct = true;
    float S, r;
    static constexpr ScalePair of(float S) { return ScalePair{S, 1.0f / S}; }
};

template <class Entry> struct ScaleTable { Entry of[256]; };
template <int FMT, class Entry>
constexpr ScaleTable<Entry> make_scale_table()
{
    ScaleTable<Entry> t{};
    for (int c = 1; c <= ScaleFmt<FMT>::kMaxCode; ++c) {
        float S = (c < 8) ? (float)c : (float)(8 + (c & 7));             // in units of the code's binade
        for (int e = (c < 8) ? 0 : (c >> 3) - 1; e > 0; --e) S *= 2.0f;
        for (int e = ScaleFmt<FMT>::kBias + 2; e > 0; --e) S *= 0.5f;
        t.of[c] = Entry::of(S);
    }
    return t;
}
template <int FMT, class Entry>
static __device__ constexpr ScaleTable<Entry> kScaleTable = make_scale_table<FMT, Entry>();

// Copied from memory, where the compiler has put the entries, or formed here (FORMED): a division and 25 instructions
// in every wavefront while the first loads are under way, against a load that all workgroups of a launch make at once
// and that those loads stand behind.  Copied -> formed, abs-max b = 16: 128 x 4096 bf16 2.41 -> 2.34 us, fp32 2.63 -> 2.57;
// 512 x 4096 3.08 -> 2.98, 3.67 -> 3.61; 4096 x 4096 9.0 -> 8.8, 14.5 -> 14.2; 4096 x 14336 28.3 -> 28.0, 4-over-6 b = 8 30.6 ->
// 30.1.  bf16 under a tensor scale has enough to compute there already: 512 x 4096 3.46 -> 3.63, 1024 x 4096 4.23 -> 4.50.
template <int FMT, bool FORMED, class Entry>
__device__ __forceinline__ void fill_scale_table(Entry* tab)
{
    const uint32_t c = threadIdx.x;                                      // 256 threads, 256 codes
    if constexpr (!FORMED) {
        tab[c] = kScaleTable<FMT, Entry>.of[c];
    } else {
        Entry e{};
        if (c >= 1u && c <= (uint32_t)ScaleFmt<FMT>::kMaxCode) {
            e.S = sf_decode<FMT>(c);
            if constexpr (Entry::kOneProduct) {
                e.r = 1.0f / e.S;
            } else {
                const Recip r = make_recip(e.S);
                e.rhi = r.hi;
                e.rlo = r.lo;
            }
        }
        tab[c] = e;
    }
    __syncthreads();
}

// The same, where the scale mantissas 1 + i/8 with bit i of `above` set take the reciprocal above the nearest one.
template <int FMT>
__device__ __forceinline__ void fill_scale_table(ScalePair* tab, uint32_t above)
{
    ScalePair e = kScaleTable<FMT, ScalePair>.of[threadIdx.x];
    e.r = lean_reciprocal(e.S, e.r, above);
    tab[threadIdx.x] = e;
    __syncthreads();
}

// quot_truncated() of the lane's 8 values by NBLK reciprocals: 8 products and two mode switches instead of the
// 16 instructions of quot().  The rounding mode of the wavefront's fp32 arithmetic is switched inside one asm
// block, so that no other instruction can get between.  Two writes of the mode register have to be two wait states
// apart, and the compiler, which sees to that between its own, does not look into asm: each block brings them
// (s_nop 1), whatever write lies before it.  Two-part product -> this with its half as large table entries, 4-over-6 on
// 4096 x 14336 bf16: b = 16 30.9 -> 29.8 us, 32 30.8 -> 28.9, 64 31.5 -> 29.3; UE5M3 b = 16 32.1 -> 29.7, b = 2 58.6 ->
// 55.6; b = 8 32.2 -> 32.0 (bound by memory).
template <int NBLK>
__device__ __forceinline__ void quot8_truncated(const float (&v)[8], const float (&r)[NBLK], float (&y)[8])
{
    static_assert(NBLK == 1 || NBLK == 2 || NBLK == 4, "blocks inside a lane");
    const float r0 = r[0], r1 = r[2 * NBLK / 8], r2 = r[4 * NBLK / 8], r3 = r[6 * NBLK / 8];
    asm("s_nop 1\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3\n\t"
        "v_mul_f32 %0, %8, %16\n\t"
        "v_mul_f32 %1, %9, %16\n\t"
        "v_mul_f32 %2, %10, %17\n\t"
        "v_mul_f32 %3, %11, %17\n\t"
        "v_mul_f32 %4, %12, %18\n\t"
        "v_mul_f32 %5, %13, %18\n\t"
        "v_mul_f32 %6, %14, %19\n\t"
        "v_mul_f32 %7, %15, %19\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]), "=&v"(y[4]), "=&v"(y[5]), "=&v"(y[6]), "=&v"(y[7])
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]),
          "v"(r0), "v"(r1), "v"(r2), "v"(r3));
}

static __device__ constexpr LeanPairs kLeanPairs = make_lean_pairs();

// Whether both shorter sequences are exact for every bf16 input under this T: two mantissas and one of the 32
// pairs in every lane, so that no wavefront waits for another.  Bit i of `above`: the scale mantissa 1 + i/8
// takes the reciprocal above the nearest one.  (All but the rounding mode and the ballots is in mxq_arith.hpp.)
__device__ __forceinline__ bool lean_T(LeanPair pair, float T, float rT, Recip r, uint32_t& above)
{
    const uint32_t lane = threadIdx.x & 63u;
    float x, y, y_above;
    const bool near = lean_quotient_candidate(pair.td, T, x);
    const float v = div_by_T(x, T, rT);
    asm("s_nop 1\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3\n\t"
        "v_mul_f32 %0, %2, %3\n\t"
        "v_mul_f32 %1, %2, %4\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
        : "=&v"(y), "=&v"(y_above) : "v"(v), "v"(pair.rd), "v"(float_above(pair.rd)));
    const bool divides = lean_division_exact(lane, T, rT, r) && lean_division_exact(lane + 64u, T, rT, r);
    above = lean_of_mantissas((uint32_t)__builtin_amdgcn_ballot_w64(near && !lean_decides(pair, v, y)));
    const uint32_t above_fails = lean_of_mantissas((uint32_t)__builtin_amdgcn_ballot_w64(near && !lean_decides(pair, v, y_above)));
    return (above & above_fails) == 0u && __builtin_amdgcn_ballot_w64(!divides) == 0ull;
}

// ---------------------------------------------------------------------------------------
// E2M1 (Section 2 value set {0, .5, 1, 1.5, 2, 3, 4, 6}).
// ---------------------------------------------------------------------------------------

// Rounding to E2M1 uses the gfx950 conversion instructions v_cvt_scalef32_pk_fp4_f32 /
// v_cvt_scalef32_pk_f32_fp4.  The forward one divides two fp32 inputs by a power-of-two scale
// (only the exponent of the scale operand is used), rounds to nearest even onto
// {0, .5, 1, 1.5, 2, 3, 4, 6}, saturates at 6, keeps the sign bit also for zero results, and
// writes the two 4-bit codes (first input in the low nibble) into the selected byte of the
// destination; the inverse one returns the two values times the scale.  Mid-points go to the
// even code: 0.25->0, 0.75->1, 1.25->1, 1.75->2, 2.5->2, 3.5->4, 5->4.
using f32x2 = float __attribute__((ext_vector_type(2)));
using f32x4 = float __attribute__((ext_vector_type(4)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));

template <int SEL>
__device__ __forceinline__ uint32_t e2m1_pack2(uint32_t old, float a, float b, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, a, b, scale, SEL);
}

template <int SEL>
__device__ __forceinline__ void e2m1_unpack2(uint32_t packed, float scale, float& a, float& b)
{
    const f32x2 r = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(packed, scale, SEL);
    a = r.x;
    b = r.y;
}

// 8 values -> one dword of codes (element j in nibble j).  The four conversions overwrite all
// four bytes, so the register they accumulate into needs no initial value; the empty asm
// statement defines it without emitting an instruction.
__device__ __forceinline__ uint32_t e2m1_pack8(const float (&y)[8], float scale)
{
    uint32_t r;
    asm volatile("" : "=v"(r));
    r = e2m1_pack2<0>(r, y[0], y[1], scale);
    r = e2m1_pack2<1>(r, y[2], y[3], scale);
    r = e2m1_pack2<2>(r, y[4], y[5], scale);
    r = e2m1_pack2<3>(r, y[6], y[7], scale);
    return r;
}

// The same with one power-of-two scale per block of EPB elements inside the lane (EPB even, so
// a pair never straddles two blocks).
template <int EPB>
__device__ __forceinline__ uint32_t e2m1_pack8_scales(const float (&y)[8], const float (&scale)[8 / EPB])
{
    uint32_t r;
    asm volatile("" : "=v"(r));
    r = e2m1_pack2<0>(r, y[0], y[1], scale[0 / EPB]);
    r = e2m1_pack2<1>(r, y[2], y[3], scale[2 / EPB]);
    r = e2m1_pack2<2>(r, y[4], y[5], scale[4 / EPB]);
    r = e2m1_pack2<3>(r, y[6], y[7], scale[6 / EPB]);
    return r;
}

__device__ __forceinline__ void e2m1_unpack8(uint32_t packed, float scale, float (&q)[8])
{
    e2m1_unpack2<0>(packed, scale, q[0], q[1]);
    e2m1_unpack2<1>(packed, scale, q[2], q[3]);
    e2m1_unpack2<2>(packed, scale, q[4], q[5]);
    e2m1_unpack2<3>(packed, scale, q[6], q[7]);
}

// ---------------------------------------------------------------------------------------
// Wavefront helpers.  A block of more than 8 elements is spread over 2, 4, 8 or 16
// neighbouring lanes (8 elements each); xor-butterflies inside a 16-lane DPP row combine
// them.  After a butterfly level every lane of a pair holds the same value, so the mirror
// patterns (lane i <-> 7-i, i <-> 15-i) deliver the partner group's value for the xor-4 and
// xor-8 levels.  fp32 addition is commutative, so all lanes of a block end with the same
// bits, equal to the balanced binary tree in index order.
// ---------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i inside each group of 8
constexpr int kDppMirror = 0x140;     // lane i <-> 15-i inside each row of 16

// Maximum of non-negative floats: their bit patterns order like unsigned integers.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

template <int LANES>
__device__ __forceinline__ float group_max(float nonneg)
{
    uint32_t v = f2u(nonneg);
    if constexpr (LANES >= 2) v = max(v, dpp_u<kDppXor1>(v));
    if constexpr (LANES >= 4) v = max(v, dpp_u<kDppXor2>(v));
    if constexpr (LANES >= 8) v = max(v, dpp_u<kDppHalfMirror>(v));
    if constexpr (LANES >= 16) v = max(v, dpp_u<kDppMirror>(v));
    return u2f(v);
}

template <int LANES>
__device__ __forceinline__ float group_sum(float v)
{
    if constexpr (LANES >= 2) v = v + dpp_f<kDppXor1>(v);
    if constexpr (LANES >= 4) v = v + dpp_f<kDppXor2>(v);
    if constexpr (LANES >= 8) v = v + dpp_f<kDppHalfMirror>(v);
    if constexpr (LANES >= 16) v = v + dpp_f<kDppMirror>(v);
    return v;
}

// Block SSE: balanced tree in index order, inside the lane and then across the block's lanes.
// For b < 8 the lane holds 8/b blocks; their sums come back in sse[0 .. 8/b).
template <int B>
__device__ __forceinline__ void block_sse(const float (&sq)[8], float (&sse)[4])
{
    const float p0 = sq[0] + sq[1], p1 = sq[2] + sq[3], p2 = sq[4] + sq[5], p3 = sq[6] + sq[7];
    if constexpr (B == 2) {
        sse[0] = p0; sse[1] = p1; sse[2] = p2; sse[3] = p3;
    } else if constexpr (B == 4) {
        sse[0] = p0 + p1; sse[1] = p2 + p3;
    } else {
        sse[0] = group_sum<B / 8>((p0 + p1) + (p2 + p3));
    }
}

// Division by the per-tensor scale T of hierarchical scaling: div_by_T (reciprocal + one FMA
// refinement, exact inside the range fast_division_ok / fast_division_unsafe_amax delimit) or the
// plain IEEE division.
enum : int { kNoT = 0, kFastT = 1, kSlowT = 2, kDynT = 3,     // kDynT: T comes from device memory, one of
                                                              // the other three is chosen at run time
             kLeanT = 4 };    // bf16, T for which lean_T holds: the two parts of 1/T in the place of (T, 1/T)

template <int NBLK, int EPB, int LANES>
__device__ __forceinline__ void block_amax(const float (&v)[8], float (&amax)[NBLK])
{
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < EPB; ++i) a = fmaxf(a, __builtin_fabsf(v[k * EPB + i]));
        amax[k] = group_max<LANES>(a);
    }
}

// Division by the per-tensor scale (MODE: none / reciprocal-refined / plain / in two parts) and the block
// abs-max of the adjusted values.
template <int MODE, int NBLK, int EPB, int LANES>
__device__ __forceinline__ void adjust_and_amax(float (&v)[8], float T, float rT, float (&amax)[NBLK])
{
    if constexpr (MODE == kSlowT) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = v[i] / T;            // IEEE division
        block_amax<NBLK, EPB, LANES>(v, amax);
    } else if constexpr (MODE == kLeanT) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = quot(v[i], Recip{T, rT});
        block_amax<NBLK, EPB, LANES>(v, amax);
    } else if constexpr (MODE == kFastT) {
        float raw[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { raw[i] = v[i]; v[i] = div_by_T(raw[i], T, rT); }
        block_amax<NBLK, EPB, LANES>(v, amax);
        bool unsafe = false;
#pragma unroll
        for (int k = 0; k < NBLK; ++k)                  // 0 < amax < 2^-40  or  amax > 2^90
            unsafe |= fast_division_unsafe_amax(amax[k]);
        if (__builtin_amdgcn_ballot_w64(unsafe) != 0ull) {       // rare, wave-uniform
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = raw[i] / T;
            block_amax<NBLK, EPB, LANES>(v, amax);
        }
    } else {
        block_amax<NBLK, EPB, LANES>(v, amax);
    }
}

// ---------------------------------------------------------------------------------------
// Loads: 8 consecutive elements per lane, widened to fp32.
// ---------------------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ void load8(const void* x, int64_t first, float (&v)[8])
{
    if constexpr (DT == kBF16) {
        const uint4 r = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(x) + first);
        v[0] = u2f(r.x << 16); v[1] = u2f(r.x & 0xFFFF0000u);
        v[2] = u2f(r.y << 16); v[3] = u2f(r.y & 0xFFFF0000u);
        v[4] = u2f(r.z << 16); v[5] = u2f(r.z & 0xFFFF0000u);
        v[6] = u2f(r.w << 16); v[7] = u2f(r.w & 0xFFFF0000u);
    } else {
        const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(x) + first);
        const float4 a = p[0], b = p[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

// Ragged tail: `count` < 8 valid elements, the rest read as +0.
template <int DT>
__device__ __forceinline__ void load_partial(const void* x, int64_t first, int count, float (&v)[8])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float f = 0.0f;
        if (i < count) {
            if constexpr (DT == kBF16)
                f = u2f((uint32_t)static_cast<const uint16_t*>(x)[first + i] << 16);
            else
                f = static_cast<const float*>(x)[first + i];
        }
        v[i] = f;
    }
}

}  // namespace mxq
