// Scalar arithmetic of the libmxq kernels that replaces a literal IEEE division (or a search over
// a value table) by a cheaper instruction sequence.  Every function here is plain fp32 / integer
// C++ without any GPU intrinsic, so the SAME source is compiled twice: by hipcc into the gfx950
// kernels (mxq_device.hpp includes this file) and by the host compiler into
// tests/host/kernel_arithmetic_check.cpp, which runs each sequence over (near-)exhaustive input
// sets against exact arithmetic.  An edit here is therefore re-proved by the CPU test suite.
//
// The operations follow Section 2 of "Finer is Better (with the Right Scaling)": Eq. 1 (power-of-
// two scale), Eq. 2 (abs-max scale rounded to the scale format), the element quotient v / S in
// front of the E2M1 rounding, and the division by the per-tensor scale of hierarchical scaling.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define MXQ_HD __host__ __device__ __forceinline__
#else
#define MXQ_HD inline
#endif

namespace mxq {

MXQ_HD uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
MXQ_HD float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }

// ---------------------------------------------------------------------------------------
// 8-bit floating-point scale formats with 3 mantissa bits and exponent bias BIAS (Background;
// eps under Eq. 3): E4M3 has bias 7, UE5M3 bias 15.
// ---------------------------------------------------------------------------------------

// Value of a finite scale code: m * 2^(1-bias-3) below the first binade, else
// (1 + m/8) * 2^(e-bias), built directly as fp32 bits.
template <int BIAS>
MXQ_HD float sf_decode_bias(uint32_t code)
{
    const float sub = (float)(code & 7u) * u2f((uint32_t)(127 + 1 - BIAS - 3) << 23);
    const float nrm = u2f((code + ((127u - (uint32_t)BIAS) << 3)) << 20);
    return (code < 8u) ? sub : nrm;
}

// Round_SF of Eq. 2 for 0 <= y <= max_value (the caller clips): round to nearest even into the
// format.  Normal range: RNE of the fp32 mantissa to 3 bits by the usual
// add-half-minus-one-plus-lsb on the bit pattern.  Sub-normal range: adding 2^(emin+20) makes
// the fp32 adder itself round y to a multiple of eps (ties to even).
template <int BIAS>
MXQ_HD uint32_t sf_encode_bits(float y)
{
    const uint32_t b = f2u(y);
    const uint32_t nrm = ((b + 0x7FFFFu + ((b >> 20) & 1u)) >> 20) - ((127u - (uint32_t)BIAS) << 3);
    const float magic = u2f((uint32_t)(127 + (1 - BIAS) + 20) << 23);
    const uint32_t sub = f2u(y + magic) - f2u(magic);
    const float min_normal = u2f((uint32_t)(127 + 1 - BIAS) << 23);
    return (y < min_normal) ? sub : nrm;
}

// ---------------------------------------------------------------------------------------
// Quotients whose rounding decisions are exact.
//
// The method divides in IEEE fp32 (v / S, amax / M) and then rounds the quotient to a very
// coarse grid (E2M1, or an 8-bit scale format).  Only the side of each grid mid-point t the
// quotient falls on matters.  For a divisor d with at most 4 significant bits and a
// mid-point t with at most 5, the product t*d is exact in fp32, and for fp32 v
//     fl32(v / d) <, =, > t   <=>   v <, =, > t*d,
// because v != t*d implies |v/(t*d) - 1| >= 2^-24, which is more than half an ulp of t away.
// The same holds for  y = fl32(v*r_hi + fl32(v*r_lo))  with r_hi + r_lo = 1/d to 2^-47
// relative (r_hi need not be the nearest float for that): y is within 2^-46 relative of v/d
// before its single rounding, far inside the 2^-28 margin the inequality above leaves.  So y
// may stand in for the IEEE quotient wherever only the rounded code is needed.  (The residual
// v - q*S is computed from v, q and S, never from y.)
// ---------------------------------------------------------------------------------------
struct Recip { float hi, lo; };

// r_hi = 1/d rounded toward zero, r_lo = fl32(rho * r_hi) >= 0 with rho = 1 - r_hi*d exact (fma).
// Both parts are non-negative, so both products in quot() carry the sign of v and a zero
// quotient (v = -0, or an underflowing product) keeps the sign bit of v.
MXQ_HD Recip make_recip(float d)
{
    Recip r;
    r.hi = 1.0f / d;
    if (__builtin_fmaf(-r.hi, d, 1.0f) < 0.0f) r.hi = u2f(f2u(r.hi) - 1u);      // was rounded up
    const float rho = __builtin_fmaf(-r.hi, d, 1.0f);
    r.lo = rho * r.hi;
    return r;
}

// The same from a hardware reciprocal: `approx` is 1/d to within one ulp.  Scaled down by 2^-22 it
// is certainly below 1/d, so rho > 0; rho < 2^-21 and has at most 7 significant bits (hi*d ends at
// 2^-28), so the fma is exact; hi + lo = 1/d to within 2^-41.
MXQ_HD Recip make_recip_from(float d, float approx)
{
    Recip r;
    r.hi = approx * (1.0f - 0x1p-22f);
    r.lo = __builtin_fmaf(-r.hi, d, 1.0f) * r.hi;
    return r;
}

MXQ_HD float quot(float v, Recip r)
{
    return __builtin_fmaf(v, r.hi, v * r.lo);
}

// A single multiplication by a rounded reciprocal, rounded to nearest, is NOT enough for the code, not even
// for bf16 inputs with their 8 significant bits: an input that sits exactly on a tie (v = t*d) must produce
// exactly t for the ties-to-even rule of the E2M1 rounding, and t*d*fl(1/d) misses t by an ulp for most d
// (the host-side check shows the failures when quot is replaced by one product).  Where only the
// residual is needed and not the code, one product does for 8 significant bits: an exact tie leaves the
// same |residual| on either side, and every other quotient is 2^-8 away from a mid-point (walk_sse).
//
// One product that is TRUNCATED does for the code too.  The float nearest to 1/d is (1/d)*(1 + e*2^-24) with
// e = 0, .125, .25 .. .875 for the eight scale mantissas 1, 1.125 .. 1.875: never below 1/d.  An exact
// tie gives t*(1 + e*2^-24), less than an ulp (2^-23) above t, which truncates to t; every other quotient is
// 2^-8 away from a mid-point.  quot_truncated() says what the kernels' products compute (quot8_truncated in
// mxq_device.hpp switches the rounding mode around them).
#if !defined(__HIP_DEVICE_COMPILE__)
inline float quot_truncated(float v, float nearest_reciprocal)
{
    const double exact = (double)v * (double)nearest_reciprocal;                // at most 48 bits
    const float f = (float)exact;
    return __builtin_fabs((double)f) > __builtin_fabs(exact) ? u2f(f2u(f) - 1u) : f;      // away from zero: one step back
}
#endif

// ---------------------------------------------------------------------------------------
// Scalar rules of the pruned scale search (the search itself is brute_search_pruned; the host check
// tests/host/search_walk_check.cpp searches single blocks with these same functions).
// ---------------------------------------------------------------------------------------

// Value of a scale code, sub-normal codes included: the code's bits moved into the fp32 exponent and
// mantissa are off by a power of two only, and the multiplication is exact.  (Beyond the last code
// the value is meaningless but harmless.)
template <int BIAS>
MXQ_HD float walk_scale_bias(uint32_t code)
{
    return u2f(code << 20) * u2f((uint32_t)(127 + 127 - BIAS) << 23);
}

// The first code with 3.5 S >= amax, one past the last code if there is none; `h` is the code that
// amax * kHalvedAt rounds to, at most one too low (3.5 S is exact).
constexpr float kHalvedAt = (float)(1.0 / 3.5);
template <int BIAS>
MXQ_HD uint32_t walk_halved(uint32_t h, float amax)
{
    return h + ((3.5f * walk_scale_bias<BIAS>(h) < amax) ? 1u : 0u);
}

// Below code 16 (spacing eps, half of an odd code is no code): the first code >= 1 with S >= 4 amax,
// 15 if there is none.  From S = 4 amax on every element quantises to zero.
template <int BIAS>
MXQ_HD uint32_t walk_last_odd(float amax)
{
    const float inv_eps4 = 4.0f * u2f((uint32_t)(127 + BIAS + 2) << 23);      // 4 / eps
    return (uint32_t)__builtin_fminf(__builtin_fmaxf(__builtin_ceilf(amax * inv_eps4), 1.0f), 15.0f);
}

// An element with |v| > 6 S saturates and leaves fl(fl(|v| - 6 S)^2) in the SSE (6 S is exact); this is
// that term, +0 for every other element.  It does not grow with S.
MXQ_HD float saturation_loss(float v, float S)
{
    const float over = __builtin_fmaxf(__builtin_fabsf(v) - 6.0f * S, 0.0f);
    return over * over;
}

// Steps down after which the walk looks for its floor: a few more than ordinary wavefronts take, whose
// number grows with the block.  (With three, b = 16 took 47 instead of 36 us on 4096 x 4096 and b = 128
// 59 instead of 44; with twelve at b = 2, values beyond the format 107 instead of 62.)
MXQ_HD constexpr uint32_t walk_patience(int b) { return b <= 4 ? 3u : b == 8 ? 4u : b == 16 ? 6u : b == 32 ? 10u : 16u; }

// The window of a block that starts at code 17 or above: the eight codes from the one below its start on (the last eight of
// the format at its end) and, one by one, up to kWindowDown below them (so code 8, the first normal one, is the lowest).
constexpr uint32_t kWindowDown = 8u;
MXQ_HD uint32_t window_first(uint32_t start, uint32_t last) { return start - 1u < last - 7u ? start - 1u : last - 7u; }

// Steps that a walk has behind it which goes on down from there: the codes above are not tried again.  (Values spread
// evenly, b = 128, take some 15 steps: 4096 x 4096 UE5M3 bf16 99 us with a walk from the start, 56 like this, fp32 117 and 64.)
MXQ_HD constexpr uint32_t window_steps(int b) { return walk_patience(b) < kWindowDown + 1u ? walk_patience(b) : kWindowDown + 1u; }

// ---------------------------------------------------------------------------------------
// Residuals whose squares are exact.  v a bf16 value (8 significant bits), S a scale of 4 bits with 2^e <= S < 2^(e+1),
// r = v - q*S its residual under the E2M1 value q.  Where |v| < 512 S, r has at most 12 significant bits, so r*r has at
// most 24:
//   q = 0:             r = v, 8 bits.
//   |v| <= 6 S, q > 0: |v| >= S/4, so v is a multiple of 2^(e-9) and q*S of 2^(e-4); |r| <= S < 2^(e+1): 10 bits.
//   |v| > 6 S:         q*S = 6 S is a multiple of 2^(e-2).  With 2^k <= |v| < 2^(k+1), e+2 <= k <= e+9, v is one of 2^(k-7);
//                      |r| < 2^(k+1): 8 bits for k <= e+5, k-e+3 <= 12 beyond.
// And r*r does not underflow below the fp32 grid where r is a multiple of 2^-74: a bf16 value from 2^-67 on is, and so
// is q*S (S >= 2^-17).  So a square and its sum with another are one fused multiply-add with the bits of the two
// separately rounded operations.
// ---------------------------------------------------------------------------------------
// A zero leaves a residual of zero: only other elements below kSmallestSquared are too small.  Their magnitudes by rank, a
// zero's above all, so that a minimum over many tells whether one of them is.
constexpr float kSmallestSquared = 0x1p-67f;
MXQ_HD constexpr uint32_t square_rank(uint32_t float_bits) { return (float_bits << 1) - 1u; }
constexpr uint32_t kSmallestSquareRank = square_rank(__builtin_bit_cast(uint32_t, kSmallestSquared));
// Below this many times a scale the squares are exact under it and, for the steps of a walk, down to a quarter of it.
constexpr float kExactScales = 128.0f;

// amax / 6 and amax / 4 in front of Round_SF (Eq. 2, M = 6; Eq. 4, M = 4): the first by the
// two-part reciprocal above (6 has 2 significant bits), the second is exact.
constexpr float kSixthHi = (float)(1.0 / 6.0);
constexpr float kSixthLo = (float)(1.0 / 6.0 - (double)kSixthHi);
MXQ_HD float sixth_of(float amax) { return __builtin_fmaf(amax, kSixthHi, amax * kSixthLo); }
MXQ_HD float quarter_of(float amax) { return amax * 0.25f; }

// Eq. 1: k = floor(log2(amax / 6)).  With amax = m * 2^e, 1 <= m < 2: k = e - 2 when
// m >= 1.5, else e - 3; byte = k + 127, never below 0 (sub-normal or zero amax gives 0).
MXQ_HD uint32_t pow2_code(float amax)
{
    const uint32_t b = f2u(amax);
    const int c = (int)(b >> 23) - 3 + (int)((b >> 22) & 1u);
    return (uint32_t)(c > 0 ? c : 0);
}

// ---------------------------------------------------------------------------------------
// Hierarchical scaling divides every input by the per-tensor scale T in IEEE fp32.  T is the
// same for the whole tensor, so its correctly rounded reciprocal r is formed once and each
// quotient is refined once:
//     q0 = v*r;  q1 = q0 - r*(q0*T - v)                                 (remainder by FMA)
// q0 is within 1.5 ulp of v/T and the value rounded into q1 differs from the exact quotient by
// less than 3 * 2^-24 ulp, so q1 is the correctly rounded quotient unless v/T lies that close
// to the midpoint of two floats; all mantissa pairs that come so close (an integer congruence
// lists them) are checked one by one on the host, the all-ones mantissa of T excluded.  The
// remainder is formed with the opposite sign (q0*T - v) and subtracted, which keeps a signed
// zero: for v = -0 the last step is (-0)*r + (-0) = -0, whereas v - q0*T would give +0 and
// lose the sign.  The argument needs intermediate results free of
// overflow and underflow: the host takes this path only for 2^-20 <= T <= 2^20 with a
// mantissa that is not all ones, and a block whose adjusted abs-max leaves [2^-40, 2^90]
// (zero excepted) sends its whole wavefront through the plain division instead.  An element far
// below its block's abs-max can still have |v/T| < 2^-78, where the remainder may underflow and
// q1 be off by one ulp; nothing observes that: the element quantises to a signed zero and its
// squared residual underflows to zero either way.
// ---------------------------------------------------------------------------------------
MXQ_HD float div_by_T(float v, float T, float rT)
{
    const float q0 = v * rT;
    const float neg_rem = __builtin_fmaf(q0, T, -v);                 // q0*T - v, exact
    return __builtin_fmaf(-neg_rem, rT, q0);
}

// The reciprocal-refined division is exact for these T only.
MXQ_HD bool fast_division_ok(float T)
{
    return T >= 0x1p-20f && T <= 0x1p20f && (f2u(T) & 0x7FFFFFu) != 0x7FFFFFu;
}

// An adjusted block abs-max a >= 0 outside [2^-40, 2^90], zero excepted, falls back to the plain
// division.
MXQ_HD bool fast_division_unsafe_amax(float a)
{
    return (f2u(a) - 0x2B800000u) > (0x6C800000u - 0x2B800000u) && f2u(a) != 0u;
}

// bf16 inputs have 128 mantissas only, so for one T it can be SEEN whether shorter sequences are exact:
//   * the quotient x/T as quot(x, lean_recip(T)), two instructions instead of three: tried on every mantissa
//     (lean_division_exact).  Of 3 * 10^6 random T six fail.
//   * the quotient of v = fl(x/T) by a scale S as one truncated product with the float nearest to 1/S or the
//     next one above: it is within 2^-21 of x/(T*S), so it can take a wrong decision only for an x that close
//     to t*S*T, and there is at most one such mantissa for each of the 8 mantissas of S and the 4 of the
//     mid-points t.  That one is tried with both reciprocals, and the nearer one taken for a mantissa of S
//     unless it fails (lean_quotient_candidate; lean_T in mxq_device.hpp).  Of 3 * 10^6 random T 331 take one from above
//     and one is left without; of the 128 tensor scales that tensor_scale_from makes of a bf16 abs-max, whose quotients are
//     ratios of small numbers, two take one from above and four are left without.
// Both hold for every exponent of x: below |x/T| = 2^-78 the small product of the first may lose bits, but
// such an element quantises to a signed zero under every E4M3 or UE5M3 scale and its square underflows.
// T beyond 2^+-60 or with an all-ones mantissa is not tried (the reference, div_by_T, is not exact for the
// latter; within the range nothing on these mantissas over- or underflows).
MXQ_HD bool lean_T_in_range(float T)
{
    return T >= 0x1p-60f && T <= 0x1p60f && (f2u(T) & 0x7FFFFFu) != 0x7FFFFFu;
}

// The two parts of 1/T for it.  For a power of two the second part is zero, and an infinite x would give
// inf*0 = NaN where x/T is infinite; any positive part below half an ulp of every finite quotient mends that
// (in the range of T all other second parts are above 2^-110).  The quotient is the IEEE one for them too; div_by_T,
// which gives a NaN for every x/T that is infinite, is not, and stream_scaled_kernel follows div_by_T where that is
// what the general kernel takes.
MXQ_HD Recip lean_recip(float T)
{
    Recip r = make_recip(T);
    r.lo = __builtin_fmaxf(r.lo, 0x1p-126f);
    return r;
}

MXQ_HD bool lean_division_exact(uint32_t mantissa, float T, float rT, Recip r)
{
    const float x = u2f(0x3F800000u | (mantissa << 16));
    return quot(x, r) == div_by_T(x, T, rT);
}

// The bf16 value nearest to (t*d)*T, and whether it is close enough to matter.
MXQ_HD bool lean_quotient_candidate(float td, float T, float& x)
{
    const float p = td * T;
    x = u2f((f2u(p) + 0x8000u) & 0xFFFF0000u);
    return __builtin_fabsf(x - p) <= p * 0x1p-20f;
}

// The 32 pairs of a scale mantissa d (index & 7) and a mid-point mantissa t.  The even code lies above the mid-points
// .75 and 1.75: a quotient AT them goes up, so they are represented by the float below.
struct __attribute__((aligned(16))) LeanPair { float td, rd, y_at, v_at; };
struct LeanPairs { LeanPair of[32]; };
constexpr LeanPairs make_lean_pairs()
{
    LeanPairs p{};
    for (int i = 0; i < 32; ++i) {
        const float d = 1.0f + 0.125f * (float)(i & 7), t = 1.0f + 0.25f * (float)(i >> 3);
        const uint32_t below = (i >> 3) >= 2 ? 1u : 0u;
        p.of[i] = LeanPair{t * d, 1.0f / d, __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, t) - below),
                           __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, t * d) - below)};
    }
    return p;
}

MXQ_HD float float_above(float positive) { return u2f(f2u(positive) + 1u); }

// What is tried for a candidate: its truncated product y lies on the same side of t as v = fl(x/T) does of t*d.
MXQ_HD bool lean_decides(LeanPair pair, float v, float y) { return (y > pair.y_at) == (v > pair.v_at); }

// Bits of the 32 pairs -> of the 8 scale mantissas: the four mid-points of a scale mantissa together.
MXQ_HD uint32_t lean_of_mantissas(uint32_t pairs)
{
    return (pairs | (pairs >> 8) | (pairs >> 16) | (pairs >> 24)) & 0xFFu;
}

// The reciprocal that scale value S takes: bit i of `above` set, the one above the nearest for the mantissa 1 + i/8.
// Code 0 (S = 0) keeps its zero.
MXQ_HD float lean_reciprocal(float S, float nearest, uint32_t above)
{
    const uint32_t up = (S == 0.0f) ? 0u : (above >> ((f2u(S) >> 20) & 7u)) & 1u;
    return u2f(f2u(nearest) + up);
}

// Per-tensor scale of hierarchical scaling (Section 2, two-stage process) from the tensor
// abs-max: the abs-max lands on (largest element magnitude) x (largest scale value); 1 for an
// all-zero tensor or when the quotient vanishes or overflows.
MXQ_HD float tensor_scale_from(float absmax, float sf_max)
{
    if (!(absmax > 0.0f)) return 1.0f;
    const float t = absmax / (6.0f * sf_max);
    return (t > 0.0f && t < __builtin_inff()) ? t : 1.0f;
}

}  // namespace mxq
