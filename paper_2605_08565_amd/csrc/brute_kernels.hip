// Brute-force scale search (last paragraph of Section 2): for every block, every finite,
// strictly positive scale code is tried; the code of minimal block SSE wins, the lowest code
// on a tie.  Same lane mapping as the streaming kernels (8 elements per lane).  The tensor is
// read once and every candidate costs only ALU work, so this kernel is bound by the fp32
// vector units, not by HBM.
//
// A scale is S = m * 2^e with m in {1, 1.125, .., 1.875}.  Dividing by 2^e commutes with
// rounding, so the quotient v / S is formed once per mantissa (w_m = v / m, 7 divisions per
// element instead of one per candidate) and the E2M1 conversion instruction applies 2^e.
// The inverse conversion returns q * 2^e, and the residual v - (q * 2^e) * m needs a single
// FMA because the product is exact.  Candidates are visited in ascending code order, one
// binade (8 codes) at a time, so a strict "less than" between binades and the first position
// inside one keep the lowest code on ties.
//
// Power-of-two scales (E8M0, every byte 0x00 .. 0xFE is a finite positive value, 255 candidates)
// need no quotient at all: the conversion instruction divides by 2^k itself.
#include "mxq_device.hpp"
#include "mxq_launch.hpp"

#include <type_traits>

namespace mxq {

// hi/lo split of 1/m for m = 1 + i/8 (see "Quotients whose rounding decisions are exact").
__device__ constexpr float mant_value(int i) { return 1.0f + (float)i * 0.125f; }
__device__ constexpr float mant_rhi(int i)                          // 1/m rounded toward zero
{
    const double d = 1.0 / (1.0 + i * 0.125);
    const float r = (float)d;
    return ((double)r > d) ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, r) - 1u) : r;
}
__device__ constexpr float mant_rlo(int i) { return (float)(1.0 / (1.0 + i * 0.125) - (double)mant_rhi(i)); }

template <int B>
struct BruteState {
    static constexpr int NBLK = (B < 8) ? 8 / B : 1;
    float best_sse[NBLK];
    uint32_t best_code[NBLK];
};

// Arg-min over a group of up to 8 consecutive codes (one binade): begin(), put<POS>(k, sse) per
// candidate and block slot, end(st, code0) -- the code of position p is code0 + p.  The
// candidates only deposit their block SSEs; the group's minimum (three-input minimum
// instructions) is compared with the running best once per group, and only when some lane of
// the wavefront improved is the position of the minimum looked up (the first position that
// equals it: the lowest code on a tie inside the group; between groups "strictly less" keeps
// the earlier, lower code).  A candidate costs half an instruction here; measured against a
// compare and two selects per candidate it is faster also when most groups improve.
template <int B>
struct GroupArgMin {
    static constexpr int NBLK = BruteState<B>::NBLK;
    float s[NBLK][8];

    // Position 7 is the only one that can be without a candidate (the 7 sub-normal codes; the
    // NaN code at the top of the last binade): +inf never wins.
    __device__ __forceinline__ void begin()
    {
#pragma unroll
        for (int k = 0; k < NBLK; ++k) s[k][7] = __builtin_inff();
    }
    template <int POS>
    __device__ __forceinline__ void put(int k, float sse) { s[k][POS] = sse; }
    __device__ __forceinline__ void end(BruteState<B>& st, uint32_t code0) const
    {
        float gmin[NBLK];
        bool any = false;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            const float a = fminf(fminf(s[k][0], s[k][1]), s[k][2]);
            const float b = fminf(fminf(s[k][3], s[k][4]), s[k][5]);
            gmin[k] = fminf(fminf(a, b), fminf(s[k][6], s[k][7]));
            any |= gmin[k] < st.best_sse[k];
        }
        if (__builtin_amdgcn_ballot_w64(any) == 0ull) return;           // wave-uniform
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            uint32_t pos = 7u;
#pragma unroll
            for (int i = 6; i >= 0; --i) pos = (s[k][i] == gmin[k]) ? (uint32_t)i : pos;
            const bool better = gmin[k] < st.best_sse[k];
            st.best_code[k] = better ? code0 + pos : st.best_code[k];
            st.best_sse[k] = better ? gmin[k] : st.best_sse[k];
        }
    }
};

// Block SSE of the lane's residuals: separately rounded squares in a balanced tree.  FUSED: every square is exact
// ("Residuals whose squares are exact" in mxq_arith.hpp), so the first level of the tree may take one of the two squares by
// a fused multiply-add with the same bits, and four of the 15 instructions go.
template <int B, bool FUSED>
__device__ __forceinline__ void residual_sse(const float (&e)[8], float (&sse)[4])
{
    if constexpr (FUSED) {
        const float s0 = e[0] * e[0], s2 = e[2] * e[2], s4 = e[4] * e[4], s6 = e[6] * e[6];
        const float p0 = __builtin_fmaf(e[1], e[1], s0), p1 = __builtin_fmaf(e[3], e[3], s2);
        const float p2 = __builtin_fmaf(e[5], e[5], s4), p3 = __builtin_fmaf(e[7], e[7], s6);
        if constexpr (B == 2) { sse[0] = p0; sse[1] = p1; sse[2] = p2; sse[3] = p3; }
        else if constexpr (B == 4) { sse[0] = p0 + p1; sse[1] = p2 + p3; }
        else sse[0] = group_sum<B / 8>((p0 + p1) + (p2 + p3));
    } else {
        float sq[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sq[j] = e[j] * e[j];
        block_sse<B>(sq, sse);
    }
}

// SSE of the lane's blocks under S = mant_value(MI) * scale2.  Of scale2 only the exponent counts, one for each
// block (scale2[k]).  w holds the lane's quotients v / mant_value(MI).
template <int B, int MI, bool FUSED>
__device__ __forceinline__ void mantissa_sse(const float (&v)[8], const float (&w)[8], const float (&scale2)[BruteState<B>::NBLK],
                                             float (&sse)[4])
{
    constexpr int EPB = (B < 8) ? B : 8;
    const uint32_t packed = e2m1_pack8_scales<EPB>(w, scale2);
    float q2[8], e[8];                                                 // q * 2^e
    e2m1_unpack2<0>(packed, scale2[0 / EPB], q2[0], q2[1]);
    e2m1_unpack2<1>(packed, scale2[2 / EPB], q2[2], q2[3]);
    e2m1_unpack2<2>(packed, scale2[4 / EPB], q2[4], q2[5]);
    e2m1_unpack2<3>(packed, scale2[6 / EPB], q2[6], q2[7]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (MI == 0) e[j] = v[j] - q2[j];
        else e[j] = __builtin_fmaf(-q2[j], mant_value(MI), v[j]);
    }
    residual_sse<B, FUSED>(e, sse);
}

// The same under one scale for all blocks, entered into the group at position POS.
template <int B, int MI, int POS, bool FUSED, class G>
__device__ __forceinline__ void try_candidate(const float (&v)[8], const float (&w)[8], float scale2, G& g)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    float scales[NBLK], sse[4];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) scales[k] = scale2;
    mantissa_sse<B, MI, FUSED>(v, w, scales, sse);
#pragma unroll
    for (int k = 0; k < NBLK; ++k) g.template put<POS>(k, sse[k]);
    // One candidate at a time: left alone, the instruction scheduler interleaves several
    // candidates, which costs registers and 10 % of the kernel's speed (measured).
    __builtin_amdgcn_sched_barrier(0);
}

template <int B, int MI, bool FUSED, class G>
__device__ __forceinline__ void try_binade_from(const float (&v)[8], const float (&w)[8][8], float scale2, bool eighth, G& g)
{
    if constexpr (MI < 7) {
        try_candidate<B, MI, MI, FUSED>(v, w[MI], scale2, g);
        try_binade_from<B, MI + 1, FUSED>(v, w, scale2, eighth, g);
    } else {
        if (eighth) try_candidate<B, 7, 7, FUSED>(v, w[7], scale2, g);
    }
}

// The 8 codes code0 .. code0 + 7 of one binade: (1 + mi/8) * scale2; the first seven where the eighth is the NaN code.
template <int B, bool FUSED>
__device__ __forceinline__ void try_binade(const float (&v)[8], const float (&w)[8][8], float scale2,
                                           uint32_t code0, bool eighth, BruteState<B>& st)
{
    GroupArgMin<B> g;
    g.begin();
    try_binade_from<B, 0, FUSED>(v, w, scale2, eighth, g);
    g.end(st, code0);
}

// ---------------------------------------------------------------------------------------
// Pruned search (recipe BRUTE_PRUNED): same result as the full enumeration, bit for bit, from about
// ten candidates per block.  Two facts bound the codes that can win a block with abs-max `amax`:
//   (hi) A scale S >= amax / 3.5 is never better than S / 2 where S / 2 is itself a code.  The grid
//        of S / 2 is {0, .25, .5, .75, 1, 1.5, 2, 3} S: it holds every point of the grid of S up to
//        3 S, and no element lies beyond 3.5 S, so none is nearer to 4 S or 6 S than to 3 S (at
//        exactly 3.5 S the two are equally far).  Every residual under S / 2 is therefore no larger
//        than under S; fp32 rounding, squaring and the sum tree are monotone, so the same holds for
//        the pinned fp32 SSE, and on a tie the lower code S / 2 wins.  S / 2 is a code for every
//        code from 16 on and for the even ones below; what is left above amax / 3.5 are the odd
//        codes below 16 (the sub-normals and the first binade, spaced by eps), and of those none
//        above the first S >= 4 amax, from which on everything quantises to zero.
//   (lo) While 6 S < amax the abs-max element saturates and alone contributes fl(fl(amax - 6 S)^2);
//        fp32 sums of non-negative terms never fall below a term, so that is a lower bound of the
//        candidate's SSE.  Once it exceeds the best SSE found so far, this code loses and, because the
//        bound grows as S falls, so do all lower ones.
// So the codes that can win a block lie between its own abs-max code (Eq. 2) and amax / 3.5 (five to seven codes, in 2 % of
// the blocks eight; odd codes to 15 beyond that where the scales are that small), and below it until (lo) stops (one to
// three codes a block of up to 16, four to seven a wavefront at b = 64 and 128; blocks beyond the format see
// walk_saturated).  Every block tries its OWN codes: blocks of very different magnitude cost each other nothing, and a
// block that is done goes on trying codes: one that cannot win changes nothing, and masking it out would cost more.
//   * Where every block of a wavefront starts at code 17 or above and lies within the format (all of UE5M3 in practice, E4M3
//     under a per-tensor scale), eight neighbouring codes hold each mantissa once.  The eight from the one below the start
//     on are tried mantissa by mantissa (try_window): w = v / mantissa is a multiplication by a constant, the same for all
//     blocks, each block's exponent goes into the conversions, and no reciprocal is formed; the order in which a block's
//     codes come does not matter to keep_less.  What is needed beyond them is tried one by one, after eight steps down
//     as in the walk, from where they ended.
//   * Any other wavefront walks code by code (walk_from_any), scale and reciprocal in per-lane registers; a block of nothing but
//     zeros, whose code is 1, makes it one of these.
// Bound by vector issue, about eleven codes.  What an instruction costs here, measured in a loop of
// independent ones over 8 wavefronts per SIMD, cycles per wavefront: fp32 add, multiply, FMA and logic
// on vector registers 2.5; the same with a scalar-register operand, minimum, maximum, compare, shift,
// DPP, unpacking and the fp64 minimum 4.8; packing to E2M1 and the reciprocal 8.4.
// Code by code throughout -> as it is, 4096 x 4096 bf16: UE5M3 b = 2 57.7 -> 52.3 us, b = 4 44.6 -> 35.5, b = 8 36.9 -> 33.3, b = 16
// 38.5 -> 34.7, b = 128 46.3 -> 41.2, with 1 % zeros b = 4 44.7 -> 35.9, with half zeros b = 16 37.0 -> 33.9, values spread evenly b = 128
// 59.5 -> 54.6; fp32 b = 4 50.5 -> 39.7; E4M3 under a per-tensor scale b = 4 57.4 -> 45.6, b = 16 50.2 -> 45.4; 4096 x 14336 UE5M3
// b = 4 129 -> 100.  Wavefronts that walk, E4M3 weights: b = 4 47.3 -> 46.3, b = 16 38.7 -> 37.5, b = 2 64.3 -> 63.7, fp32 b = 16 42.8 -> 43.1,
// b = 8 44.4 -> 45.7; UE5M3 with half zeros, b = 2 62.8 -> 62.6.
// ---------------------------------------------------------------------------------------

template <int FMT>
__device__ __forceinline__ float walk_scale(uint32_t code) { return walk_scale_bias<ScaleFmt<FMT>::kBias>(code); }

// Whether no element of the wavefront is too small for an exact square.  Wavefronts without a zero are through with the
// first test.  (Where a zero counted as too small: 4096 x 4096 bf16 with 1 % zeros, b = 4, pruned UE5M3 49.2 us instead of 37.3,
// all codes of E4M3 246 instead of 225.)
__device__ __forceinline__ bool none_vanishes(const float (&v)[8])
{
    float m = __builtin_fabsf(v[0]);
#pragma unroll
    for (int j = 1; j < 8; ++j) m = __builtin_fminf(m, __builtin_fabsf(v[j]));
    if (__builtin_amdgcn_ballot_w64(!(m >= kSmallestSquared)) == 0ull) return true;         // uniform
    uint32_t rank = square_rank(f2u(v[0]));
#pragma unroll
    for (int j = 1; j < 8; ++j) rank = min(rank, square_rank(f2u(v[j])));
    return __builtin_amdgcn_ballot_w64(rank < kSmallestSquareRank) == 0ull;
}

// SSE of the lane's blocks under the scales S.  ONE_MUL (bf16 input, no per-tensor scale): the
// quotient is one product with the hardware reciprocal.  With 8 significant bits in v and 4 in S an
// element that is not exactly half way between two grid points is at least 2^-9 (relative) away from
// the mid-point, far more than the 2^-22 that the product is off, so it rounds to the right side; an
// element exactly half way may round to either neighbour, but both leave the same |residual| and
// hence the same SSE.  (The codes come from the exact quotient, once, in walk_codes.)
template <int B, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void walk_sse(const float (&v)[8], const float (&S)[BruteState<B>::NBLK], float (&sse)[4])
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr int EPB = (B < 8) ? B : 8;
    float y[8];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        const float approx = __builtin_amdgcn_rcpf(S[k]);
        if constexpr (ONE_MUL) {
#pragma unroll
            for (int i = 0; i < EPB; ++i) y[k * EPB + i] = v[k * EPB + i] * approx;
        } else {
            const Recip r = make_recip_from(S[k], approx);
#pragma unroll
            for (int i = 0; i < EPB; ++i) y[k * EPB + i] = quot(v[k * EPB + i], r);
        }
    }
    const uint32_t packed = e2m1_pack8(y, 1.0f);
    float q[8], e[8];
    e2m1_unpack8(packed, 1.0f, q);
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = __builtin_fmaf(-q[j], S[j / EPB], v[j]);
    residual_sse<B, FUSED>(e, sse);
}

// Codes of the lane's blocks under the scales S.
template <int B>
__device__ __forceinline__ uint32_t walk_codes(const float (&v)[8], const float (&S)[BruteState<B>::NBLK])
{
    constexpr int EPB = (B < 8) ? B : 8;
    float y[8];
#pragma unroll
    for (int k = 0; k < BruteState<B>::NBLK; ++k) {
        const Recip r = make_recip_from(S[k], __builtin_amdgcn_rcpf(S[k]));
#pragma unroll
        for (int i = 0; i < EPB; ++i) y[k * EPB + i] = quot(v[k * EPB + i], r);
    }
    return e2m1_pack8(y, 1.0f);
}

// One step upwards: a strictly lower SSE wins.  Trying a code that cannot win, or the last code again,
// changes nothing, so no block needs to be masked.
template <int B, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void walk_up(const float (&v)[8], const float (&S)[BruteState<B>::NBLK],
                                        const uint32_t (&code)[BruteState<B>::NBLK], BruteState<B>& st)
{
    float sse[4];
    walk_sse<B, ONE_MUL, FUSED>(v, S, sse);
#pragma unroll
    for (int k = 0; k < BruteState<B>::NBLK; ++k) {
        const bool better = sse[k] < st.best_sse[k];
        st.best_code[k] = better ? code[k] : st.best_code[k];
        st.best_sse[k] = better ? sse[k] : st.best_sse[k];
    }
}

// What the saturated elements of the lane's blocks leave in the SSE under the scales S.
template <int B>
__device__ __forceinline__ void walk_loss(const float (&v)[8], const float (&S)[BruteState<B>::NBLK], float (&loss)[4])
{
    constexpr int EPB = (B < 8) ? B : 8;
    float sq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sq[j] = saturation_loss(v[j], S[j / EPB]);
    block_sse<B>(sq, loss);
}

// Blocks beyond the format (amax > 6 times its largest value): one element's loss hardly tells the codes
// apart there, and the walk down would try them all.  The loss of ALL saturated elements is a lower bound
// of the SSE too, tree sum against tree sum, and it does not fall as S falls.  Bisection finds the lowest
// code at which it does not exceed the best SSE so far: the floor of the walk.  And where the SSE of the
// floor is no more than the loss at the code the walk has reached, no code in between is better, and the
// lower code wins the tie: the walk is over (values so large that the codes hardly matter, or not at all).
// Called when a wavefront has gone walk_patience steps down.
// 4096 x 4096 bf16 Student-t values, with the walk alone -> with the floor: E4M3, values times 2^16, b = 2
// 653 -> 69 us, b = 16 357 -> 44, b = 128 392 -> 76 (full enumeration 251 to 278); UE5M3, times 2^30, b = 2
// 1287 -> 63 us, b = 16 735 -> 46, b = 128 711 -> 77 (457 to 530); values inside the formats within 2 %, for
// which the compiler has to be told that this is the rare path (b = 128 with a tensor scale 177 -> 175 us).
template <int B, int FMT, bool ONE_MUL>
__device__ __forceinline__ void walk_saturated(const float (&v)[8], uint32_t (&code)[BruteState<B>::NBLK],
                                               uint32_t (&floor)[BruteState<B>::NBLK], BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    float S[NBLK], reached[4], at_mid[4], sse[4];
    uint32_t hi[NBLK];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) { hi[k] = code[k]; S[k] = walk_scale<FMT>(code[k]); }
    walk_loss<B>(v, S, reached);
#pragma unroll 1
    for (uint32_t range = (uint32_t)ScaleFmt<FMT>::kMaxCode; range != 0u; range >>= 1) {       // uniform; halves [floor, hi] until one code is left
        uint32_t mid[NBLK];
#pragma unroll
        for (int k = 0; k < NBLK; ++k) { mid[k] = (floor[k] + hi[k]) >> 1; S[k] = walk_scale<FMT>(mid[k]); }
        walk_loss<B>(v, S, at_mid);
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            const bool loses = at_mid[k] > st.best_sse[k];
            floor[k] = loses ? min(mid[k] + 1u, hi[k]) : floor[k];
            hi[k] = loses ? hi[k] : mid[k];
        }
    }
#pragma unroll
    for (int k = 0; k < NBLK; ++k) { floor[k] = hi[k]; S[k] = walk_scale<FMT>(hi[k]); }
    walk_sse<B, ONE_MUL, false>(v, S, sse);
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        const bool over = sse[k] <= reached[k] && sse[k] <= st.best_sse[k];
        st.best_code[k] = over ? floor[k] : st.best_code[k];
        st.best_sse[k] = over ? sse[k] : st.best_sse[k];
        code[k] = over ? floor[k] : code[k];
    }
}

// The way up from any start, for wavefronts with a block among theirs that the window below does not take.
template <int B, int FMT, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void walk_from_any(const float (&v)[8], float (&amax)[BruteState<B>::NBLK],
                                              uint32_t (&start)[BruteState<B>::NBLK], BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr uint32_t kMax = (uint32_t)ScaleFmt<FMT>::kMaxCode;
    constexpr int kBias = ScaleFmt<FMT>::kBias;

    float S[NBLK], sse[4];
    uint32_t code[NBLK], halved[NBLK], last_odd[NBLK];
    bool none = false;
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        start[k] = max(start[k], 1u);
        halved[k] = walk_halved<kBias>(sf_encode_rne<FMT>(amax[k] * kHalvedAt), amax[k]);
        S[k] = walk_scale<FMT>(start[k]);
    }
    walk_sse<B, ONE_MUL, FUSED>(v, S, sse);
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        const bool better = sse[k] < __builtin_inff();                  // nothing wins where every SSE overflows
        st.best_code[k] = better ? start[k] : 1u;
        st.best_sse[k] = better ? sse[k] : __builtin_inff();
        none |= !better;
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(none) != 0ull, 0)) {                    // uniform
        // Under every code a NaN stays a NaN, and where the saturated elements alone overflow here they
        // do under every lower code (there is none above).  Such a block walks like one of zeros: not at
        // all, with code 1 as the full enumeration has it.
        float loss[4];
        walk_loss<B>(v, S, loss);
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            const bool dead = sse[k] != sse[k] || loss[k] == __builtin_inff();
            start[k] = dead ? 1u : start[k];
            halved[k] = dead ? 1u : halved[k];
            amax[k] = dead ? 0.0f : amax[k];
        }
    }

#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        last_odd[k] = walk_last_odd<kBias>(amax[k]);
        code[k] = start[k];
    }
    while (true) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            code[k] += 1u;
            const bool below = code[k] < halved[k];
            code[k] = below ? code[k] : (code[k] | 1u);
            any |= below || code[k] <= last_odd[k];
            code[k] = min(code[k], kMax);
            S[k] = walk_scale<FMT>(code[k]);
        }
        if (__builtin_amdgcn_ballot_w64(any) == 0ull) break;            // uniform
        walk_up<B, ONE_MUL, FUSED>(v, S, code, st);
    }
}

// The way down from `code`, `step` steps of which have been taken: the lower code wins a tie.  Beyond the patience the
// squares need not be exact any more.
template <int B, int FMT, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void walk_down(const float (&v)[8], const float (&amax)[BruteState<B>::NBLK],
                                          uint32_t (&code)[BruteState<B>::NBLK], uint32_t step, BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    float S[NBLK], sse[4];
    uint32_t floor[NBLK];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) floor[k] = 1u;
    const auto down = [&](uint32_t end, auto fused) {
        for (;; ++step) {
            if (FUSED && step == end) return true;
            if (!decltype(fused)::value && __builtin_expect(step == walk_patience(B), 0))
                walk_saturated<B, FMT, ONE_MUL>(v, code, floor, st);
            bool any = false;
#pragma unroll
            for (int k = 0; k < NBLK; ++k) {
                const bool first = code[k] <= floor[k];                 // nothing below: the floor once more
                code[k] = max(code[k] - 1u, floor[k]);
                S[k] = walk_scale<FMT>(code[k]);
                const float over = amax[k] - 6.0f * S[k];
                any |= !first && !(over > 0.0f && over * over > st.best_sse[k]);
            }
            if (__builtin_amdgcn_ballot_w64(any) == 0ull) return false; // uniform
            walk_sse<B, ONE_MUL, decltype(fused)::value>(v, S, sse);
#pragma unroll
            for (int k = 0; k < NBLK; ++k) {
                const bool better = sse[k] <= st.best_sse[k];
                st.best_code[k] = better ? code[k] : st.best_code[k];
                st.best_sse[k] = better ? sse[k] : st.best_sse[k];
            }
        }
    };
    if constexpr (FUSED) {
        if (__builtin_expect(down(walk_patience(B), std::true_type{}), 0)) down(0xFFFFFFFFu, std::false_type{});
    } else {
        down(0u, std::false_type{});
    }
}

// The best of a block in the window below as one 64-bit number: the SSE above the bits of its scale, which order like
// the codes.  The lower SSE wins and, on a tie, the lower code, in one instruction and whatever the order in which they are
// tried: as a double such a pair is a positive number (an infinite SSE included), and pairs order like the doubles.
__device__ __forceinline__ void keep_less(uint64_t& best, float sse, float S)
{
    const uint64_t other = ((uint64_t)f2u(sse) << 32) | f2u(S);
    asm("v_min_f64 %0, %0, %1" : "+v"(best) : "v"(other));
}
__device__ __forceinline__ float sse_of(uint64_t best) { return u2f((uint32_t)(best >> 32)); }

// What is formed from v behind this is not formed before it.  Left alone, the compiler formed the quotients of all mantissas
// before the second: with blocks of two 112 to 114 vector registers for UE5M3, four wavefronts a SIMD.  Halved once it is 80
// to 82 and five or six: 4096 x 4096 bf16 with every other element zero, whose wavefronts walk, 64.7 -> 62.2 us, random values,
// in the window, 42.9 -> 43.8.  (At every mantissa, seven wavefronts, 61.6 and 44.2.)  Blocks of four hold them back at every
// mantissa: 36.1 -> 35.6.
__device__ __forceinline__ void formed_below(float (&v)[8])
{
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
}

// The codes of mantissa MI and of those behind it, one for each block: the one among the eight from `first` (a scale's bits) on.
template <int B, int MI, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void try_window(float (&v)[8], const uint32_t (&first)[BruteState<B>::NBLK],
                                           uint64_t (&best)[BruteState<B>::NBLK])
{
    constexpr int NBLK = BruteState<B>::NBLK;
    if constexpr (MI < 8) {
        float S[NBLK], w[8], sse[4];
#pragma unroll
        for (int k = 0; k < NBLK; ++k)
            S[k] = u2f(((first[k] + ((uint32_t)(7 - MI) << 20)) & 0xFF800000u) | ((uint32_t)MI << 20));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if constexpr (MI == 0) w[j] = v[j];
            else if constexpr (ONE_MUL) w[j] = v[j] * (1.0f / mant_value(MI));
            else w[j] = quot(v[j], Recip{mant_rhi(MI), mant_rlo(MI)});
        }
        mantissa_sse<B, MI, FUSED>(v, w, S, sse);
#pragma unroll
        for (int k = 0; k < NBLK; ++k) keep_less(best[k], sse[k], S[k]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (B == 2 ? MI == 3 : B == 4) formed_below(v);
        try_window<B, MI + 1, ONE_MUL, FUSED>(v, first, best);
    }
}

template <int B, int FMT, bool ONE_MUL, bool FUSED>
__device__ __forceinline__ void brute_search_pruned(float (&v)[8], uint32_t& packed, BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr int LANES = (B < 8) ? 1 : B / 8;
    constexpr int EPB = (B < 8) ? B : 8;
    constexpr uint32_t kMax = (uint32_t)ScaleFmt<FMT>::kMaxCode;
    constexpr uint32_t kBits0 = (127u - (uint32_t)ScaleFmt<FMT>::kBias) << 3;       // code + kBits0: the scale's upper bits
    // bf16 wavefronts whose squares are not all exact hold an element below 2^-67 that is not zero, or one far beyond the format:
    // the code of a second window in the kernel costs the others more than it gains those (4096 x 14336 UE5M3 b = 4 104.6 us
    // with it, 98.8 without).
    constexpr bool kWindow = !ONE_MUL || FUSED || B == 2;

    float amax[NBLK], S[NBLK], sse[4];
    uint32_t start[NBLK];
    bool outside = false;
    block_amax<NBLK, EPB, LANES>(v, amax);
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        start[k] = sf_encode_rne<FMT>(sixth_of(amax[k]));
        outside |= start[k] < 17u || amax[k] > 6.5f * ScaleFmt<FMT>::kMaxValue;
    }
    uint32_t step = 0u;                                                  // uniform: steps down so far
    bool done = false, whole = true;                                    // uniform: over, all codes are still to be tried
    if (kWindow && __builtin_amdgcn_ballot_w64(outside) == 0ull) {
        // Every code the blocks try is a normal number with a code at half its value: neighbouring codes are 2^20
        // apart as floats.  amax / 3.5 lies five to seven codes above the start, in 2 % of the blocks eight.  The eight codes
        // from the one below the start on (from the eighth last on at the end of the format) hold each mantissa once, so they
        // are tried mantissa by mantissa.
        uint32_t bits[NBLK];
        uint64_t best[NBLK];
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            bits[k] = (window_first(start[k], kMax) + kBits0) << 20;
            best[k] = (uint64_t)0x7F800000u << 32;
        }
        try_window<B, 0, ONE_MUL, FUSED>(v, bits, best);
        bool any = false;
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            S[k] = u2f(bits[k] + (8u << 20));
            any |= 3.5f * S[k] < amax[k] && S[k] <= ScaleFmt<FMT>::kMaxValue;
            S[k] = fminf(S[k], ScaleFmt<FMT>::kMaxValue);
        }
        if (__builtin_amdgcn_ballot_w64(any) != 0ull) {                 // uniform
            walk_sse<B, ONE_MUL, FUSED>(v, S, sse);
#pragma unroll
            for (int k = 0; k < NBLK; ++k) keep_less(best[k], sse[k], S[k]);
        }
#pragma unroll
        for (int k = 0; k < NBLK; ++k) S[k] = u2f(bits[k]);
#pragma unroll 1
        for (uint32_t i = 0u; i < kWindowDown; ++i) {
            any = false;
#pragma unroll
            for (int k = 0; k < NBLK; ++k) {
                S[k] = u2f(f2u(S[k]) - (1u << 20));
                const float over = __builtin_fmaf(-6.0f, S[k], amax[k]);               // 6 S is exact: as amax - 6 S
                any |= !(over * __builtin_fabsf(over) > sse_of(best[k]));
            }
            if (__builtin_amdgcn_ballot_w64(any) == 0ull) { done = true; break; }      // uniform
            walk_sse<B, ONE_MUL, FUSED>(v, S, sse);
#pragma unroll
            for (int k = 0; k < NBLK; ++k) keep_less(best[k], sse[k], S[k]);
        }
        bool bad = false;                                               // an SSE that is not a finite number
#pragma unroll
        for (int k = 0; k < NBLK; ++k) {
            bad |= !(sse_of(best[k]) < __builtin_inff());
            st.best_sse[k] = sse_of(best[k]);
            st.best_code[k] = ((uint32_t)best[k] >> 20) - kBits0;
        }
        done = done && __builtin_amdgcn_ballot_w64(bad) == 0ull;
        if (__builtin_expect(!done, 0)) {                               // on down from here, unless all is to be tried again
            whole = __builtin_amdgcn_ballot_w64(bad) != 0ull;
            step = whole ? 0u : window_steps(B);
#pragma unroll
            for (int k = 0; k < NBLK; ++k) start[k] = whole ? start[k] : (bits[k] >> 20) - kBits0 - kWindowDown;
        }
    }
    if (!done) {
        if (whole) walk_from_any<B, FMT, ONE_MUL, FUSED>(v, amax, start, st);
        walk_down<B, FMT, ONE_MUL, FUSED>(v, amax, start, step, st);
    }

#pragma unroll
    for (int k = 0; k < NBLK; ++k) S[k] = walk_scale<FMT>(st.best_code[k]);
    packed = walk_codes<B>(v, S);
}

// FUSED for the wavefronts whose squares are all exact: no element but zeros nearly vanishes, none is far beyond the format.  (The walk
// starts at a scale of at least amax / 9, or at the largest, above amax / 128, and takes up to 16 steps (walk_patience) down with
// it: from a normal code to a quarter of its value, amax / 512, or from code 17 and below to code 1, amax / 114 at most.)
template <int B, int FMT, bool ONE_MUL>
__device__ __forceinline__ void search_pruned(float (&v)[8], uint32_t& packed, BruteState<B>& st)
{
    if constexpr (ONE_MUL && B != 2) {
        float largest = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) largest = __builtin_fmaxf(largest, __builtin_fabsf(v[j]));
        const bool beyond = !(largest < kExactScales * ScaleFmt<FMT>::kMaxValue);
        if (__builtin_amdgcn_ballot_w64(beyond) == 0ull && none_vanishes(v)) {               // uniform
            brute_search_pruned<B, FMT, true, true>(v, packed, st);
            return;
        }
    }
    brute_search_pruned<B, FMT, ONE_MUL, false>(v, packed, st);
}

// Value of a power-of-two scale byte (0 .. 254); 2^-127 is a sub-normal float.
__device__ __forceinline__ float pow2_scale(uint32_t code)
{
    return (code == 0u) ? u2f(0x00400000u) : u2f(code << 23);
}

// The 8 codes code0 .. code0 + 7 of the power-of-two format; code 255 is not a number.
template <int B, int POS, class G>
__device__ __forceinline__ void try_pow2_from(const float (&v)[8], uint32_t code0, G& g)
{
    if constexpr (POS < 8) {
        if (POS < 7 || code0 + 7u <= 254u) try_candidate<B, 0, POS, false>(v, v, pow2_scale(code0 + POS), g);
        try_pow2_from<B, POS + 1>(v, code0, g);
    }
}

// The sub-normal codes 1 .. 7 = j * s1: 1, 2, 3 = 1.5 * 2, 4, 5 = 1.25 * 4, 6 = 1.5 * 4, 7 = 1.75 * 4.
template <int B>
__device__ __forceinline__ void try_subnormals(const float (&v)[8], const float (&w)[8][8], float s1, float s2, float s4, BruteState<B>& st)
{
    GroupArgMin<B> g;
    g.begin();
    try_candidate<B, 0, 0, false>(v, w[0], s1, g);
    try_candidate<B, 0, 1, false>(v, w[0], s2, g);
    try_candidate<B, 4, 2, false>(v, w[4], s2, g);
    try_candidate<B, 0, 3, false>(v, w[0], s4, g);
    try_candidate<B, 2, 4, false>(v, w[2], s4, g);
    try_candidate<B, 4, 5, false>(v, w[4], s4, g);
    try_candidate<B, 6, 6, false>(v, w[6], s4, g);
    g.end(st, 1u);
}

// Search for the lane's 8 values (already divided by T): winner codes, packed nibbles, SSE.
template <int B, int FMT, bool SHORT>
__device__ __forceinline__ void brute_search(const float (&v)[8], uint32_t& packed, BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr int EPB = (B < 8) ? B : 8;
    constexpr int bias = ScaleFmt<FMT>::kBias;
    constexpr int emin = 1 - bias;                                      // exponent of the first binade

    float w[8][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) w[0][j] = v[j];
#pragma unroll
    for (int i = 1; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < 8; ++j) w[i][j] = quot(v[j], Recip{mant_rhi(i), mant_rlo(i)});
    }
#pragma unroll
    for (int k = 0; k < NBLK; ++k) { st.best_sse[k] = __builtin_inff(); st.best_code[k] = 1u; }

    const float s1 = u2f((uint32_t)(127 + emin - 3) << 23);
    const float s2 = u2f((uint32_t)(127 + emin - 2) << 23);
    const float s4 = u2f((uint32_t)(127 + emin - 1) << 23);
    // SHORT (bf16 that nothing has divided): from the first binade on whose squares are all exact, four of a candidate's
    // instructions go.  (Two loops: with both kinds in one, more registers and 2 % slower.)  4096 x 4096 E4M3, separate roundings ->
    // as it is: b = 4 247 -> 224 us, b = 16 237 -> 216, b = 32 243 -> 221, b = 128 259 -> 239; UE5M3 b = 16 460 -> 423; 4096 x 14336 E4M3 b = 16
    // 801 -> 739.  b = 2, of whose sums too little is left, not.
    float largest = 0.0f;
    bool regular = false;
    if constexpr (SHORT) {
        regular = none_vanishes(v);
#pragma unroll
        for (int j = 0; j < 8; ++j) largest = __builtin_fmaxf(largest, __builtin_fabsf(v[j]));
    }
    const auto exact = [&](float lowest) {
        return SHORT && regular && __builtin_amdgcn_ballot_w64(!(largest < kExactScales * lowest)) == 0ull;
    };
    try_subnormals<B>(v, w, s1, s2, s4, st);

    // normal codes: exponent field ef = 1 .. kMaxCode >> 3, value (1 + mi/8) * 2^(ef - bias)
    constexpr uint32_t kMax = (uint32_t)ScaleFmt<FMT>::kMaxCode, last = kMax >> 3;
    const auto scale2 = [](uint32_t ef) { return u2f((ef + (uint32_t)(127 - bias)) << 23); };
    if constexpr (SHORT) {
        // The last binade, without the NaN code, by itself: with two loops the compiler does not take it out of them, and they
        // branch around the eighth code (4096 x 4096 bf16 UE5M3 b = 4, squares exact 446 us like that, not exact 483; as it is 423, 456).
        static_assert((kMax & 7u) == 6u);
        uint32_t ef = 1u;
        for (; ef < last; ++ef) {
            if (exact(scale2(ef))) break;                               // and all above it
            try_binade<B, false>(v, w, scale2(ef), ef << 3, true, st);
        }
        for (; ef < last; ++ef) try_binade<B, true>(v, w, scale2(ef), ef << 3, true, st);
        try_binade<B, false>(v, w, scale2(last), last << 3, false, st);
    } else {
        for (uint32_t ef = 1u; ef <= last; ++ef) try_binade<B, false>(v, w, scale2(ef), ef << 3, (ef << 3) + 7u <= kMax, st);
    }

    // codes of the winners
    float y[8];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) {
        const Recip r = make_recip(sf_decode<FMT>(st.best_code[k]));
#pragma unroll
        for (int i = 0; i < EPB; ++i) y[k * EPB + i] = quot(v[k * EPB + i], r);
    }
    packed = e2m1_pack8(y, 1.0f);
}

// The same over the 255 power-of-two scales (bytes 0x00 .. 0xFE): no quotient, the conversion
// applies 2^k itself, for the candidates and for the winners' codes.
template <int B>
__device__ __forceinline__ void brute_search_pow2(const float (&v)[8], uint32_t& packed, BruteState<B>& st)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr int EPB = (B < 8) ? B : 8;
#pragma unroll
    for (int k = 0; k < NBLK; ++k) { st.best_sse[k] = __builtin_inff(); st.best_code[k] = 0u; }
    for (uint32_t code0 = 0u; code0 < 256u; code0 += 8u) {
        GroupArgMin<B> g;
        g.begin();
        try_pow2_from<B, 0>(v, code0, g);
        g.end(st, code0);
    }
    float S[NBLK];
#pragma unroll
    for (int k = 0; k < NBLK; ++k) S[k] = pow2_scale(st.best_code[k]);
    packed = e2m1_pack8_scales<EPB>(v, S);
}

// Scale value of a winner byte.
template <int FMT>
__device__ __forceinline__ float brute_scale_value(uint32_t code)
{
    if constexpr (FMT == kE8M0) return pow2_scale(code);
    else return sf_decode<FMT>(code);
}

// Clipping-only part of the winners' block SSE (appendix figure "Clipping only MSE"): elements with
// |v| > 6 S quantise to +-6; their squared residuals, summed by the tree of the block SSE.
template <int B>
__device__ __forceinline__ void brute_clip_sse(const float (&v)[8], const float (&S)[BruteState<B>::NBLK], float (&clip)[4])
{
    constexpr int EPB = (B < 8) ? B : 8;
    float sq[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float s = S[j / EPB];
        const float q = u2f(0x40C00000u | (f2u(v[j]) & 0x80000000u));          // +-6
        const float e = __builtin_fmaf(-q, s, v[j]);
        sq[j] = (__builtin_fabsf(v[j]) > 6.0f * s) ? e * e : 0.0f;
    }
    const float p0 = sq[0] + sq[1], p1 = sq[2] + sq[3], p2 = sq[4] + sq[5], p3 = sq[6] + sq[7];
    if constexpr (B == 2) { clip[0] = p0; clip[1] = p1; clip[2] = p2; clip[3] = p3; }
    else if constexpr (B == 4) { clip[0] = p0 + p1; clip[1] = p2 + p3; }
    else clip[0] = group_sum<B / 8>((p0 + p1) + (p2 + p3));
}

template <int DT, int B, int FMT, bool HAS_T, bool PRUNE>
__device__ __forceinline__ void brute_body(const void* __restrict__ x, int64_t n_full, int tail, float T_arg,
                                           const float* __restrict__ absmax_dev, float* __restrict__ t_out,
                                           uint32_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ sse_out,
                                           float* __restrict__ clip_out)
{
    constexpr int NBLK = BruteState<B>::NBLK;
    constexpr int LANES = (B < 8) ? 1 : B / 8;
    float T = T_arg;
    if constexpr (HAS_T) {
        if (absmax_dev) {                                            // T from the abs-max in device memory
            T = tensor_scale_of<FMT>(*absmax_dev);
            if (t_out && blockIdx.x == 0 && threadIdx.x == 0) *t_out = T;
        }
    }

    const int64_t stride = (int64_t)gridDim.x * kThreads;
    int64_t chunk = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int64_t base = chunk - (threadIdx.x & 63);
    // n not a multiple of 8 (b = 2 or 4 only): one more chunk, of `tail` elements, read and written
    // element-wise by the lane it falls to
    const int64_t n_chunks = n_full + ((B < 8 && tail != 0) ? 1 : 0);

    for (; base < n_chunks; base += stride, chunk += stride) {
        float v[8];
        if (chunk < n_full) load8<DT>(x, chunk << 3, v);
        else if (B < 8 && chunk < n_chunks) load_partial<DT>(x, chunk << 3, tail, v);
        else {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = 0.0f;
        }
        if constexpr (HAS_T) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = v[i] / T;
        }
        uint32_t packed;
        BruteState<B> st;
        if constexpr (FMT == kE8M0) brute_search_pow2<B>(v, packed, st);
        else if constexpr (PRUNE) search_pruned<B, FMT, DT == kBF16 && !HAS_T>(v, packed, st);
        else brute_search<B, FMT, DT == kBF16 && !HAS_T && B != 2>(v, packed, st);
        float clip[4];
        if (clip_out) {                                                 // uniform
            float S_best[NBLK];
#pragma unroll
            for (int k = 0; k < NBLK; ++k) S_best[k] = brute_scale_value<FMT>(st.best_code[k]);
            brute_clip_sse<B>(v, S_best, clip);
        }

        if (chunk < n_full) {
            codes[chunk] = packed;
            if constexpr (B >= 8) {
                if ((threadIdx.x & (LANES - 1)) == 0) {
                    const int64_t blk = chunk / LANES;
                    scales[blk] = (uint8_t)st.best_code[0];
                    if (sse_out) sse_out[blk] = st.best_sse[0];
                    if (clip_out) clip_out[blk] = clip[0];
                }
            } else {
                const int64_t blk0 = chunk * NBLK;
#pragma unroll
                for (int k = 0; k < NBLK; ++k) {
                    scales[blk0 + k] = (uint8_t)st.best_code[k];
                    if (sse_out) sse_out[blk0 + k] = st.best_sse[k];
                    if (clip_out) clip_out[blk0 + k] = clip[k];
                }
            }
        } else if (B < 8 && chunk < n_chunks) {
            for (int i = 0; i < tail / 2; ++i) reinterpret_cast<uint8_t*>(codes)[chunk * 4 + i] = (uint8_t)(packed >> (8 * i));
#pragma unroll
            for (int k = 0; k < NBLK; ++k) {
                if (k < tail / B) {
                    scales[chunk * NBLK + k] = (uint8_t)st.best_code[k];
                    if (sse_out) sse_out[chunk * NBLK + k] = st.best_sse[k];
                    if (clip_out) clip_out[chunk * NBLK + k] = clip[k];
                }
            }
        }
    }
}

// One argument costs the host less than ten (see StreamKernelArgs).
struct BruteKernelArgs {
    const void* x;
    int64_t n_full;
    int tail;
    float T;
    const float* absmax_dev;
    float* t_out;
    uint32_t* codes;
    uint8_t* scales;
    float* sse;
    float* clip;
};

template <int DT, int B, int FMT, bool HAS_T, bool PRUNE>
__global__ void __launch_bounds__(kThreads)
brute_kernel(const BruteKernelArgs a)
{
    brute_body<DT, B, FMT, HAS_T, PRUNE>(a.x, a.n_full, a.tail, a.T, a.absmax_dev, a.t_out, a.codes, a.scales, a.sse, a.clip);
}

template <int DT, int B, int FMT, bool PRUNE>
static hipError_t launch_f(const StreamArgs& a)
{
    const int64_t n_full = a.n / 8;
    const int count = (int)(a.n - n_full * 8);
    const bool has_t = (a.absmax_dev != nullptr) || (a.T != 1.0f);
    const int64_t need = (n_full + (count != 0 ? 1 : 0) + kThreads - 1) / kThreads;
    const dim3 grid((unsigned)(need < 256 * 8 ? need : 256 * 8)), block(kThreads);
    const BruteKernelArgs args{a.x, n_full, count, a.T, a.absmax_dev, a.t_out, (uint32_t*)a.codes, a.scales, a.sse, a.clip};
    if (has_t) hipLaunchKernelGGL((brute_kernel<DT, B, FMT, true, PRUNE>), grid, block, 0, a.stream, args);
    else hipLaunchKernelGGL((brute_kernel<DT, B, FMT, false, PRUNE>), grid, block, 0, a.stream, args);
    return hipGetLastError();
}

template <int DT, int B>
static hipError_t launch_b(const StreamArgs& a)
{
    const bool prune = (a.recipe == 5);
    if (a.scale_fmt == kE8M0) return launch_f<DT, B, kE8M0, false>(a);          // the host refuses the pruned form
    if (a.scale_fmt == kE4M3) return prune ? launch_f<DT, B, kE4M3, true>(a) : launch_f<DT, B, kE4M3, false>(a);
    return prune ? launch_f<DT, B, kUE5M3, true>(a) : launch_f<DT, B, kUE5M3, false>(a);
}

template <int DT>
static hipError_t launch_d(const StreamArgs& a)
{
    switch (a.block) {
        case 2: return launch_b<DT, 2>(a);
        case 4: return launch_b<DT, 4>(a);
        case 8: return launch_b<DT, 8>(a);
        case 16: return launch_b<DT, 16>(a);
        case 32: return launch_b<DT, 32>(a);
        case 64: return launch_b<DT, 64>(a);
        default: return launch_b<DT, 128>(a);
    }
}

hipError_t launch_brute(const StreamArgs& a)
{
    return (a.dtype == kBF16) ? launch_d<kBF16>(a) : launch_d<kF32>(a);
}

}  // namespace mxq
