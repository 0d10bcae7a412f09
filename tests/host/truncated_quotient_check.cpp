/*
 * Element quotients by one truncated product (mxq_arith.hpp: quot_truncated) on the CPU: for every bf16 value
 * of both signs and every scale code of E4M3 and UE5M3 the E2M1 decision must be the exact one and the
 * quotient must keep the sign of the value.  Then bf16 values under a tensor scale, for every such scale that a
 * bf16 abs-max gives and 3007 others.  Prints "<name> cases=<n> bad=<m>".
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2605_08565_amd/csrc/mxq_arith.hpp"

static const double kTie[7] = {0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0};
static const int kUp[7] = {0, 1, 0, 1, 0, 1, 0};           /* the even code lies above the tie */

/* E2M1 index of a / b for a >= 0, taken exactly: tie * b fits a double */
static int index_of(double a, double b)
{
    int m = 0;
    for (int i = 0; i < 7; ++i) m += kUp[i] ? (a >= kTie[i] * b) : (a > kTie[i] * b);
    return m;
}

static void bf16_values(void)
{
    long n = 0, bad = 0;
    for (int bias = 7; bias <= 15; bias += 8)
        for (uint32_t code = 1; code <= (bias == 7 ? 0x7Eu : 0xFEu); ++code) {
            const float S = bias == 7 ? mxq::sf_decode_bias<7>(code) : mxq::sf_decode_bias<15>(code);
            const float r = 1.0f / S;
            for (uint32_t h = 0; h < 0x7F80u; ++h) {
                const float v = mxq::u2f(h << 16), y = mxq::quot_truncated(v, r), z = mxq::quot_truncated(-v, r);
                ++n;
                bad += index_of(y, 1.0) != index_of(v, S) || signbit(y) || z != -y || !signbit(z);
            }
        }
    printf("bf16_values cases=%ld bad=%ld\n", n, bad);
}

/* lean_T of mxq_device.hpp with the ballots and the rounding mode spelt out: 0 no, 1 yes, and which scale mantissas
 * take the reciprocal above */
static const mxq::LeanPairs kPairs = mxq::make_lean_pairs();
static int lean(float T, mxq::Recip r, uint32_t* above)
{
    const float rT = 1.0f / T;
    uint32_t near_bad = 0, above_bad = 0;
    for (uint32_t m = 0; m < 128; ++m)
        if (!mxq::lean_division_exact(m, T, rT, r)) return 0;
    for (int i = 0; i < 32; ++i) {
        const mxq::LeanPair pair = kPairs.of[i];
        float x;
        if (!mxq::lean_quotient_candidate(pair.td, T, x)) continue;
        const float v = mxq::div_by_T(x, T, rT);
        near_bad |= (uint32_t)!mxq::lean_decides(pair, v, mxq::quot_truncated(v, pair.rd)) << i;
        above_bad |= (uint32_t)!mxq::lean_decides(pair, v, mxq::quot_truncated(v, mxq::float_above(pair.rd))) << i;
    }
    *above = mxq::lean_of_mantissas(near_bad);
    return (*above & mxq::lean_of_mantissas(above_bad)) == 0;
}

/* For every T that lean() accepts: quotient by T and decision under every scale mantissa, for every bf16
 * mantissa at the exponents that contain a mid-point, equal to the IEEE quotient and the exact decision. */
static long g_n, g_bad, g_refused;
static void tensor_scale(float T)
{
    const mxq::Recip r = mxq::lean_recip(T);
    uint32_t above = 0;
    if (!mxq::lean_T_in_range(T) || !lean(T, r, &above)) { ++g_refused; return; }
    for (uint32_t m = 0; m < 128; ++m)
        for (int e = -4; e <= 5; ++e) {
            const float x = ldexpf(mxq::u2f(0x3F800000u | (m << 16)), e + ilogbf(T));
            const float v = mxq::quot(x, r), w = x / T;
            g_bad += v != w || mxq::quot(-x, r) != -w;
            for (int i = 0; i < 8; ++i) {
                const float S = 1.0f + 0.125f * i, rS = mxq::lean_reciprocal(S, 1.0f / S, above);
                const float y = mxq::quot_truncated(v, rS);
                ++g_n;
                g_bad += index_of(y, 1.0) != index_of(v, S) || mxq::quot_truncated(-v, rS) != -y;
            }
        }
}

static void tensor_scales(void)
{
    for (int f = 0; f < 2; ++f)                                  /* every T that a bf16 abs-max gives, four exponents */
        for (uint32_t m = 0; m < 128; ++m)
            for (int e = -20; e <= 16; e += 12)
                tensor_scale(mxq::tensor_scale_from(ldexpf(mxq::u2f(0x3F800000u | (m << 16)), e), f ? 114688.0f : 448.0f));
    printf("tensor_scales_of_bf16_absmax cases=%ld bad=%ld refused=%ld\n", g_n, g_bad, g_refused);
    g_n = g_bad = g_refused = 0;
    uint32_t s = 12345u;
    for (int i = 0; i < 1500; ++i) {
        s = s * 1664525u + 1013904223u;
        tensor_scale(mxq::u2f(((67u + (s >> 25)) << 23) | ((s >> 1) & 0x7FFFFFu)));
        const float td = (1.0f + 0.125f * (s & 7u)) * (1.0f + 0.25f * ((s >> 3) & 3u));      /* and T's with a pair close to a tie */
        tensor_scale(mxq::u2f(mxq::f2u(mxq::u2f(0x3F800000u | ((s >> 9) & 0x7F0000u)) / td) + ((s >> 5) & 3u) - 1u));
    }
    const float edges[7] = {1.0f, 0x1p-60f, 0x1p60f, 0x1p-61f, 0x1.fffffep3f, 3.0f, 0.1f};
    for (int i = 0; i < 7; ++i) tensor_scale(edges[i]);
    printf("tensor_scales cases=%ld bad=%ld refused=%ld\n", g_n, g_bad, g_refused);
}

/* Powers of two: every bf16 value, zeros, subnormals and infinities among them, bits of the quotient (NaN: a NaN). */
static void powers_of_two(void)
{
    long n = 0, bad = 0;
    for (int k = -60; k <= 60; ++k) {
        const float T = ldexpf(1.0f, k);
        const mxq::Recip r = mxq::lean_recip(T);
        for (uint32_t u = 0; u < 65536u; ++u, ++n) {
            const float x = mxq::u2f(u << 16), v = mxq::quot(x, r), w = x / T;
            bad += (x != x) ? v == v : mxq::f2u(v) != mxq::f2u(w);
        }
    }
    printf("powers_of_two cases=%ld bad=%ld\n", n, bad);
}

int main()
{
    bf16_values();
    tensor_scales();
    powers_of_two();
    return 0;
}
