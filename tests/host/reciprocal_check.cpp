/*
 * Element quotients from a hardware reciprocal (mxq_arith.hpp: make_recip_from) on the CPU: the E2M1
 * decision for v / S must be the exact one whatever the last bit of the approximation is, and a quotient
 * of zero keeps the sign of v.  For every scale mantissa, twelve exponents and an approximation that is
 * one ulp low, nearest, and one ulp high: every tie t * S and its 64 neighbours on either side, 2^15 values
 * spread over seven binades (other mantissas at every exponent, 12 * 2^15 for each scale mantissa and
 * approximation), all of these with both signs, both zeros and values whose products underflow.
 * Prints "<name> cases=<n> bad=<m>".
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2605_08565_amd/csrc/mxq_arith.hpp"

static const double kTie[7] = {0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0};
static const int kUp[7] = {0, 1, 0, 1, 0, 1, 0};           /* the even code lies above the tie */

static int index_of(double y)
{
    int m = 0;
    for (int i = 0; i < 7; ++i) m += kUp[i] ? (y >= kTie[i]) : (y > kTie[i]);
    return m;
}
static int index_exact(double v, double S)
{
    int m = 0;
    for (int i = 0; i < 7; ++i) m += kUp[i] ? (v >= kTie[i] * S) : (v > kTie[i] * S);
    return m;
}

static const uint32_t kTiny[5] = {0u, 1u, 0x00400000u, 0x00800000u, 0x01000001u};
static long g_n = 0, g_bad = 0;

static void one(float v, float S, const mxq::Recip r)
{
    const float y = mxq::quot(v, r), z = mxq::quot(-v, r);
    ++g_n;
    g_bad += index_of(y) != index_exact(v, S) || signbit(y) || z != -y || !signbit(z);
}

int main()
{
    for (int mi = 0; mi < 8; ++mi)
        for (int ex = -17, round = 0; ex <= 16; ex += 3, ++round)
            for (int off = -1; off <= 1; ++off) {
                const float S = ldexpf(1.0f + mi * 0.125f, ex);
                const mxq::Recip r = mxq::make_recip_from(S, mxq::u2f(mxq::f2u(1.0f / S) + (uint32_t)off));
                if (!(r.hi > 0.0f && r.lo >= 0.0f)) ++g_bad;
                for (int i = 0; i < 7; ++i)
                    for (int d = -64; d <= 64; ++d) one(mxq::u2f(mxq::f2u((float)(kTie[i] * S)) + (uint32_t)d), S, r);
                for (uint32_t j = 0; j < (1u << 15); ++j) one(mxq::u2f(mxq::f2u(S) - (4u << 23) + j * 1723u + (uint32_t)round * 143u), S, r);
                for (const uint32_t bits : kTiny) one(mxq::u2f(bits), S, r);
            }
    printf("reciprocal_quotient cases=%ld bad=%ld\n", g_n, g_bad);
    return g_bad != 0;
}
