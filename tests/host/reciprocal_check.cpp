/*
 * Element quotients from a hardware reciprocal (mxq_arith.hpp: make_recip_from) on the CPU: the E2M1
 * decision for v / S must be the exact one whatever the last bit of the approximation is.  Every tie
 * t * S and its 64 neighbours on either side, and 2^20 values spread over the range, for every scale
 * mantissa and an approximation that is one ulp low, nearest, and one ulp high.
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

int main()
{
    long n = 0, bad = 0;
    for (int mi = 0; mi < 8; ++mi)
        for (int ex = -17; ex <= 16; ex += 3)
            for (int off = -1; off <= 1; ++off) {
                const float S = ldexpf(1.0f + mi * 0.125f, ex);
                const mxq::Recip r = mxq::make_recip_from(S, mxq::u2f(mxq::f2u(1.0f / S) + (uint32_t)off));
                if (!(r.hi > 0.0f && r.lo >= 0.0f)) ++bad;                 /* a zero quotient keeps its sign */
                for (int i = 0; i < 7; ++i)
                    for (int d = -64; d <= 64; ++d) {
                        const float v = mxq::u2f(mxq::f2u((float)(kTie[i] * S)) + (uint32_t)d);
                        ++n;
                        bad += index_of(mxq::quot(v, r)) != index_exact(v, S);
                    }
                for (uint32_t j = 0; j < (1u << 15); ++j) {
                    const float v = mxq::u2f(mxq::f2u(S) - (4u << 23) + j * 1723u);
                    ++n;
                    bad += index_of(mxq::quot(v, r)) != index_exact(v, S);
                }
            }
    printf("reciprocal_quotient cases=%ld bad=%ld\n", n, bad);
    return bad != 0;
}
