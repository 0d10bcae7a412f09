/*
 * Exact squares of residuals (mxq_arith.hpp): where the header says that they are exact, a square and its sum with another
 * in one fused multiply-add have the bits of the separately rounded operations.  Every bf16 magnitude that the rules let
 * pass, zero among them, under every scale code of both formats that kExactScales allows for it, beside random other
 * residuals of the same scale.  Beyond the rules the two must differ somewhere, or the inputs show nothing.
 * Prints "<name> cases=<n> differ=<m>".
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2605_08565_amd/csrc/mxq_arith.hpp"

using namespace mxq;

static float residual(float v, float S)                     /* under the nearest E2M1 value, ties to even */
{
    static const float grid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};
    static const double tie[7] = {0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0};
    const double y = fabs((double)v) / (double)S;
    int m = 0;
    for (int i = 0; i < 7; ++i) m += (i & 1) ? (y >= tie[i]) : (y > tie[i]);
    return fmaf(-copysignf(grid[m], v), S, v);
}

static uint64_t g_rng = 88172645463325252ull;
static uint32_t next()
{
    g_rng ^= g_rng << 13; g_rng ^= g_rng >> 7; g_rng ^= g_rng << 17;
    return (uint32_t)(g_rng >> 32);
}

static bool small_enough(float v, float S) { return v < kExactScales * S; }
static bool large_enough(float v) { return square_rank(f2u(v)) >= kSmallestSquareRank; }

template <int BIAS, int MAX>
static void run(const char* name)
{
    long n = 0, differ = 0, n_small = 0, differ_small = 0, n_large = 0, differ_large = 0;
    for (uint32_t code = 1u; code <= (uint32_t)MAX; ++code) {
        const float S = walk_scale_bias<BIAS>(code);
        for (uint32_t b = 0u; b < 0x7F80u; ++b) {
            const float v = u2f(b << 16);
            /* a neighbour of like magnitude, so that neither square is lost in the sum, and one of any magnitude */
            for (int k = 0; k < 2; ++k) {
                const uint32_t near = b + next() % 256u - (b < 256u ? 0u : 128u);
                const float other = u2f((k == 0 ? (near < 0x7F80u ? near : b) : next() % 0x7F80u) << 16);
                const float e = residual(v, S), f = residual(other, S);
                const bool same = f2u(fmaf(e, e, f * f)) == f2u(e * e + f * f);
                const bool low = large_enough(v) && large_enough(other), high = small_enough(v, S) && small_enough(other, S);
                if (!(f * f < INFINITY && e * e < INFINITY)) continue;
                if (low && high) { ++n; differ += !same; }
                else if (high) { ++n_small; differ_small += !same; }
                else if (low) { ++n_large; differ_large += !same; }
            }
        }
    }
    printf("%s_inside cases=%ld differ=%ld\n", name, n, differ);
    printf("%s_too_small cases=%ld differ=%ld\n", name, n_small, differ_small);
    printf("%s_too_large cases=%ld differ=%ld\n", name, n_large, differ_large);
}

int main()
{
    printf("zeros cases=2 differ=%d\n", (int)!(large_enough(0.0f) && large_enough(-0.0f)));
    printf("edge cases=3 differ=%d\n", (int)!(large_enough(kSmallestSquared) && !large_enough(u2f(f2u(kSmallestSquared) - 1u)) && !large_enough(u2f(1u))));
    run<7, 0x7E>("e4m3");
    run<15, 0xFE>("ue5m3");
    return 0;
}
