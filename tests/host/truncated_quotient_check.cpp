/*
 * Element quotients by one truncated product (mxq_arith.hpp: quot_truncated) on the CPU: for every bf16 value
 * of both signs and every scale code of E4M3 and UE5M3 the E2M1 decision must be the exact one and the
 * quotient must keep the sign of the value.  Prints "<name> cases=<n> bad=<m>".
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

int main()
{
    bf16_values();
    return 0;
}
