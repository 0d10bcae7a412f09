/*
 * The pruned scale search on the CPU, one block at a time, with the scalar rules of mxq_arith.hpp that
 * the kernel uses (walk_scale_bias, walk_halved, walk_last_odd, saturation_loss, walk_patience, the
 * quotients) and the kernel's order of steps: abs-max code, up, down, with a floor for long ways down.  The winner and its
 * SSE must be those of the full enumeration, and no block may cost many candidates.
 *
 * Blocks: every scale code times the factors at which the rules switch and their neighbours, over grid
 * points and ties; random blocks of every magnitude from 2^-40 to overflow; NaN and infinity.
 * Prints "<name> cases=<n> bad=<m> most=<candidates of the costliest block>".
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "../../paper_2605_08565_amd/csrc/mxq_arith.hpp"

using namespace mxq;

static const float kGrid[8] = {0.0f, 0.5f, 1.0f, 1.5f, 2.0f, 3.0f, 4.0f, 6.0f};

static float e2m1(float y)                                  /* nearest even code, saturating */
{
    const float a = fabsf(y);
    int m = 0;
    static const float tie[7] = {0.25f, 0.75f, 1.25f, 1.75f, 2.5f, 3.5f, 5.0f};
    for (int i = 0; i < 7; ++i) m += (i & 1) ? (a >= tie[i]) : (a > tie[i]);
    return copysignf(kGrid[m], y);
}

static float tree(std::vector<float> s)
{
    for (size_t n = s.size(); n > 1; n /= 2)
        for (size_t i = 0; i < n / 2; ++i) s[i] = s[2 * i] + s[2 * i + 1];
    return s[0];
}

template <int BIAS, int MAX, bool ONE_MUL> struct Search {
    std::vector<float> v;
    int tried = 0;

    float sse(uint32_t code, bool exact = false)
    {
        const float S = walk_scale_bias<BIAS>(code);
        const Recip r = make_recip_from(S, 1.0f / S);
        std::vector<float> sq(v.size());
        for (size_t i = 0; i < v.size(); ++i) {
            const float y = (ONE_MUL && !exact) ? v[i] * (1.0f / S) : quot(v[i], r);
            const float e = fmaf(-e2m1(y), S, v[i]);
            sq[i] = e * e;
        }
        return tree(sq);
    }
    float loss(uint32_t code)
    {
        std::vector<float> sq(v.size());
        for (size_t i = 0; i < v.size(); ++i) sq[i] = saturation_loss(v[i], walk_scale_bias<BIAS>(code));
        return tree(sq);
    }

    void full(uint32_t& best, float& best_sse)
    {
        best = 1u;
        best_sse = INFINITY;
        for (uint32_t c = 1u; c <= (uint32_t)MAX; ++c) {
            const float s = sse(c, true);
            if (s < best_sse) { best = c; best_sse = s; }
        }
    }

    void walk(uint32_t& best, float& best_sse)
    {
        float amax = 0.0f;
        for (float x : v) amax = fmaxf(amax, fabsf(x));
        const float top = walk_scale_bias<BIAS>(MAX);
        uint32_t start = sf_encode_bits<BIAS>(fminf(sixth_of(amax), top));
        if (start < 1u) start = 1u;
        uint32_t halved = walk_halved<BIAS>(sf_encode_bits<BIAS>(fminf(amax * kHalvedAt, top)), amax), floor = 1u;
        const bool low = start < 16u || start + 7u > (uint32_t)MAX;
        auto up = [&](uint32_t c) { ++tried; const float s = sse(c); if (s < best_sse) { best = c; best_sse = s; } };

        const float first = sse(start);
        ++tried;
        best = first < INFINITY ? start : 1u;
        best_sse = first < INFINITY ? first : INFINITY;
        if (!(first < INFINITY) && (first != first || loss(start) == INFINITY)) { start = 1u; halved = 1u; amax = 0.0f; }
        if (!low) {
            for (uint32_t i = 1u; i <= 7u; ++i) {
                if (i > 4u && start + i >= halved) break;
                up(start + i);
            }
        } else {
            const uint32_t last_odd = walk_last_odd<BIAS>(amax);
            for (uint32_t c = start;;) {
                c += 1u;
                const bool below = c < halved;
                c = below ? c : (c | 1u);
                const bool go = below || c <= last_odd;
                c = c < (uint32_t)MAX ? c : (uint32_t)MAX;
                if (!go) break;
                up(c);
            }
        }
        for (uint32_t c = start, step = 0u;; ++step) {
            if (step == walk_patience((int)v.size())) {
                uint32_t hi = c;
                const float reached = loss(c);
                for (uint32_t range = MAX; range != 0u; range >>= 1) {
                    const uint32_t mid = (floor + hi) >> 1;
                    if (loss(mid) > best_sse) floor = (mid + 1u < hi) ? mid + 1u : hi; else hi = mid;
                }
                floor = hi;
                ++tried;
                const float s = sse(floor);
                if (s <= reached && s <= best_sse) { best = floor; best_sse = s; c = floor; }
            }
            if (c <= floor) break;
            c -= 1u;
            const float over = amax - 6.0f * walk_scale_bias<BIAS>(c);
            if (over > 0.0f && over * over > best_sse) break;
            ++tried;
            const float s = sse(c);
            if (s <= best_sse) { best = c; best_sse = s; }
        }
    }
};

static uint64_t g_rng = 88172645463325252ull;
static double uniform()
{
    g_rng ^= g_rng << 13; g_rng ^= g_rng >> 7; g_rng ^= g_rng << 17;
    return (double)(g_rng >> 11) * 0x1p-53;
}
static double normal() { return sqrt(-2.0 * log(uniform() + 1e-300)) * cos(6.283185307179586 * uniform()); }
static float as_bf16(float f) { return u2f(f2u(f) & 0xFFFF0000u); }

struct Count { long n = 0, bad = 0; int most = 0; };

template <int BIAS, int MAX, bool BF16>
static void one(Count& c, std::vector<float> v)
{
    if (BF16) for (float& x : v) x = as_bf16(x);
    Search<BIAS, MAX, BF16> s;
    s.v = v;
    uint32_t a, b;
    float x, y;
    s.full(a, x);
    s.walk(b, y);
    ++c.n;
    if (a != b || f2u(x) != f2u(y)) {
        if (c.bad++ < 5) printf("  bias %d b %zu: code %u sse %g, full search %u %g; v0 = %a\n", BIAS, v.size(), b, y, a, x, v[0]);
    }
    if (s.tried > c.most) c.most = s.tried;
}

template <int BIAS, int MAX, bool BF16>
static void run(const char* fmt)
{
    const int sizes[4] = {2, 4, 16, 128};
    Count edges, inside, beyond, special;
    /* the factors of a scale at which a rule switches, and the neighbours of the abs-max there */
    for (uint32_t code = 1u; code <= (uint32_t)MAX; ++code) {
        const float S = walk_scale_bias<BIAS>(code), factors[6] = {3.5f, 4.0f, 5.0f, 6.0f, 0.25f, 40.0f};
        for (float f : factors)
            for (int d = -1; d <= 1; ++d)
                for (int b : {2, 16}) {
                    const float amax = BF16 ? u2f((f2u(f * S) & 0xFFFF0000u) + (uint32_t)(d * 65536)) : u2f(f2u(f * S) + (uint32_t)d);
                    std::vector<float> v(b);
                    for (float& x : v) x = fminf(0.25f * (float)(int)(uniform() * 15.0) * S, amax) * (uniform() < 0.5 ? -1.0f : 1.0f);
                    v[(int)(uniform() * b)] = amax;
                    one<BIAS, MAX, BF16>(edges, v);
                }
    }
    for (int e = -40; e <= 126; e += 3)
        for (int b : sizes)
            for (int kind = 0; kind < 6; ++kind)
                for (int rep = 0; rep < (b == 128 ? 2 : 8); ++rep) {
                    std::vector<float> v(b);
                    for (int i = 0; i < b; ++i) {
                        double z = normal();
                        if (kind == 1) z = 1.0 + 0.05 * uniform();                        /* all alike */
                        if (kind == 2) z = 1.0;
                        if (kind == 3 && i == 0) z = 50.0;                                /* one outlier */
                        if (kind == 4) z *= pow(2.0, -20.0 * uniform());                  /* magnitudes mixed */
                        if (kind == 5) z *= (i & 1) ? 1.0 : 0x1p-12;
                        v[i] = (float)ldexp(z, e);
                        if (!isfinite(v[i])) v[i] = 3e38f;
                    }
                    float amax = 0.0f;
                    for (float x : v) amax = fmaxf(amax, fabsf(x));
                    one<BIAS, MAX, BF16>(amax > 6.0f * walk_scale_bias<BIAS>(MAX) ? beyond : inside, v);
                }
    for (int b : sizes)
        for (float x : {NAN, INFINITY, -INFINITY, 3e38f, 1.8e19f, 1.9e19f})
            for (float scale : {0.0f, 1e-5f, 1.0f, 1e5f, 1e18f, 3e37f}) {
                std::vector<float> v(b);
                for (float& y : v) y = (float)normal() * scale;
                v[(int)(uniform() * b)] = x;
                one<BIAS, MAX, BF16>(special, v);
            }
    const struct { const char* name; Count* c; } all[4] = {{"edges", &edges}, {"inside", &inside}, {"beyond", &beyond}, {"special", &special}};
    for (auto& a : all) printf("%s_%s_%s cases=%ld bad=%ld most=%d\n", fmt, BF16 ? "bf16" : "f32", a.name, a.c->n, a.c->bad, a.c->most);
}

int main()
{
    run<7, 0x7E, false>("e4m3");
    run<7, 0x7E, true>("e4m3");
    run<15, 0xFE, false>("ue5m3");
    run<15, 0xFE, true>("ue5m3");
    return 0;
}
