/*
 * The pruned scale search on the CPU, one block at a time, with the scalar rules of mxq_arith.hpp that
 * the kernel uses (walk_scale_bias, walk_halved, walk_last_odd, saturation_loss, walk_patience, window_first, window_steps,
 * the quotients) and the kernel's order of steps: blocks that the window takes try its eight codes mantissa by mantissa, the
 * one above where it is needed and up to kWindowDown below, the best kept by the order of (SSE, scale) pairs as doubles;
 * the others the abs-max code, up; both go on down from there, with a floor for long ways.  The winner and its
 * SSE must be those of the full enumeration, and no block may cost many candidates.
 *
 * Blocks: every scale code times the factors at which the rules switch and their neighbours, over grid
 * points and ties; random blocks of every magnitude from 2^-40 to overflow; NaN and infinity.
 * Prints "<name> cases=<n> bad=<m> most=<candidates of the costliest block that does not go on down behind its
 * window> window=<blocks that it decided> on=<blocks that went on down behind it> most_on=<candidates of the costliest of these> far=<abs-max over the lowest scale tried where squares count as exact>".
 */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

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
    bool in_window = false, went_on = false;
    float far = 0.0f;                                       /* amax over the lowest scale tried before the patience is out */

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
    /* Under the same code from quotients by its mantissa alone, as in the window. */
    float sse_by_mantissa(uint32_t code)
    {
        const float m = 1.0f + 0.125f * (float)(code & 7u), pow2 = walk_scale_bias<BIAS>(code) / m;
        const double inverse = 1.0 / (double)m;
        const float hi = (double)(float)inverse > inverse ? u2f(f2u((float)inverse) - 1u) : (float)inverse;
        const Recip r{hi, (float)(inverse - (double)hi)};
        std::vector<float> sq(v.size());
        for (size_t i = 0; i < v.size(); ++i) {
            const float w = (code & 7u) == 0u ? v[i] : ONE_MUL ? v[i] * (1.0f / m) : quot(v[i], r);
            const float e = fmaf(-(e2m1(w / pow2) * pow2), m, v[i]);
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

    /* The window and the codes below it.  False: all codes are still to be tried.  `done`: over; else the walk goes on down
       from `code`. */
    bool window(uint32_t& best, float& best_sse, float amax, uint32_t start, uint32_t& code, bool& done)
    {
        if (start < 17u || amax > 6.5f * walk_scale_bias<BIAS>(MAX)) return false;
        const uint32_t first = window_first(start, (uint32_t)MAX), above = first + 8u;
        uint64_t least = (uint64_t)0x7F800000u << 32;
        auto keep = [&](uint32_t c, float s) {
            ++tried;
            const uint64_t other = ((uint64_t)f2u(s) << 32) | c;
            double x, y;
            memcpy(&x, &least, 8);
            memcpy(&y, &other, 8);
            x = fmin(x, y);
            memcpy(&least, &x, 8);
        };
        for (uint32_t m = 0u; m < 8u; ++m) {
            const uint32_t c = ((first + 7u - m) & ~7u) | m;
            keep(c, sse_by_mantissa(c));
        }
        if (above <= (uint32_t)MAX && 3.5f * walk_scale_bias<BIAS>(above) < amax) keep(above, sse(above));
        done = false;
        code = first;
        for (uint32_t i = 0u; i < kWindowDown; ++i) {
            code -= 1u;
            const float over = fmaf(-6.0f, walk_scale_bias<BIAS>(code), amax);
            if (over * fabsf(over) > u2f((uint32_t)(least >> 32))) { done = true; break; }
            far = fmaxf(far, amax / walk_scale_bias<BIAS>(code));
            keep(code, sse(code));
        }
        best = (uint32_t)least;
        best_sse = u2f((uint32_t)(least >> 32));
        return best_sse < INFINITY;
    }

    void walk(uint32_t& best, float& best_sse)
    {
        float amax = 0.0f;
        for (float x : v) amax = fmaxf(amax, fabsf(x));
        const float top = walk_scale_bias<BIAS>(MAX);
        uint32_t start = sf_encode_bits<BIAS>(fminf(sixth_of(amax), top)), code = 0u, step = 0u;
        bool done = false;
        if (window(best, best_sse, amax, start, code, done)) {
            in_window = true;
            if (done) return;
            went_on = true;
            step = window_steps((int)v.size());
        } else {
            up_from(best, best_sse, amax, start, top);
            code = start;
        }
        down_from(best, best_sse, amax, code, step);
    }

    void up_from(uint32_t& best, float& best_sse, float& amax, uint32_t& start, float top)
    {
        if (start < 1u) start = 1u;
        uint32_t halved = walk_halved<BIAS>(sf_encode_bits<BIAS>(fminf(amax * kHalvedAt, top)), amax);
        const float first = sse(start);
        ++tried;
        best = first < INFINITY ? start : 1u;
        best_sse = first < INFINITY ? first : INFINITY;
        if (!(first < INFINITY) && (first != first || loss(start) == INFINITY)) { start = 1u; halved = 1u; amax = 0.0f; }
        const uint32_t last_odd = walk_last_odd<BIAS>(amax);
        for (uint32_t c = start;;) {
            c += 1u;
            const bool below = c < halved;
            c = below ? c : (c | 1u);
            const bool go = below || c <= last_odd;
            c = c < (uint32_t)MAX ? c : (uint32_t)MAX;
            if (!go) break;
            ++tried;
            const float s = sse(c);
            if (s < best_sse) { best = c; best_sse = s; }
        }
    }

    void down_from(uint32_t& best, float& best_sse, float amax, uint32_t c, uint32_t step)
    {
        uint32_t floor = 1u;
        for (;; ++step) {
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
            if (step < walk_patience((int)v.size())) far = fmaxf(far, amax / walk_scale_bias<BIAS>(c));
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

struct Count { long n = 0, bad = 0, window = 0, on = 0; int most = 0, most_on = 0; float far = 0.0f; };

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
    int& most = s.went_on ? c.most_on : c.most;
    if (s.tried > most) most = s.tried;
    c.window += s.in_window;
    c.on += s.went_on;
    float amax = 0.0f;
    for (float x : v) amax = fmaxf(amax, fabsf(x));
    if (amax < kExactScales * walk_scale_bias<BIAS>(MAX)) c.far = fmaxf(c.far, s.far);
}

template <int BIAS, int MAX, bool BF16>
static void run(const char* fmt)
{
    const int sizes[5] = {2, 4, 16, 32, 128};
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
            for (int kind = 0; kind < 8; ++kind)
                for (int rep = 0; rep < (b >= 32 ? 2 : 8); ++rep) {
                    std::vector<float> v(b);
                    for (int i = 0; i < b; ++i) {
                        double z = normal();
                        if (kind == 1) z = 1.0 + 0.05 * uniform();                        /* all alike */
                        if (kind == 2) z = 1.0;
                        if (kind == 3 && i == 0) z = 50.0;                                /* one outlier */
                        if (kind == 4) z *= pow(2.0, -20.0 * uniform());                  /* magnitudes mixed */
                        if (kind == 5) z *= (i & 1) ? 1.0 : 0x1p-12;
                        if (kind == 6) z = 2.0 * uniform() - 1.0;                         /* light tails: a long way down */
                        if (kind == 7) z = i == 0 ? 6.0 : uniform() < 0.5 ? 5.0 : -2.5;   /* on ties under the abs-max code */
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
    for (auto& a : all)
        printf("%s_%s_%s cases=%ld bad=%ld most=%d window=%ld on=%ld most_on=%d far=%.9g\n", fmt, BF16 ? "bf16" : "f32", a.name, a.c->n, a.c->bad,
               a.c->most, a.c->window, a.c->on, a.c->most_on, a.c->far);
}

int main()
{
    run<7, 0x7E, false>("e4m3");
    run<7, 0x7E, true>("e4m3");
    run<15, 0xFE, false>("ue5m3");
    run<15, 0xFE, true>("ue5m3");
    return 0;
}
