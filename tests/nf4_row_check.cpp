// nf4_row_check.cpp — TEST INFRASTRUCTURE ONLY: the row table of nf4.hpp and
// the lookup arithmetic of the NF4 engine kernels (nf4_ops.hpp) replayed on
// the host over every float x with |x| <= 1 + 2^-22, and the general lookup
// over special values too. Each code is compared with the number of
// midpoints strictly below x (read from stdin as in nf4_table_check.cpp).
// Fast mode's form takes x = w r unrounded: replayed over weights next to the
// midpoints of blocks of many maxima m, with r = 1 / m and both floats beside
// it, in gathers of four different elements, each of which must come out with
// its own code (the product has at most 48 bits, so double compares it exactly).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "nf4.hpp"

static uint32_t bits(float x)
{
    uint32_t u;
    std::memcpy(&u, &x, 4);
    return u;
}

static float from_bits(uint32_t u)
{
    float x;
    std::memcpy(&x, &u, 4);
    return x;
}

using mezo::kNF4RowMagic;
using mezo::kNF4RowMask;
using mezo::kNF4Rows;
using mezo::kNF4Steep;

static uint32_t code_usual(float x)
{
    const uint32_t off = bits(std::fmaf(x, 512.0f, kNF4RowMagic)) & kNF4RowMask;
    if (off / 8 >= uint32_t(kNF4Rows)) return 99;  // past the table
    const mezo::NF4Row& e = mezo::kNF4RowTable.row[off / 8];
    const float up = std::fmin(std::fmax(std::fmaf(x, kNF4Steep, e.thr), 0.0f), 1.0f);
    // the gathered code of four equal elements: exact, in the low 16 bits
    float g = 128.0f;
    for (int j = 0; j < 4; ++j) g = std::fmaf(g, 16.0f, e.lo) + up;
    const uint32_t p = bits(g) & 0xFFFFu;
    return p == (p & 15u) * 0x1111u ? (p & 15u) : 99u;
}

static uint32_t code_general(float x)
{
    const float xs = x == x ? x : -2.0f;
    const int k = int(bits(std::fmaf(xs, 512.0f, kNF4RowMagic))) - int(mezo::kNF4BinBase);
    const uint32_t off = uint32_t(k < 0 ? 0 : (k > 1028 ? 1028 : k)) & kNF4RowMask;
    const mezo::NF4Row& e = mezo::kNF4RowTable.row[off / 8];
    return uint32_t(e.lo) + (std::fmaf(x, kNF4Steep, e.thr) > 0.0f ? 1u : 0u);
}

// Fast mode's gathered codes of w[0 .. 3] in a block of reciprocal r.
static uint32_t codes_fast(const float (&w)[4], float r)
{
    const float r512 = r * 512.0f, rs = r * kNF4Steep;
    float g = 0.0f;
    for (int j = 3; j >= 0; --j) {
        const uint32_t off = bits(std::fmaf(w[j], r512, kNF4RowMagic)) & kNF4RowMask;
        if (off / 8 >= uint32_t(kNF4Rows)) return 0xFFFFFFFFu;  // past the table
        const mezo::NF4Row& e = mezo::kNF4RowTable.row[off / 8];
        const float up = std::fmin(std::fmax(std::fmaf(w[j], rs, e.thr), 0.0f), 1.0f);
        g = std::fmaf(j == 3 ? 128.0f : g, 16.0f, e.lo) + up;
    }
    return bits(g) & 0xFFFFu;
}

static uint64_t g_state = 1;
static uint32_t rnd()
{
    g_state = g_state * 6364136223846793005ull + 1442695040888963407ull;
    return uint32_t(g_state >> 32);
}

int main()
{
    float mid[15];
    for (int i = 0; i < 15; ++i) {
        unsigned u;
        if (std::scanf("%x", &u) != 1) return 2;
        mid[i] = from_bits(u);
    }
    const auto want = [&](float x) {
        uint32_t c = 0;
        for (int i = 0; i < 15; ++i) c += mid[i] < x ? 1u : 0u;
        return c;
    };
    unsigned long long bad = 0, n = 0;
    const uint32_t end = bits(1.0f) + 3, threads = 8;  // past 1 + 2^-22
    std::vector<unsigned long long> wrong(threads, 0);
    std::vector<std::thread> pool;
    for (uint32_t t = 0; t < threads; ++t)
        pool.emplace_back([&, t] {
            unsigned long long b = 0;
            for (uint32_t m = t; m < end; m += threads)
                for (uint32_t s = 0; s < 2; ++s) {
                    const float x = from_bits(m | (s << 31));
                    const uint32_t w = want(x);
                    b += code_usual(x) != w;
                    b += code_general(x) != w;
                }
            wrong[t] = b;
        });
    for (auto& t : pool) t.join();
    for (unsigned long long b : wrong) bad += b;
    n = 2ull * end;
    const float special[] = {0.0f,   -0.0f, 1e-30f, -1e-30f, 1e-45f, INFINITY, -INFINITY, NAN,
                             3.4e38f, -3.4e38f, 2.0f, -2.0f, 1e6f, -1e6f};
    for (float x : special) {
        const uint32_t w = x == x ? want(x) : 0u;  // NaN: no midpoint is below it
        bad += code_general(x) != w;
        if (std::fabs(x) <= 1.0f) bad += code_usual(x) != w;
        ++n;
    }
    // fast mode: four different elements against their own codes, the one next
    // to a midpoint in every place of the gather
    unsigned long long fast = 0, bad_fast = 0;
    const auto want_product = [&](float w, float r) {
        uint32_t c = 0;
        for (int i = 0; i < 15; ++i) c += double(mid[i]) < double(w) * double(r) ? 1u : 0u;
        return c;
    };
    const auto check_fast = [&](float near, float m, float r, int place) {
        float w[4];
        for (int j = 0; j < 4; ++j) w[j] = m * (float(int32_t(rnd())) * 0x1p-31f);
        w[(place + 1) & 3] = 0.0f;
        w[place] = near;
        uint32_t c = 0;
        for (int j = 0; j < 4; ++j) c |= want_product(w[j], r) << (4 * j);
        ++fast;
        bad_fast += codes_fast(w, r) != c;
    };
    // products a hair above a midpoint
    const float pairs[][2] = {{0x1.60bc6cp-5f, 0x1.c1222cp-10f}, {0x1.4a47d6p-5f, -0x1.6c657ep-8f}};
    for (const auto& p : pairs)
        for (int place = 0; place < 4; ++place) check_fast(p[1], p[0], 1.0f / p[0], place);
    for (uint32_t k = 0; k < (1u << 21); ++k) {
        // a maximum in [2^-64, 2^64), one in eight of an ordinary weight's size
        const int ex = k & 7 ? int(rnd() % 128u) - 64 : -5;
        const float m = std::ldexp(1.0f + float(rnd() >> 9) * 0x1p-23f, ex);
        const float inv = 1.0f / m;
        for (int d = -1; d <= 1; ++d) {
            const float r = from_bits(bits(inv) + uint32_t(d));
            const int i = int(rnd() % 15u);
            const float at = float(double(mid[i]) / double(r));
            for (int e = -1; e <= 1; ++e) check_fast(from_bits(bits(at) + uint32_t(e)), m, r, int(k & 3u));
        }
    }
    std::printf("fast mode: %llu gathers, %llu wrong\n", fast, bad_fast);
    bad += bad_fast;
    std::printf("%llu values, %llu mismatches\n", n, bad);
    return bad ? 1 : 0;
}
