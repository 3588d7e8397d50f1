// nf4.hpp — the 4-bit NormalFloat storage of the 4-bit forward-only variant
// (Section 3: weights dequantized before the noise is added and quantized
// again afterwards, in QLoRA's 4-bit format, which the paper cites there).
//
// The 16 values are QLoRA's NF4: quantiles of N(0, 1) for an asymmetric pair
// of halves (8 positive, 7 negative, an exact zero), scaled to [-1, 1],
// rounded to fp32. Quantizing x in [-1, 1] picks the nearest value, a tie
// going to the lower code: code = number of midpoints m_i = fl32((v_i +
// v_{i+1}) / 2) strictly below x.
//
// Fast exact lookup: x maps to one of a few more than 128 bins by a
// monotone function b(x), and no bin holds two midpoints (the values are more
// than 1/64 apart). For x in bin b, every midpoint in a lower bin is below x
// and every midpoint in a higher bin above it, so code = (midpoints in bins
// below b) + (x > the midpoint in bin b, if any). The tables are built at
// compile time from the same b() the kernels evaluate. Three bin functions:
//
// - kNF4RowTable, 129 rows, used by the engine's kernels: b(x) = (the integer
//   nearest to 512 x + 516) / 8, whole part. One fma gives the integer as the
//   low bits of t = fl32(512 x + kNF4RowMagic), kNF4RowMagic = 1.5 * 2^23 + 516,
//   and t & kNF4RowMask is 8 b, the byte offset of the row. For |x| <= 1 +
//   2^-22, b is in [0, 128] with no clamp. A row holds what the code takes in
//   float arithmetic, whose instructions issue in pairs where compares and
//   integer packing issue alone: code = lo + clamp(2^60 x + thr, 0, 1) with
//   thr = -2^60 midpoint (-inf for a row without one). The clamp must give 0 or
//   1 and never a fraction, which would carry into the codes gathered beside
//   it: the fma has the sign of x - midpoint, and where that is not zero it is
//   at least 2^8. In a row with a midpoint |x| > 2^-5, so a float x and the
//   midpoint are multiples of 2^-28; fast mode's x, the unrounded product w r
//   of two floats, has 48 bits and is a multiple of 2^-52. (r <= 2^64, so 2^60 r
//   is finite.)
// - kNF4Table, 128 bins: b(x) = floor(fl32(64 x + 64)) clamped to [0, 127]
//   (fma rounds 64 x + 64 once, exactly as the double expression below
//   rounded to float does); the rule the row table is checked against below.
// - kNF4RoundTable, 129 bins: b(x) = the integer nearest to 64 x + 64 (ties to
//   even), which one fma gives directly: t = fl32(64 x + kNF4BinMagic),
//   kNF4BinMagic = 1.5 * 2^23 + 64, lies in [2^23, 2^24) where floats are 1
//   apart, so t is 64 x + 64 rounded once to the nearest integer plus 1.5 *
//   2^23, and the bit pattern of t is kNF4BinBase + b. For |x| <= 1 + 2^-23
//   (every x of a block whose maximum has a normal reciprocal), b is in
//   [0, 128] with no clamp; used by the standalone quantization.
#pragma once

#include <stdint.h>

#include "records.hpp"

namespace mezo {

constexpr int kNF4Codes = 16;
constexpr uint32_t kNF4ZeroCode = 7;
constexpr int kNF4Bins = 128;
constexpr int kNF4RoundBins = 129;
constexpr float kNF4BinMagic = 12582976.0f;      // 1.5 * 2^23 + 64
constexpr uint32_t kNF4BinBase = 0x4B400000u;    // bit pattern of 1.5 * 2^23
constexpr int kNF4Pairs = 256;                   // byte -> the values of its two codes

constexpr float kNF4Values[kNF4Codes] = {
    -0x1.000000p+0f, -0x1.647362p-1f, -0x1.0cd65cp-1f, -0x1.94653cp-2f,
    -0x1.234496p-2f, -0x1.7a6a7ap-3f, -0x1.74f0d2p-4f, 0.0f,
    0x1.45f602p-4f,  0x1.4995bep-3f,  0x1.f809b4p-3f,  0x1.5a066cp-2f,
    0x1.c3496ap-2f,  0x1.200f52p-1f,  0x1.722760p-1f,  0x1.000000p+0f,
};

constexpr float nf4_midpoint(int i)
{
    return static_cast<float>((double(kNF4Values[i]) + double(kNF4Values[i + 1])) * 0.5);
}

// b(x) as the kernels compute it: fma(x, 64, 64), truncated to int, clamped.
constexpr int nf4_bin_of(float x)
{
    const float t = static_cast<float>(double(x) * 64.0 + 64.0);
    const int b = static_cast<int>(t);
    return b < 0 ? 0 : (b > kNF4Bins - 1 ? kNF4Bins - 1 : b);
}

// The round-to-nearest bin function: 64 x + 64 (exact in double for a float
// x) rounded to the nearest integer, ties to even, clamped to [0, 128].
constexpr int nf4_round_bin_of(float x)
{
    const double t = double(x) * 64.0 + 64.0;
    if (t <= 0.0) return 0;
    if (t >= double(kNF4RoundBins - 1)) return kNF4RoundBins - 1;
    const int f = static_cast<int>(t);  // floor, t > 0
    const double d = t - double(f);
    return d > 0.5 ? f + 1 : (d < 0.5 ? f : (f % 2 == 0 ? f : f + 1));
}

// One bin: its midpoint (+inf if none) and the code below it.
struct alignas(8) NF4Bin {
    float mid;
    uint32_t lo;
};

template <int kBins>
struct NF4Table {
    NF4Bin bin[kBins];
    bool ok;  // no bin holds two midpoints
};

template <int kBins, int (*kBinOf)(float)>
constexpr NF4Table<kBins> make_nf4_table()
{
    NF4Table<kBins> t{};
    t.ok = true;
    for (int b = 0; b < kBins; ++b) {
        uint32_t lo = 0;
        int in_bin = 0;
        float mid = __builtin_huge_valf();
        for (int i = 0; i < kNF4Codes - 1; ++i) {
            const int mb = kBinOf(nf4_midpoint(i));
            if (mb < b) ++lo;
            if (mb == b) {
                mid = nf4_midpoint(i);
                ++in_bin;
            }
        }
        if (in_bin > 1) t.ok = false;
        t.bin[b].mid = mid;
        t.bin[b].lo = lo;
    }
    return t;
}

constexpr NF4Table<kNF4Bins> kNF4Table = make_nf4_table<kNF4Bins, nf4_bin_of>();
static_assert(kNF4Table.ok, "two NF4 midpoints share a bin");
static_assert(nf4_bin_of(-1.0f) == 0 && nf4_bin_of(1.0f) == kNF4Bins - 1, "bin range");

constexpr NF4Table<kNF4RoundBins> kNF4RoundTable = make_nf4_table<kNF4RoundBins, nf4_round_bin_of>();
static_assert(kNF4RoundTable.ok, "two NF4 midpoints share a bin");
// the extremes of a block with a normal reciprocal: |x| <= 1 + 2^-23
static_assert(nf4_round_bin_of(-1.00000012f) == 0 && nf4_round_bin_of(1.00000012f) == kNF4RoundBins - 1,
              "bin range");

// ---- the engine's row table -------------------------------------------------

constexpr int kNF4Rows = 129;
constexpr float kNF4RowMagic = 12583428.0f;  // 1.5 * 2^23 + 516
constexpr uint32_t kNF4RowMask = 0x7F8u;     // byte offset of the row in t's bit pattern
constexpr float kNF4Steep = 0x1p60f;

struct alignas(8) NF4Row {
    float thr;  // -2^60 midpoint, or -inf
    float lo;   // the code below the midpoint
};

// The row of x: 512 x + 516 (exact in double for a float x) rounded to the
// nearest integer, ties to even, over 8; clamped to [0, 128].
constexpr int nf4_row_of(float x)
{
    const double t = double(x) * 512.0 + 516.0;
    if (t <= 0.0) return 0;
    if (t >= 1028.0) return kNF4Rows - 1;
    const int f = static_cast<int>(t);
    const double d = t - double(f);
    return (d > 0.5 ? f + 1 : (d < 0.5 ? f : (f % 2 == 0 ? f : f + 1))) / 8;
}

struct NF4RowTable {
    NF4Row row[kNF4Rows];
    bool ok;  // no row holds two midpoints
};

constexpr NF4RowTable make_nf4_rows()
{
    NF4RowTable t{};
    t.ok = true;
    for (int b = 0; b < kNF4Rows; ++b) {
        int lo = 0, in_row = 0;
        t.row[b].thr = -__builtin_huge_valf();
        for (int i = 0; i < kNF4Codes - 1; ++i) {
            const int mb = nf4_row_of(nf4_midpoint(i));
            if (mb < b) ++lo;
            if (mb == b) {
                t.row[b].thr = -kNF4Steep * nf4_midpoint(i);
                ++in_row;
            }
        }
        if (in_row > 1) t.ok = false;
        t.row[b].lo = static_cast<float>(lo);
    }
    return t;
}
constexpr NF4RowTable kNF4RowTable = make_nf4_rows();
static_assert(kNF4RowTable.ok, "two NF4 midpoints share a row");
static_assert(nf4_row_of(-1.0f) == 0 && nf4_row_of(1.0f) == kNF4Rows - 1, "row range");
// |x| > 2^-5 in every row with a midpoint (what the slope is chosen for).
constexpr bool nf4_rows_near_zero_free()
{
    for (int b = nf4_row_of(-0x1p-5f); b <= nf4_row_of(0x1p-5f); ++b)
        if (kNF4RowTable.row[b].thr != -__builtin_huge_valf()) return false;
    return true;
}
static_assert(nf4_rows_near_zero_free(), "a midpoint's row reaches below 2^-5");

// The code of x by either table.
constexpr int nf4_row_code(float x)
{
    const NF4Row r = kNF4RowTable.row[nf4_row_of(x)];
    return static_cast<int>(r.lo) + (double(x) * double(kNF4Steep) + double(r.thr) > 0.0 ? 1 : 0);
}
constexpr int nf4_bin_code(float x)
{
    const NF4Bin b = kNF4Table.bin[nf4_bin_of(x)];
    return static_cast<int>(b.lo) + (x > b.mid ? 1 : 0);
}
// The two agree at every midpoint, on both sides of it, and at every row's edges.
constexpr bool nf4_tables_agree()
{
    for (int i = 0; i < kNF4Codes - 1; ++i)
        for (int d = -1; d <= 1; ++d) {
            const float x = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, nf4_midpoint(i)) + uint32_t(d));
            if (nf4_row_code(x) != nf4_bin_code(x)) return false;
        }
    for (int k = -1024; k <= 1024; ++k) {
        const float x = static_cast<float>(k) / 1024.0f;
        if (nf4_row_code(x) != nf4_bin_code(x)) return false;
    }
    return true;
}
static_assert(nf4_tables_agree(), "the row table's codes");
static_assert(__builtin_bit_cast(uint32_t, 12582912.0f) == kNF4BinBase, "magic base");
static_assert(kNF4RowMagic == 12582912.0f + 516.0f && (kNF4BinBase & 0x7FFu) == 0, "row magic");
static_assert(kNF4BinMagic == 12582912.0f + 64.0f, "magic constant");

}  // namespace mezo
