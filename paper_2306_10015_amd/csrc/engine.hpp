// engine.hpp — device-side building blocks of the seeded perturbation engine
// for gfx950 (MI355X): the Philox generator, the Gaussian transform and the
// storage conversions.
//
// z for (seed, tensor t, element e) is defined in include/mezo.h: Philox4x32-10
// with key = machine id and counter = (e >> 2, t, sample, step), then
// Box-Muller on 24-bit uniforms. The paper only requires an RNG that every
// machine can reset to the same seed and replay (Algorithm 1,
// PerturbParameters; Appendix B on reproducing noise across devices); a
// counter-based generator lets every lane compute its own elements' noise in
// registers, so z is never stored.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "engine_launch.hpp"
#include "records.hpp"

namespace mezo {

__device__ __forceinline__ void mul_wide(uint32_t m, uint32_t x, uint32_t& hi, uint32_t& lo)
{
    uint64_t p = uint64_t(m) * uint64_t(x);
    hi = uint32_t(p >> 32);
    lo = uint32_t(p);
}

// a ^ b ^ c in one gfx950 v_bitop3_b32 (truth table 0x96 = three-way xor).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Per-call values that are the same for every element of one tensor: the
// round-1 words that do not depend on the element, and the round-2 product
// of the (element-independent) word 0. All scalar.
struct SeedUniform {
    uint32_t y1;        // round-1 output word 1
    uint32_t kx;        // step ^ key1: folded into round-1 output word 2
    uint32_t r2_hi;     // round 2: high word of kMulA * y0
    uint32_t r2_lo;     // round 2: low  word of kMulA * y0 (= output word 3)
    uint32_t k0, k1;    // round-2 key
};

__device__ __forceinline__ SeedUniform seed_uniform(const SeedRec& r, uint32_t tensor_id)
{
    SeedUniform u;
    // Round 1 on counter (blk, t, sample, step) with key (key0, key1):
    //   word 0 = hi(kMulB*sample) ^ t ^ key0   (element-independent)
    //   word 1 = lo(kMulB*sample)              (element-independent)
    //   word 2 = hi(kMulA*blk) ^ step ^ key1   (per element)
    //   word 3 = lo(kMulA*blk)                 (per element, seed-independent)
    uint32_t y0 = r.mb_hi ^ tensor_id ^ r.key0;
    u.y1 = r.mb_lo;
    u.kx = r.step ^ r.key1;
    u.k0 = r.key0 + kWeylA;
    u.k1 = r.key1 + kWeylB;
    mul_wide(kMulA, y0, u.r2_hi, u.r2_lo);
    return u;
}

// Seed-independent part of round 1 for block blk: kMulA * blk.
struct BlockPre {
    uint32_t hi, lo;
};

__device__ __forceinline__ BlockPre block_pre(uint32_t blk)
{
    BlockPre b;
    mul_wide(kMulA, blk, b.hi, b.lo);
    return b;
}

// The four Philox4x32-10 output words of one block, from the hoisted round-1
// values: rounds 2..10 with the per-element products on the vector unit.
__device__ __forceinline__ void philox_words(const SeedUniform& u, BlockPre b, uint32_t& x0,
                                             uint32_t& x1, uint32_t& x2, uint32_t& x3)
{
    // end of round 1
    uint32_t y2 = b.hi ^ u.kx;
    uint32_t y3 = b.lo;
    // round 2 (key k0, k1): products kMulA*y0 (scalar, precomputed) and kMulB*y2
    uint32_t hb, lb;
    mul_wide(kMulB, y2, hb, lb);
    x0 = hb ^ u.y1 ^ u.k0;
    x1 = lb;
    x2 = u.r2_hi ^ y3 ^ u.k1;
    x3 = u.r2_lo;
    uint32_t k0 = u.k0, k1 = u.k1;
#pragma unroll
    for (int round = 3; round <= 10; ++round) {
        k0 += kWeylA;
        k1 += kWeylB;
        uint32_t ha, la;
        mul_wide(kMulA, x0, ha, la);
        mul_wide(kMulB, x2, hb, lb);
        const uint32_t n0 = xor3(hb, x1, k0);
        const uint32_t n2 = xor3(ha, x3, k1);
        x0 = n0;
        x1 = lb;
        x2 = n2;
        x3 = la;
    }
}

// ---- issue phases -----------------------------------------------------------
// What bounds the record loops is vector issue, and on gfx950 that is decided
// by which instructions share an issue slot. Measured per SIMD with 8 waves,
// cycles per wave64 instruction at 2.4 GHz: wide multiplies, conversions,
// compares, bit-field and three-input integer ops other than v_bitop3 4.2,
// never two at once; xor / and / shift / add / v_bitop3 2.2 when another
// wave has one to issue beside it (two that both read a scalar register
// cannot pair); float add, multiply and fma 2.2, beside either kind;
// transcendentals 8.1, beside nothing. The hardware serves the oldest wave
// first, so in a stream that alternates both kinds every waiting wave is soon
// parked at a multiply and the pairs never form: 4 multiplies + 4 xors take
// 32.5 cycles. With the waves in their multiplies (and transcendentals) at a
// raised wave priority, the others collect at their cheap instructions and
// issue them in pairs: 25.0 cycles. (The figures carry loop overhead and a
// clock a little under 2.4 GHz; the pipes' own times are 4, 2 and 8 cycles.) A
// raised wave also issues before other streams' waves on its CU. Measured beside
// a K = 64 update of 12.2 ms (13.5 not raised), raised, not raised: a 4096^3
// matrix product 2.51, 2.79 ms; an elementwise pass over a 0.27 GB buffer 2.46,
// 2.72; a softmax that takes 27 us alone 0.25, 0.26 (0.21 beside the former
// kernels of one group per lane). Beside a portable update: 3.81, 4.05; 3.79,
// 3.81; 0.40, 0.29 (0.40).
// So the loops below handle several Philox blocks per lane and work in phases:
// issue_alone() before instructions that nothing pairs with, issue_paired()
// before those that pair. Both take the values that cross the boundary as
// operands, so that what makes them stays before it and what uses them after it
// (a bare fence would order neither: this arithmetic has no side effects); the
// scheduling fences keep the rest.
#define MEZO_SETPRIO(n)                                                                                     \
    template <class T>                                                                                      \
    __device__ __forceinline__ void setprio##n(T (&v)[1])                                                   \
    {                                                                                                       \
        asm volatile("s_setprio " #n : "+v"(v[0]));                                                         \
    }                                                                                                       \
    template <class T>                                                                                      \
    __device__ __forceinline__ void setprio##n(T (&v)[2])                                                   \
    {                                                                                                       \
        asm volatile("s_setprio " #n : "+v"(v[0]), "+v"(v[1]));                                             \
    }                                                                                                       \
    template <class T>                                                                                      \
    __device__ __forceinline__ void setprio##n(T (&v)[4])                                                   \
    {                                                                                                       \
        asm volatile("s_setprio " #n : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));                     \
    }                                                                                                       \
    template <class T>                                                                                      \
    __device__ __forceinline__ void setprio##n(T (&v)[8])                                                   \
    {                                                                                                       \
        asm volatile("s_setprio " #n                                                                        \
                     : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]),  \
                       "+v"(v[7]));                                                                         \
    }
MEZO_SETPRIO(0)
MEZO_SETPRIO(1)
#undef MEZO_SETPRIO

template <bool kPhases = true, class T, int kN>
__device__ __forceinline__ void issue_alone(T (&v)[kN])
{
    if constexpr (kPhases) {
        __builtin_amdgcn_sched_barrier(0);
        setprio1(v);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <bool kPhases = true, class T, int kN>
__device__ __forceinline__ void issue_paired(T (&v)[kN])
{
    if constexpr (kPhases) {
        __builtin_amdgcn_sched_barrier(0);
        setprio0(v);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// philox_words for kBlocks blocks of a lane, in issue phases: the wide
// multiplies of every block's round, then its three-way xors. From 4 blocks
// on, one of a round's two keys is moved to a vector register (8 moves per
// record and wave), so that a xor reading it can pair with one reading the
// other from its scalar register: 237 -> 230 -> 225 cycles per block and wave
// for the whole record (2 blocks; 4 blocks; 4 blocks with such keys), 251
// before the phases. kPhases false: the same, in the compiler's order.
template <int kBlocks, bool kPhases = true>
__device__ __forceinline__ void philox_blocks(const SeedUniform& u, const BlockPre (&b)[kBlocks],
                                              uint32_t (&x)[kBlocks][4])
{
    uint32_t ka[8], kb[8];  // keys of rounds 3 .. 10
    uint32_t k0 = u.k0, k1 = u.k1;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        k0 += kWeylA;
        k1 += kWeylB;
        ka[r] = k0;
        if constexpr (kBlocks >= 4)
            asm("v_mov_b32 %0, %1" : "=v"(kb[r]) : "s"(k1));
        else
            kb[r] = k1;
    }
    // y[0 .. kBlocks): the words kMulB multiplies, y[kBlocks ..): kMulA's;
    // p: their products
    uint32_t y1[kBlocks], y[2 * kBlocks];
    uint64_t p1[kBlocks], p[2 * kBlocks];
    // end of round 1, and round 2 (its kMulA product is scalar)
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) y1[i] = b[i].hi ^ u.kx;
    issue_alone<kPhases>(y1);
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) p1[i] = uint64_t(kMulB) * y1[i];
    issue_paired<kPhases>(p1);
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
        y[i] = (u.r2_hi ^ u.k1) ^ b[i].lo;
        y[kBlocks + i] = uint32_t(p1[i] >> 32) ^ (u.y1 ^ u.k0);
        x[i][1] = uint32_t(p1[i]);
        x[i][3] = u.r2_lo;
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        issue_alone<kPhases>(y);
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) {
            p[kBlocks + i] = uint64_t(kMulA) * y[kBlocks + i];
            p[i] = uint64_t(kMulB) * y[i];
        }
        issue_paired<kPhases>(p);
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) {
            y[kBlocks + i] = xor3(uint32_t(p[i] >> 32), x[i][1], ka[r]);
            y[i] = xor3(uint32_t(p[kBlocks + i] >> 32), x[i][3], kb[r]);
            x[i][1] = uint32_t(p[i]);
            x[i][3] = uint32_t(p[kBlocks + i]);
        }
    }
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
        x[i][0] = y[kBlocks + i];
        x[i][2] = y[i];
    }
}

// ---- Box-Muller -----------------------------------------------------------
// Box & Muller (1958). u1 = ((w_a >> 8) + 1) 2^-24 in (0, 1] and
// u2 = (w_b >> 8) 2^-24 in [0, 1) are exact in fp32. v_log_f32 is log2, so
// sqrt(-2 ln u1) = sqrt(2 ln 2) sqrt(-log2 u1); v_sin_f32 / v_cos_f32 take
// revolutions, so sin(2 pi u2) needs no multiply by 2 pi.
//
// gauss4_unit returns z / sqrt(2 ln 2): the constant factor is left to the
// caller, which folds it into the record's coefficient (one multiply per
// record on the host instead of two per Gaussian pair on the device).
struct Z4 {
    float z0, z1, z2, z3;
};

// sqrt(2 ln 2): z = kZScale * (the unit-scaled value below).
constexpr float kZScale = 1.17741002251547469101f;

__device__ __forceinline__ void box_muller_pair_unit(uint32_t wa, uint32_t wb, float& zc, float& zs)
{
    constexpr float kTwoM24 = 0x1p-24f;
    // (t + 1) 2^-24 as one fma: t < 2^24, so the product, the sum and the
    // result are exact.
    const float u1 = __builtin_fmaf(float(wa >> 8), kTwoM24, kTwoM24);
    const float u2 = float(wb >> 8) * kTwoM24;
    const float r = __builtin_amdgcn_sqrtf(-__builtin_amdgcn_logf(u1));
    zc = r * __builtin_amdgcn_cosf(u2);
    zs = r * __builtin_amdgcn_sinf(u2);
}

__device__ __forceinline__ Z4 gauss4_unit(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    Z4 z;
    box_muller_pair_unit(w0, w1, z.z0, z.z1);
    box_muller_pair_unit(w2, w3, z.z2, z.z3);
    return z;
}

// The four Gaussians themselves (inspection path).
__device__ __forceinline__ Z4 gauss4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    Z4 z = gauss4_unit(w0, w1, w2, w3);
    z.z0 *= kZScale;
    z.z1 *= kZScale;
    z.z2 *= kZScale;
    z.z3 *= kZScale;
    return z;
}

// ---- portable Box-Muller ----------------------------------------------------
// The same Gaussian from binary32 +, -, *, fma, correctly rounded / and sqrt
// and exact scalings only, so that any IEEE device (a CPU included) computes
// it bit for bit (Appendix B: identical noise on every machine). -ln u1 comes
// from 2 atanh((m-1)/(m+1)) after an exact reduction of u1 to m 2^e with m in
// [sqrt(1/2), sqrt(2)); sin and cos of 2 pi u2 from the eighth of a turn that
// u2 falls in and Taylor polynomials on [0, pi/4] (coefficients 1/k! rounded
// to binary32). Division and sqrt are correctly rounded for every operand the
// transform meets, which is checked exhaustively: the GPU's z is bit-identical
// to the oracle's, which uses IEEE / and sqrt, over all 2^24 values of u1 and
// all of u2.

// n / d correctly rounded for normal n, d with a normal quotient and no
// overflow in the steps (the NF4 quantizer's 1 / m for a block maximum m in
// [2^-64, 2^64]): the reciprocal from v_rcp_f32 refined once, then two
// residual corrections of the quotient — the general sequence without its
// operand scaling and special-value fix-up, which only act outside that range.
__device__ __forceinline__ float div_rn_normal(float n, float d)
{
    float y = __builtin_amdgcn_rcpf(d);
    y = __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
    float q = n * y;
    q = __builtin_fmaf(__builtin_fmaf(-d, q, n), y, q);
    return __builtin_fmaf(__builtin_fmaf(-d, q, n), y, q);
}

// z of kPairs pairs of words (wa[p], wb[p]), step by step over all pairs, in
// issue phases. Bit for bit the definition's z, in fewer and cheaper
// instructions than its own steps:
// - u1 = m 2^e: with off = bits(fl32(sqrt 2) / 2), the exponent field of
//   bits(u1) - off is e, and taking it off bits(u1) leaves m. e stays scaled
//   by 2^23 (the constant it multiplies carries 2^-23).
// - s = (m - 1) / (m + 1) from v_rcp_f32 and one residual correction.
// - the radius from x / 4 = -ln(u1) / 2 (a scaling by a power of two changes
//   no rounding): y = 1 / sqrt(x / 4) from v_rsq_f32, g = (x / 4) y, and
//   r = fma(x / 4 - g^2, y, 2 g). For u1 = 1 (x = -0) the added 2^-100 keeps
//   y finite and r = -0, as sqrt(-0); any other x / 4 absorbs it.
// - the angle from the nearest quarter turn n: a = (2 pi u2 - n pi / 2) in
//   [-pi/4, pi/4] is the signed 22-bit field of w_b below the top two bits of
//   w_b + 2^29, which are n. The definition's angle is |a|, its octant's signs
//   and swap are those of a and n: sin a is odd and cos a even to the bit.
//   With p = +-r cos a, q = +-r sin a (the sign of n >= 2), z is (p, q) for
//   even n and (-q, p) for odd n.
// 65 vector instructions per pair with the generator's, 84 before, and more of
// them multiplies and adds, which issue in pairs. The wave stays at the raised
// priority throughout (lowered for the multiplies and adds: 3% slower).
template <int kPairs>
__device__ __forceinline__ void gauss_portable(const uint32_t (&wa)[kPairs], const uint32_t (&wb)[kPairs],
                                               float (&zc)[kPairs], float (&zs)[kPairs])
{
    constexpr float kTwoM24 = 0x1p-24f;
    constexpr uint32_t kSqrtHalfBits = 0x3F3504F3u;  // fl32(sqrt 2) / 2
    float f[kPairs], e[kPairs], s[kPairs], x[kPairs], r[kPairs];
    uint32_t em[kPairs];
#define MEZO_EACH _Pragma("unroll") for (int i = 0; i < kPairs; ++i)
    MEZO_EACH em[i] = wa[i] >> 8;
    issue_alone(em);
    MEZO_EACH f[i] = float(em[i]);
    __builtin_amdgcn_sched_barrier(0);
    MEZO_EACH
    {
        f[i] = __builtin_fmaf(f[i], kTwoM24, kTwoM24);  // u1, exact
        const uint32_t u = __float_as_uint(f[i]);
        em[i] = (u - kSqrtHalfBits) & 0xFF800000u;       // e 2^23
        f[i] = __uint_as_float(u - em[i]) - 1.0f;        // m - 1, exact
        s[i] = f[i] + 2.0f;                              // m + 1
    }
    MEZO_EACH e[i] = float(int32_t(em[i]));
    MEZO_EACH x[i] = __builtin_amdgcn_rcpf(s[i]);
    __builtin_amdgcn_sched_barrier(0);
    MEZO_EACH
    {
        const float q = f[i] * x[i];
        s[i] = __builtin_fmaf(__builtin_fmaf(-s[i], q, f[i]), x[i], q);
        const float s2 = s[i] * s[i];
        float p = __builtin_fmaf(s2, 0x1.c71c72p-4f, 0x1.24924ap-3f);  // 1/9, 1/7
        p = __builtin_fmaf(s2, p, 0x1.99999ap-3f);                     // 1/5
        p = __builtin_fmaf(s2, p, 0x1.555556p-2f);                     // 1/3
        p = __builtin_fmaf(s2, p, 1.0f);
        // -ln(u1) / 2 = -(e fl32(ln 2) + 2 s p) / 2
        x[i] = __builtin_fmaf(e[i], -0x1.62e430p-25f, -(s[i] * p));
        s[i] = x[i] + 0x1p-100f;
    }
    MEZO_EACH r[i] = __builtin_amdgcn_rsqf(s[i]);
    // the signed angle's field, in units of a 2^22th of a quarter turn
    MEZO_EACH f[i] = float(int32_t(wb[i] << 2) >> 10);
    __builtin_amdgcn_sched_barrier(0);
    MEZO_EACH
    {
        const float g = x[i] * r[i];
        r[i] = __builtin_fmaf(__builtin_fmaf(-g, g, x[i]), r[i], g + g);
        const float a = f[i] * 0x1.921fb6p-22f;  // fl32(pi/4) 2^-21
        const float a2 = a * a;
        float sn = __builtin_fmaf(a2, 0x1.71de3ap-19f, -0x1.a01a02p-13f);  // 1/9!, -1/7!
        sn = __builtin_fmaf(a2, sn, 0x1.111112p-7f);                       // 1/5!
        sn = __builtin_fmaf(a2, sn, -0x1.555556p-3f);                      // -1/3!
        sn = __builtin_fmaf(a2, sn, 1.0f);
        s[i] = a * sn;
        float cs = __builtin_fmaf(a2, -0x1.27e4fcp-22f, 0x1.a01a02p-16f);  // -1/10!, 1/8!
        cs = __builtin_fmaf(a2, cs, -0x1.6c16c2p-10f);                     // -1/6!
        cs = __builtin_fmaf(a2, cs, 0x1.555556p-5f);                       // 1/4!
        cs = __builtin_fmaf(a2, cs, -0.5f);                                // -1/2!
        f[i] = __builtin_fmaf(a2, cs, 1.0f);
        const uint32_t n = wb[i] + 0x20000000u;  // the nearest quarter turn in the top two bits
        // the sign of n >= 2 on r
        const float rs = __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(r[i]), n, 0x80000000u, 0x78));
        const float p = rs * f[i], q = rs * s[i];
        // n odd: bit 30, the top exponent bit of n read as a float (NaNs
        // included: not below 2)
        const bool odd = !(fabsf(__uint_as_float(n)) < 2.0f);
        zc[i] = odd ? -q : p;
        zs[i] = odd ? p : q;
    }
#undef MEZO_EACH
}

__device__ __forceinline__ Z4 gauss4_portable(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3)
{
    const uint32_t wa[2] = {w0, w2}, wb[2] = {w1, w3};
    float zc[2], zs[2];
    gauss_portable<2>(wa, wb, zc, zs);
    return Z4{zc[0], zs[0], zc[1], zs[1]};
}

// The noise of one record for a lane's kBlocks blocks in fast mode, in issue
// phases: acc += c z, with c the record's coefficient (which carries
// sqrt(2 ln 2)): per pair c r is formed once and scales cos and sin inside two
// fmas. kSet: acc = c z (a step's first record: no accumulator to clear
// first); the product differs from fma(c, z, +0) only in the sign of a zero
// product, which changes theta + acc only for theta = -0 (a -0 result where
// the accumulator's +0 gives +0).
template <int kBlocks, bool kSet, bool kPhases = true>
__device__ __forceinline__ void noise_fast(const SeedUniform& u, float c, const BlockPre (&b)[kBlocks],
                                           float (&acc)[kBlocks][4])
{
    constexpr float kTwoM24 = 0x1p-24f;
    uint32_t x[kBlocks][4];
    philox_blocks<kBlocks, kPhases>(u, b, x);
    uint32_t ta[2 * kBlocks];  // u1's 24 bits
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
        ta[2 * i] = x[i][0] >> 8;
        ta[2 * i + 1] = x[i][2] >> 8;
        x[i][1] >>= 8;
        x[i][3] >>= 8;
    }
    // from the conversions on the wave stays at the raised priority: its
    // multiplies and adds pair with another wave's conversions or xors
    // (against lowering it for them: 2% faster)
    issue_alone<kPhases>(ta);
    float f[kBlocks][4];
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
        f[i][0] = float(ta[2 * i]);
        f[i][1] = float(x[i][1]);
        f[i][2] = float(ta[2 * i + 1]);
        f[i][3] = float(x[i][3]);
    }
#pragma unroll
    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            f[i][2 * p] = __builtin_fmaf(f[i][2 * p], kTwoM24, kTwoM24);  // u1
            f[i][2 * p + 1] = f[i][2 * p + 1] * kTwoM24;                  // u2
        }
    if constexpr (kPhases) __builtin_amdgcn_sched_barrier(0);
    float r[kBlocks][2], cs[kBlocks][2], sn[kBlocks][2];
#pragma unroll
    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) r[i][p] = __builtin_amdgcn_logf(f[i][2 * p]);
#pragma unroll
    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            cs[i][p] = __builtin_amdgcn_cosf(f[i][2 * p + 1]);
            sn[i][p] = __builtin_amdgcn_sinf(f[i][2 * p + 1]);
        }
#pragma unroll
    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) r[i][p] = __builtin_amdgcn_sqrtf(-r[i][p]);
    if constexpr (kPhases) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kBlocks; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const float cr = c * r[i][p];
            if constexpr (kSet) {
                acc[i][2 * p] = cr * cs[i][p];
                acc[i][2 * p + 1] = cr * sn[i][p];
            } else {
                acc[i][2 * p] = __builtin_fmaf(cr, cs[i][p], acc[i][2 * p]);
                acc[i][2 * p + 1] = __builtin_fmaf(cr, sn[i][p], acc[i][2 * p + 1]);
            }
        }
}

// The noise of one record for a lane's kBlocks blocks in portable mode:
// acc = fma(c, z, acc), or acc = c z (kSet).
template <int kBlocks, bool kSet>
__device__ __forceinline__ void noise_portable(const SeedUniform& u, float c, const BlockPre (&b)[kBlocks],
                                               float (&acc)[kBlocks][4])
{
    uint32_t w[kBlocks][4];
    philox_blocks<kBlocks>(u, b, w);
    uint32_t wa[2 * kBlocks], wb[2 * kBlocks];
    float zc[2 * kBlocks], zs[2 * kBlocks];
#pragma unroll
    for (int p = 0; p < 2 * kBlocks; ++p) {
        wa[p] = w[p / 2][2 * (p & 1)];
        wb[p] = w[p / 2][2 * (p & 1) + 1];
    }
    gauss_portable<2 * kBlocks>(wa, wb, zc, zs);
#pragma unroll
    for (int p = 0; p < 2 * kBlocks; ++p) {
        float* a2 = acc[p / 2] + 2 * (p & 1);
        a2[0] = kSet ? c * zc[p] : __builtin_fmaf(c, zc[p], a2[0]);
        a2[1] = kSet ? c * zs[p] : __builtin_fmaf(c, zs[p], a2[1]);
    }
}

// Record r of a launch: from the kernel arguments (kInline) or the staged
// device buffer. Either way a wave-uniform address in memory that nothing
// writes during the launch: read through the constant address space, so that
// the words are scalar loads into SGPRs (the issue phases' fences would
// otherwise make them vector loads).
#define MEZO_CONSTANT __attribute__((address_space(4)))
template <bool kInline>
__device__ __forceinline__ SeedRec rec_at(const EngineArgs& a, uint32_t r)
{
    if constexpr (kInline) {
        return a.inl[r];
    } else {
        typedef uint32_t words8_t __attribute__((ext_vector_type(8), aligned(16)));
        const words8_t w = reinterpret_cast<const MEZO_CONSTANT words8_t*>(reinterpret_cast<uint64_t>(a.ext))[r];
        SeedRec rec;
        rec.key0 = w[0];
        rec.key1 = w[1];
        rec.step = w[2];
        rec.mb_hi = w[3];
        rec.mb_lo = w[4];
        rec.coef = __uint_as_float(w[5]);
        rec.last = w[6];
        rec.sample = w[7];
        return rec;
    }
}

// ---- storage conversions ---------------------------------------------------

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xFFFF0000u); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two fp32 -> two bf16 (round to nearest even, one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    f32x2_t v = {lo, hi};
    bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return __builtin_bit_cast(uint32_t, b);
}

__device__ __forceinline__ uint16_t to_bf16(float x)
{
    __bf16 b = static_cast<__bf16>(x);
    return __builtin_bit_cast(uint16_t, b);
}

}  // namespace mezo
