// nf4_ops.hpp — device helpers of the 4-bit storage (the 4-bit forward-only
// variant of Section 3), shared by the NF4 engine kernel and the standalone
// conversions.
//
// In the conversions a lane owns 8 consecutive elements (one dword of codes);
// the 8 lanes tid & ~7 .. tid | 7 own one 64-element block and share its
// absmax, and values become codes through the 129-bin round-to-nearest table
// of nf4.hpp. In the engine a lane owns 16 (4 lanes per block), or 8 on small
// sets; codes become values through a table of byte -> the values of its two
// codes, values become codes through the row table of nf4.hpp.
#pragma once

#include "engine.hpp"
#include "nf4.hpp"
#include "stream_io.hpp"

namespace mezo {

// Whether any lane of the wave misses elements (valid != 0xFF; only waves
// that reach a tensor's end): a uniform test, so that the masking it guards
// stays a branch that every other wave skips instead of selects that every
// wave executes.
__device__ __forceinline__ bool partial_wave(uint32_t valid)
{
    return __builtin_amdgcn_ballot_w64(valid != 0xFFu) != 0;
}

// Which of a lane's 8 elements e0 .. e0 + 7 exist (bit j for element e0 + j).
__device__ __forceinline__ uint32_t nf4_valid(uint64_t e0, uint64_t numel)
{
    if (e0 >= numel) return 0u;
    if (e0 + 8 <= numel) return 0xFFu;
    return (1u << uint32_t(numel - e0)) - 1u;
}

// A lane's code dword and its block's absmax (zeros past the end). kFull:
// the lane's 8 elements are known to exist (a tile wholly inside its tensor).
template <bool kFull = false>
__device__ __forceinline__ void nf4_load(uint64_t codes, uint64_t absmax, uint64_t e0, uint64_t numel,
                                         uint32_t& packed, float& am)
{
    packed = 0u;
    am = 0.0f;
    if (!kFull && e0 >= numel) return;
    if (kFull || e0 + 8 <= numel) {
        packed = __builtin_nontemporal_load(reinterpret_cast<const MEZO_GLOBAL uint32_t*>(codes + e0 / 2));
    } else {
        const MEZO_GLOBAL uint8_t* b = reinterpret_cast<const MEZO_GLOBAL uint8_t*>(codes + e0 / 2);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (e0 + 2 * k < numel) packed |= uint32_t(b[k]) << (8 * k);
    }
    am = reinterpret_cast<const gfloat_t*>(absmax)[e0 / kNF4Block];
}

template <bool kFull = false>
__device__ __forceinline__ void nf4_store(uint64_t codes, uint64_t absmax, uint64_t e0, uint64_t numel,
                                          uint32_t packed, float am)
{
    if (!kFull && e0 >= numel) return;
    if (kFull || e0 + 8 <= numel) {
        __builtin_nontemporal_store(packed, reinterpret_cast<MEZO_GLOBAL uint32_t*>(codes + e0 / 2));
    } else {
        MEZO_GLOBAL uint8_t* b = reinterpret_cast<MEZO_GLOBAL uint8_t*>(codes + e0 / 2);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (e0 + 2 * k < numel) b[k] = uint8_t(packed >> (8 * k));
    }
    if ((threadIdx.x & 7u) == 0u) reinterpret_cast<gfloat_t*>(absmax)[e0 / kNF4Block] = am;
}

// max over the 8 lanes of a block (lanes 8i .. 8i + 7) of a value >= 0:
// swap neighbours, then pairs within each quad, then the two quads of each
// half-row (DPP quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror).
// Non-negative floats order like their bit patterns, so the maximum is taken
// on the integers.
__device__ __forceinline__ float max8(float m)
{
    uint32_t u = __float_as_uint(m);
    u = max(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), 0xB1, 0xF, 0xF, false)));
    u = max(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), 0x4E, 0xF, 0xF, false)));
    u = max(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), 0x141, 0xF, 0xF, false)));
    return __uint_as_float(u);
}

// Nibbles of the packed codes that hold existing elements.
__device__ __forceinline__ uint32_t nf4_nibble_mask(uint32_t valid)
{
    const uint32_t k = __builtin_popcount(valid);  // valid is a run of low bits
    return k >= 8 ? 0xFFFFFFFFu : (1u << (4 * k)) - 1u;
}

// (p << 4) | c as one v_lshl_or_b32 (left to itself the compiler splits a
// chain of these into separate shifts and three-way ors).
__device__ __forceinline__ uint32_t shl4_or(uint32_t p, uint32_t c)
{
    uint32_t r;
    asm("v_lshl_or_b32 %0, %1, 4, %2" : "=v"(r) : "v"(p), "v"(c));
    return r;
}

// Block maxima whose reciprocal takes the short sequence: [2^-64, 2^64].
constexpr uint32_t kRecipLo = 0x1F800000u;  // 2^-64
constexpr uint32_t kRecipHi = 0x5F800000u;  // 2^64

// Quantize a block held by 8 lanes (w = 0 for elements that do not exist):
// a = max |w| over the block, r = 1 / a (correctly rounded; 0 for a = 0),
// code = nearest NF4 value to fl32(w * r), ties to the lower code, on the
// round-to-nearest table. When every lane's block maximum a lies in [2^-64,
// 2^64] (the usual case), r comes from the correctly rounded division
// sequence without its operand scaling and special-value fix-up (which act
// only outside that range), every |x| <= 1 + 2^-23, and the bin's table offset
// is read off t = fl32(64 x + magic) directly. Otherwise (a = 0, tiny or huge
// blocks; x may be infinite or NaN) the wave takes the general division and
// clamps the bin to the table, a NaN x (0 * inf) taking the lowest bin like
// the comparisons it fails. Returns the packed codes (0 for missing elements)
// and the absmax. Every lane of the wave must call it (the block maximum is
// exchanged across lanes).
__device__ __forceinline__ void nf4_requant_round(const NF4Bin* bins, uint32_t valid, const float (&w)[8],
                                                  uint32_t& packed, float& am)
{
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf(w[j]));
    m = max8(m);
    const bool usual = __float_as_uint(m) - kRecipLo <= kRecipHi - kRecipLo;
    const char* base = reinterpret_cast<const char*>(bins);
    // the codes enter p from the highest element down: p = (p << 4) | code
    // (the loops below run j = 7 .. 0)
    uint32_t p = 0u;
    const auto code = [&](int j, float x, uint32_t off) {
        const float2 e = *reinterpret_cast<const float2*>(base + off);  // mid, lo
        const uint32_t c = __float_as_uint(e.y) + (x > e.x ? 1u : 0u);
        p = j == 7 ? c : shl4_or(p, c);
    };
    if (__builtin_amdgcn_ballot_w64(!usual) == 0) {  // uniform
        const float r = div_rn_normal(1.0f, m);
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            const float x = w[j] * r;
            const uint32_t t = __float_as_uint(__builtin_fmaf(x, 64.0f, kNF4BinMagic));
            code(j, x, (t << 3) - (kNF4BinBase << 3));  // 8 (t - base) = 8 b
        }
    } else {
        const float r = m > 0.0f ? 1.0f / m : 0.0f;
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            const float x = w[j] * r;
            const float xs = x == x ? x : -2.0f;
            const int k = int(__float_as_uint(__builtin_fmaf(xs, 64.0f, kNF4BinMagic))) - int(kNF4BinBase);
            code(j, x, uint32_t(k < 0 ? 0 : (k > kNF4RoundBins - 1 ? kNF4RoundBins - 1 : k)) << 3);
        }
    }
    packed = partial_wave(valid) ? p & nf4_nibble_mask(valid) : p;
    am = m;
}

// ---- the engine's kernels: 8 or 16 elements per lane -------------------------
// A lane owns kDwords code dwords: 8 or 16 consecutive elements, 2 or 4 Philox
// blocks, an eighth or a quarter of an absmax block; 256 or 128 lanes per
// 2048-element tile. 16 make the issue phases longer (engine.hpp) and spread
// the work paid per lane (tile addressing, the table copy, the block maximum
// across lanes, the reciprocal) over twice the elements; 8 make twice the waves
// on small sets.

template <int kDwords>
constexpr int kNF4Lanes = int(kTileNF4) / (8 * kDwords);  // lanes per workgroup
template <int kDwords>
constexpr uint32_t kNF4All = (1u << (8 * kDwords)) - 1u;  // all of a lane's elements exist
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef MEZO_GLOBAL u32x2_t gu32x2_t;

// The LDS tables, laid out as one image of 16-byte pieces that a workgroup
// copies from constant memory: the rows of the quantizer, then byte b -> the
// values of its two codes (b & 15, b >> 4).
struct NF4Pair {
    float v_lo, v_hi;
};
struct alignas(16) NF4Lds {
    NF4Row row[kNF4Rows + 1];  // (one unused, for the alignment)
    NF4Pair pair[kNF4Pairs];
};
constexpr uint32_t kNF4LdsPieces = sizeof(NF4Lds) / 16;
static_assert(sizeof(NF4Lds) % 16 == 0 && kNF4LdsPieces <= 2 * kNF4Lanes<2> && kNF4LdsPieces <= kNF4Lanes<1>,
              "one or two pieces per lane");

constexpr NF4Lds make_nf4_lds()
{
    NF4Lds s{};
    for (int b = 0; b < kNF4Rows; ++b) s.row[b] = kNF4RowTable.row[b];
    for (int b = 0; b < kNF4Pairs; ++b) s.pair[b] = NF4Pair{kNF4Values[b & 15], kNF4Values[b >> 4]};
    return s;
}
constexpr NF4Lds kNF4LdsImage = make_nf4_lds();

// The copy in two halves, so that the noise of a step can be computed while
// the loads are under way: load() at the kernel's start, store() (a workgroup
// barrier) before the first lookup.
template <int kDwords>
struct NF4LdsCopy {
    u32x4_t v[kDwords];

    static __device__ __forceinline__ uint32_t piece(int k) { return threadIdx.x + uint32_t(k) * kNF4Lanes<kDwords>; }
    __device__ __forceinline__ void load()
    {
        const u32x4_t* src = reinterpret_cast<const u32x4_t*>(&kNF4LdsImage);
#pragma unroll
        for (int k = 0; k < kDwords; ++k) v[k] = src[piece(k) < kNF4LdsPieces ? piece(k) : kNF4LdsPieces - 1];
    }
    __device__ __forceinline__ void store(NF4Lds& s) const
    {
        u32x4_t* dst = reinterpret_cast<u32x4_t*>(&s);
#pragma unroll
        for (int k = 0; k < kDwords; ++k)
            if (piece(k) < kNF4LdsPieces) dst[piece(k)] = v[k];
        __syncthreads();
    }
};

// Byte k of packed times 8, the LDS byte offset of its entry in the pair
// table: one shift with sub-dword (SDWA) selection of the byte.
template <int k>
__device__ __forceinline__ uint32_t byte_x8(uint32_t packed)
{
    uint32_t off;
    if constexpr (k == 0)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0"
            : "=v"(off) : "v"(packed));
    else if constexpr (k == 1)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1"
            : "=v"(off) : "v"(packed));
    else if constexpr (k == 2)
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2"
            : "=v"(off) : "v"(packed));
    else
        asm("v_lshlrev_b32_sdwa %0, 3, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3"
            : "=v"(off) : "v"(packed));
    return off;
}

template <int k>
__device__ __forceinline__ float2 nf4_pair(const NF4Lds& s, uint32_t packed)
{
    return *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s.pair) + byte_x8<k>(packed));
}

// Which of a lane's elements from e0 on exist (bit j for element e0 + j).
template <int kDwords>
__device__ __forceinline__ uint32_t nf4_lane_valid(uint64_t e0, uint64_t numel)
{
    if (e0 >= numel) return 0u;
    if (e0 + 8 * kDwords <= numel) return kNF4All<kDwords>;
    return (1u << uint32_t(numel - e0)) - 1u;
}

// Missing elements' values to zero (only waves that reach a tensor's end).
template <int kDwords>
__device__ __forceinline__ void nf4_mask_lane(uint32_t valid, float (&w)[2 * kDwords][4])
{
    if (__builtin_amdgcn_ballot_w64(valid != kNF4All<kDwords>) == 0) return;
#pragma unroll
    for (int j = 0; j < 8 * kDwords; ++j)
        if (!((valid >> j) & 1u)) w[j >> 2][j & 3] = 0.0f;
}

// w = v[code] am + acc for a lane's elements: packed[h] holds elements 8h ..
// 8h + 7. Each code byte fetches the values of its two codes at once. kFused:
// one rounding of the sum; otherwise the value rounds first, as the rule
// states.
template <bool kFused, int kDwords>
__device__ __forceinline__ void nf4_lane_values(const NF4Lds& s, const uint32_t (&packed)[kDwords], float am,
                                                const float (&acc)[2 * kDwords][4], float (&w)[2 * kDwords][4])
{
    const auto sum = [&](float v, float x) {
        if constexpr (kFused)
            return __builtin_fmaf(v, am, x);
        else
            return v * am + x;
    };
#pragma unroll
    for (int h = 0; h < kDwords; ++h) {
        const float2 p[4] = {nf4_pair<0>(s, packed[h]), nf4_pair<1>(s, packed[h]), nf4_pair<2>(s, packed[h]),
                             nf4_pair<3>(s, packed[h])};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = 2 * h + (k >> 1), j = 2 * (k & 1);
            w[i][j] = sum(p[k].x, acc[i][j]);
            w[i][j + 1] = sum(p[k].y, acc[i][j + 1]);
        }
    }
}

// max over the 4 lanes of a block (one quad) of a value >= 0, on the integers
// as in max8.
__device__ __forceinline__ float max4(float m)
{
    uint32_t u = __float_as_uint(m);
    u = max(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), 0xB1, 0xF, 0xF, false)));
    u = max(u, uint32_t(__builtin_amdgcn_update_dpp(0, int(u), 0x4E, 0xF, 0xF, false)));
    return __uint_as_float(u);
}

// Quantize a lane's elements (w = 0 for those that do not exist): a = max |w|
// over the block's lanes, r = 1 / a, code = the nearest NF4 value to w r, ties
// to the lower code, by the row table.
// kExact: r correctly rounded and x = fl32(w r), as the rule states. Otherwise
// (fast mode's calls of one and two records) r is v_rcp_f32's (within 1 ulp)
// and x is the product unrounded: a code can differ from the rule's only where
// x lies within about 2^-22 of a midpoint. In the usual case (every lane's a
// in [2^-64, 2^64]) |x| <= 1 + 2^-22 and the row needs no clamp; otherwise the
// wave takes the general division and clamps the row, a NaN x (0 * inf)
// taking the lowest row like the comparisons it fails.
// The codes of 4 elements are gathered as 2^23 + ((c3 16 + c2) 16 + c1) 16 + c0,
// exact in float, whose low 16 bits are the packed codes.
// Every lane of the wave must call it.
template <bool kExact, bool kFull, int kDwords>
__device__ __forceinline__ void nf4_requant_lane(const NF4Lds& s, uint32_t valid, const float (&w)[2 * kDwords][4],
                                                 uint32_t (&packed)[kDwords], float& am)
{
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < 8 * kDwords; ++j) m = fmaxf(m, fabsf(w[j >> 2][j & 3]));
    m = kDwords == 2 ? max4(m) : max8(m);
    const bool usual = __float_as_uint(m) - kRecipLo <= kRecipHi - kRecipLo;
    const char* base = reinterpret_cast<const char*>(s.row);
    float g[2 * kDwords];  // the gathered codes of elements 4i .. 4i + 3
    if (__builtin_amdgcn_ballot_w64(!usual) == 0) {  // uniform
        const float r = kExact ? div_rn_normal(1.0f, m) : __builtin_amdgcn_rcpf(m);
        const float r512 = kExact ? 512.0f : r * 512.0f;
        const float rs = kExact ? kNF4Steep : r * kNF4Steep;
#pragma unroll
        for (int i = 0; i < 2 * kDwords; ++i)
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const float x = kExact ? w[i][j] * r : w[i][j];
                const uint32_t t = __float_as_uint(__builtin_fmaf(x, r512, kNF4RowMagic));
                const float2 e = *reinterpret_cast<const float2*>(base + (t & kNF4RowMask));  // thr, lo
                const float up = __builtin_amdgcn_fmed3f(__builtin_fmaf(x, rs, e.x), 0.0f, 1.0f);
                g[i] = __builtin_fmaf(j == 3 ? 128.0f : g[i], 16.0f, e.y) + up;
            }
    } else {
        const float r = m > 0.0f ? 1.0f / m : 0.0f;
#pragma unroll
        for (int i = 0; i < 2 * kDwords; ++i)
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const float x = w[i][j] * r;
                const float xs = x == x ? x : -2.0f;
                const int k = int(__float_as_uint(__builtin_fmaf(xs, 512.0f, kNF4RowMagic))) - int(kNF4BinBase);
                const uint32_t off = uint32_t(k < 0 ? 0 : (k > 1028 ? 1028 : k)) & kNF4RowMask;
                const float2 e = *reinterpret_cast<const float2*>(base + off);
                const float up = __builtin_fmaf(x, kNF4Steep, e.x) > 0.0f ? 1.0f : 0.0f;
                g[i] = __builtin_fmaf(j == 3 ? 128.0f : g[i], 16.0f, e.y) + up;
            }
    }
#pragma unroll
    for (int h = 0; h < kDwords; ++h)
        packed[h] = __builtin_amdgcn_perm(__float_as_uint(g[2 * h + 1]), __float_as_uint(g[2 * h]), 0x05040100u);
    if (!kFull && __builtin_amdgcn_ballot_w64(valid != kNF4All<kDwords>) != 0) {
        // missing elements get zero nibbles
#pragma unroll
        for (int h = 0; h < kDwords; ++h) packed[h] &= nf4_nibble_mask((valid >> (8 * h)) & 0xFFu);
    }
    am = m;
}

}  // namespace mezo
