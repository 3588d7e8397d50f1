// engine_nf4.hip — the engine kernels on 4-bit NF4 storage (gfx950): the
// same records as on fp32/bf16 storage, with the block dequantized once
// before the first record and quantized again at every step end (Section 3:
// the weights are dequantized before the noise is added and quantized again
// afterwards). Three kernels by the length of the record list: one loop over
// any number of records (engine_nf4_kernel), two records
// (engine_nf4_short_kernel) and one record (engine_nf4_sweep_kernel), each with
// 16 elements per lane and 128 lanes per 2048-element tile, or 8 and 256 on
// small sets (kDwords code dwords per lane). All three are bound by vector
// issue (the record loop as on dense storage; around it the
// quantizer, nf4_ops.hpp).
#include "engine.hpp"
#include "engine_launch.hpp"
#include "launch.hpp"
#include "nf4_ops.hpp"

namespace mezo {

// The tile a workgroup handles, and a lane's share of it: its codes and the
// absmax of their block. NF4 tensors are never shards (first = 0), so element
// e of the tile is element e of the tensor.
template <int kDwords>
struct NF4Tile {
    TensorDesc d;
    uint64_t src_codes, src_absmax;
    uint32_t local;
    uint32_t valid;  // which of the lane's elements exist
    uint32_t packed[kDwords];
    float am;

    __device__ __forceinline__ explicit NF4Tile(const EngineArgs& a)
    {
        const uint32_t tile = blockIdx.x;  // the grid is exactly the tiles of this table (< 2^31)
        const uint32_t ti = a.tile_tensor[tile];
        d = a.tensors[ti];
        // out of place: read tensor ti of the source set (same layout), write d
        src_codes = a.src_tensors ? a.src_tensors[ti].data : d.data;
        src_absmax = a.src_tensors ? a.src_tensors[ti].aux : d.aux;
        local = tile - uint32_t(d.tile_begin);
    }

    // Uniform: the tile lies wholly inside its tensor (every tile but a
    // tensor's last). Such a tile takes paths compiled without bounds or
    // masks, addressed as the tile's scalar base plus a 32-bit lane offset.
    __device__ __forceinline__ bool whole() const { return local < uint32_t(d.numel / kTileNF4); }

    // The tensor's Philox block of the lane's first element.
    __device__ __forceinline__ uint32_t block() const
    {
        return local * uint32_t(kTileNF4 / 4) + 2u * kDwords * threadIdx.x;
    }

    template <bool kFull>
    __device__ __forceinline__ void load()
    {
        if constexpr (kFull) {
            valid = kNF4All<kDwords>;
            const gfloat_t* ain = reinterpret_cast<const gfloat_t*>(src_absmax) + uint64_t(local) * kBlocks;
            if constexpr (kDwords == 2) {
                const gu32x2_t* cin = reinterpret_cast<const gu32x2_t*>(src_codes) + uint64_t(local) * kLanes;
                const u32x2_t v = __builtin_nontemporal_load(cin + threadIdx.x);
                packed[0] = v.x;
                packed[1] = v.y;
            } else {
                const MEZO_GLOBAL uint32_t* cin =
                    reinterpret_cast<const MEZO_GLOBAL uint32_t*>(src_codes) + uint64_t(local) * kLanes;
                packed[0] = __builtin_nontemporal_load(cin + threadIdx.x);
            }
            am = ain[threadIdx.x / kBlockLanes];
        } else {
            const uint64_t e0 = uint64_t(local) * kTileNF4 + threadIdx.x * (8u * kDwords);
            valid = nf4_lane_valid<kDwords>(e0, d.numel);
#pragma unroll
            for (int h = 0; h < kDwords; ++h) packed[h] = 0u;
            am = 0.0f;
            if (e0 < d.numel) {
                const MEZO_GLOBAL uint8_t* cb = reinterpret_cast<const MEZO_GLOBAL uint8_t*>(src_codes + e0 / 2);
#pragma unroll
                for (uint32_t k = 0; k < 4 * kDwords; ++k)
                    if (e0 + 2 * k < d.numel) packed[k >> 2] |= uint32_t(cb[k]) << (8 * (k & 3));
                am = reinterpret_cast<const gfloat_t*>(src_absmax)[e0 / kNF4Block];
            }
        }
    }

    // The lanes of a block all store its absmax (the same value to the same
    // address).
    template <bool kFull>
    __device__ __forceinline__ void store() const
    {
        if constexpr (kFull) {
            gfloat_t* aout = reinterpret_cast<gfloat_t*>(d.aux) + uint64_t(local) * kBlocks;
            if constexpr (kDwords == 2) {
                gu32x2_t* cout = reinterpret_cast<gu32x2_t*>(d.data) + uint64_t(local) * kLanes;
                const u32x2_t o = {packed[0], packed[1]};
                __builtin_nontemporal_store(o, cout + threadIdx.x);
            } else {
                MEZO_GLOBAL uint32_t* cout =
                    reinterpret_cast<MEZO_GLOBAL uint32_t*>(d.data) + uint64_t(local) * kLanes;
                __builtin_nontemporal_store(packed[0], cout + threadIdx.x);
            }
            aout[threadIdx.x / kBlockLanes] = am;
        } else {
            const uint64_t e0 = uint64_t(local) * kTileNF4 + threadIdx.x * (8u * kDwords);
            if (e0 < d.numel) {
                MEZO_GLOBAL uint8_t* ob = reinterpret_cast<MEZO_GLOBAL uint8_t*>(d.data + e0 / 2);
#pragma unroll
                for (uint32_t k = 0; k < 4 * kDwords; ++k)
                    if (e0 + 2 * k < d.numel) ob[k] = uint8_t(packed[k >> 2] >> (8 * (k & 3)));
                reinterpret_cast<gfloat_t*>(d.aux)[e0 / kNF4Block] = am;
            }
        }
    }

    static constexpr uint32_t kLanes = kNF4Lanes<kDwords>, kBlocks = kTileNF4 / kNF4Block;  // per tile
    static constexpr uint32_t kBlockLanes = kLanes / kBlocks;
};

template <int kN>
__device__ __forceinline__ void block_pres(uint32_t blk, BlockPre (&pre)[kN])
{
#pragma unroll
    for (int h = 0; h < kN; ++h) pre[h] = block_pre(blk + h);
}

// The noise of one record for a lane's kN blocks: acc = c z (kSet, a step's
// first record, which saves zeroing the accumulators; the product can differ
// from fma(c, z, +0) only in the sign of a zero, which no code depends on, +0
// and -0 sharing the zero code's row) or acc += c z. The portable transform
// takes two blocks at a time. kPhases: fast mode in issue phases (engine.hpp).
template <bool kPortable, bool kSet, bool kPhases, int kN>
__device__ __forceinline__ void noise(const SeedRec& rec, uint32_t tensor_id, const BlockPre (&pre)[kN],
                                      float (&acc)[kN][4])
{
    const SeedUniform u = seed_uniform(rec, tensor_id);
    const float c = rec.coef;
    if constexpr (kPortable) {
#pragma unroll
        for (int h = 0; h < kN; h += 2) {
            const BlockPre p2[2] = {pre[h], pre[h + 1]};
            float a2[2][4];
#pragma unroll
            for (int j = 0; j < 8; ++j) a2[j >> 2][j & 3] = acc[h + (j >> 2)][j & 3];
            noise_portable<2, kSet>(u, c, p2, a2);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[h + (j >> 2)][j & 3] = a2[j >> 2][j & 3];
        }
    } else {
        noise_fast<kN, kSet, kPhases>(u, c, pre, acc);
    }
}

// The end of a step on a lane's elements: dequantize, add the step's noise,
// quantize. The values are formed here and not before the noise, which keeps
// their registers free for the record loop and lets the codes' load run beside
// it. kFused (fast mode's steps of one record): one rounding of the value plus
// the noise; otherwise the two that the rule states. kExact: nf4_requant_lane.
template <bool kFused, bool kExact, bool kFull, int kDwords>
__device__ __forceinline__ void step_end(const NF4Lds& lds, NF4Tile<kDwords>& t, const float (&acc)[2 * kDwords][4])
{
    float w[2 * kDwords][4];
    nf4_lane_values<kFused>(lds, t.packed, t.am, acc, w);
    if constexpr (!kFull) nf4_mask_lane<kDwords>(t.valid, w);
    nf4_requant_lane<kExact, kFull>(lds, t.valid, w, t.packed, t.am);
}

// A tile through a call of one record (a perturbation).
template <bool kPortable, bool kFull, int kDwords>
__device__ __forceinline__ void sweep_tile(const EngineArgs& a, NF4Tile<kDwords>& t, NF4Lds& lds)
{
    NF4LdsCopy<kDwords> copy;
    t.template load<kFull>();
    copy.load();
    BlockPre pre[2 * kDwords];
    block_pres(t.block(), pre);
    float acc[2 * kDwords][4];
    noise<kPortable, true, true>(a.inl[0], t.d.tensor_id, pre, acc);
    copy.store(lds);
    step_end<!kPortable, kPortable, kFull>(lds, t, acc);
    t.template store<kFull>();
}

// A call of one record (a perturbation).
template <bool kPortable, int kDwords>
__global__ __launch_bounds__(kNF4Lanes<kDwords>) void engine_nf4_sweep_kernel(EngineArgs a)
{
    __shared__ NF4Lds lds;
    NF4Tile<kDwords> t(a);
    if (t.whole())
        sweep_tile<kPortable, true>(a, t, lds);
    else
        sweep_tile<kPortable, false>(a, t, lds);
}

// A tile through a call of two records: a restore fused with the next
// perturbation, or an update of two records in one step. With no records (out
// of place with nothing to apply) the tile is copied.
template <bool kPortable, bool kFull, int kDwords, bool kPhases>
__device__ __forceinline__ void short_tile(const EngineArgs& a, NF4Tile<kDwords>& t, NF4Lds& lds)
{
    t.template load<kFull>();
    if (a.n_rec) {
        NF4LdsCopy<kDwords> copy;
        copy.load();
        BlockPre pre[2 * kDwords];
        block_pres(t.block(), pre);
        float acc[2 * kDwords][4];
        noise<kPortable, true, kPhases>(a.inl[0], t.d.tensor_id, pre, acc);
        copy.store(lds);
        if (a.inl[0].last) {
            step_end<!kPortable, kPortable, kFull>(lds, t, acc);
            noise<kPortable, true, kPhases>(a.inl[1], t.d.tensor_id, pre, acc);
            step_end<!kPortable, kPortable, kFull>(lds, t, acc);
        } else {  // two records in one step: their sum, one rounding
            noise<kPortable, false, kPhases>(a.inl[1], t.d.tensor_id, pre, acc);
            step_end<false, kPortable, kFull>(lds, t, acc);
        }
    }
    t.template store<kFull>();
}

// A call of two records (inline), or of none.
template <bool kPortable, int kDwords, bool kPhases>
__global__ __launch_bounds__(kNF4Lanes<kDwords>) void engine_nf4_short_kernel(EngineArgs a)
{
    __shared__ NF4Lds lds;
    NF4Tile<kDwords> t(a);
    if (t.whole())
        short_tile<kPortable, true, kDwords, kPhases>(a, t, lds);
    else
        short_tile<kPortable, false, kDwords, kPhases>(a, t, lds);
}

// Record lists of more than two records: one loop over the records. The
// quantizer follows the rule exactly in both modes (its cost is spread over
// the records).
template <bool kInline, bool kPortable, int kDwords, bool kPhases>
__global__ __launch_bounds__(kNF4Lanes<kDwords>) void engine_nf4_kernel(EngineArgs a)
{
    __shared__ NF4Lds lds;
    NF4Tile<kDwords> t(a);
    NF4LdsCopy<kDwords> copy;
    if (t.whole())
        t.template load<true>();
    else
        t.template load<false>();
    copy.load();
    copy.store(lds);
    BlockPre pre[2 * kDwords];
    block_pres(t.block(), pre);
    float acc[2 * kDwords][4];
    const auto clear = [&]() {
#pragma unroll
        for (int j = 0; j < 8 * kDwords; ++j) acc[j >> 2][j & 3] = 0.0f;
    };
    clear();
    // every record list ends a step with its last record
    for (uint32_t r = 0; r < a.n_rec; ++r) {
        const SeedRec rec = rec_at<kInline>(a, r);
        noise<kPortable, false, kPhases>(rec, t.d.tensor_id, pre, acc);
        if (rec.last) {
            step_end<false, true, false>(lds, t, acc);
            clear();
        }
    }
    if (t.whole())
        t.template store<true>();
    else
        t.template store<false>();
}

namespace {
template <bool kPortable, int kDwords, bool kPhases = true>
hipError_t launch_variant(const EngineArgs& args, uint32_t tiles, hipStream_t stream)
{
    constexpr int kLanes = kNF4Lanes<kDwords>;
    // (two dwords in portable mode are for short lists: launch_dwords)
    if constexpr (!(kPortable && kDwords == 2))
        if (args.n_rec > kInlineRecs)
            return launch1(engine_nf4_kernel<false, kPortable, kDwords, kPhases>, tiles, kLanes, stream, args, args.done);
    if (args.n_rec == 1) return launch1(engine_nf4_sweep_kernel<kPortable, kDwords>, tiles, kLanes, stream, args, args.done);
    if (args.n_rec <= 2)
        return launch1(engine_nf4_short_kernel<kPortable, kDwords, kPhases>, tiles, kLanes, stream, args, args.done);
    return launch1(engine_nf4_kernel<true, kPortable, kDwords, kPhases>, tiles, kLanes, stream, args, args.done);
}

// Two code dwords per lane from kTilesNF4For2 tiles on, as on dense storage
// (engine_dense.hip): fewer tiles leave too few waves. K = 8 updates with 1, 2
// dwords, against one dword and no issue phases: 4M elements 23.2 -> 21.5, 23.4
// us; 16M 67.5 -> 61.9, 62.5; 32M 125.9 -> 115.0, 113.9; 64M 242.9 -> 221.0,
// 217.0; three perturbations 16M 50.5 -> 44.7, 44.4; 64M 140.1 -> 127.7, 123.8.
// The portable transform takes two blocks at a time either way: one dword
// (16M: 122.5 -> 85.6, 89.2; 64M 453.5 -> 315.4, 318.5; K = 64 on 128M 6741 ->
// 4744, 4867), but for short lists on large sets (one record on 1.3B: 1440 ->
// 1097, 1047; three on 128M 363.5 -> 266.1, 262.9).
// Fast lists and two-record calls on up to 256 tiles go without issue phases
// (one wave per SIMD: engine_dense.hip). 250 thousand elements in a graph, before
// the phases, with, without: K = 32 16.6, 16.9, 15.9 us; K = 8 6.14, 6.22, 6.04;
// K = 2 3.46, 3.60, 3.50. 1M elements, two waves per SIMD: K = 32 21.2, 19.4,
// 22.0.
constexpr uint32_t kTilesNF4Phased = 257;
constexpr uint32_t kTilesNF4For2 = 12u << 10, kTilesNF4PortableFor2 = 48u << 10, kRecsNF4PortableFor2 = 4;
static_assert(kRecsNF4PortableFor2 <= kInlineRecs, "launch_variant has no staged kernel for these");

hipError_t launch_dwords(const EngineArgs& args, bool portable, uint32_t tiles, hipStream_t stream)
{
    if (portable && tiles >= kTilesNF4PortableFor2 && args.n_rec <= kRecsNF4PortableFor2)
        return launch_variant<true, 2>(args, tiles, stream);
    if (portable) return launch_variant<true, 1>(args, tiles, stream);
    if (tiles < kTilesNF4Phased) return launch_variant<false, 1, false>(args, tiles, stream);
    if (tiles < kTilesNF4For2) return launch_variant<false, 1>(args, tiles, stream);
    return launch_variant<false, 2>(args, tiles, stream);
}
}  // namespace

hipError_t launch_engine_nf4(const EngineArgs& args, bool portable, hipStream_t stream)
{
    if (args.total_tiles == 0) return hipSuccess;
    if (args.total_tiles > uint64_t(0x7FFFFFFF)) return hipErrorInvalidValue;
    const uint32_t tiles = uint32_t(args.total_tiles);
    return launch_dwords(args, portable, tiles, stream);
}

}  // namespace mezo
