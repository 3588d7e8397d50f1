// engine_dense.hip — the engine kernels on fp32 and bf16 storage (gfx950).
//
// A launch applies any sequence of seeded perturbations to a whole parameter
// set in one pass: PerturbParameters (one record), the fused apply loop of one
// iteration (K records, the last flagged) and the late-joiner replay (T steps
// of records, each step's last flagged). Every element is read once and
// written once; its noise is regenerated in registers for every record.
//
// In place, or out of place from a source set of the same layout (theta =
// backup + sum c z: the restore of Algorithm 1 fused into the update).
//
// Launch shape: one launch per storage type, one workgroup per 4 KiB tile
// (1024 fp32 or 2048 bf16 elements); the workgroup finds its tensor with two
// scalar loads (tile -> tensor index -> descriptor). theta streams through
// with non-temporal 16-byte loads and stores (it is touched once per call, so
// it should not displace anything in the caches). Per lane, the
// seed-independent round-1 Philox product of each owned block is computed once
// and reused by every record; seed words, tensor id and coefficient are
// wave-uniform and live in SGPRs (scalar loads from the kernel arguments or
// from the staged record buffer).
//
// Two kernels. Calls whose steps each hold one record (engine_sweep_kernel, at
// most two records) are bound by memory or near it: 256 lanes per tile, one
// 16-byte group per lane. Longer record lists (engine_kernel) are bound by
// vector issue: on large sets 4 Philox blocks per lane (fp32: 64 lanes per
// tile, bf16: 128), so that the instructions of 4 blocks form issue phases
// (engine.hpp) and the key schedule's moves are spread over them; fewer blocks
// on smaller sets, and no phases on the smallest (launch_list): 2.54 -> 2.83e12
// param-seeds/s (K = 64 update of the 6.7B bf16 set, 167.6 -> 150.4 ms; K = 16
// of the 1.3B set 8.29 -> 7.52 ms; a 6 x 8 replay of the 125M fp32 set 2.37 ->
// 2.16 ms) against one group per lane and no phases.
#include "engine.hpp"
#include "engine_launch.hpp"
#include "launch.hpp"
#include "stream_io.hpp"
#include "tiles.hpp"

namespace mezo {

// A tile as kLanes lanes hold it: each lane owns kGroups 16-byte groups,
// strided by kLanes groups, of 4 fp32 or 8 bf16 elements (one or two Philox
// blocks) each, kept as four words.
template <uint32_t kDtype, int kLanes>
struct LaneTile {
    static constexpr int kGroups = kThreads / kLanes;  // a tile is kThreads groups
    static constexpr uint64_t kPer = Layout<kDtype>::kPerGroup;
    static constexpr int kBlocksPerGroup = int(kPer / 4);
    static constexpr int kBlocks = kGroups * kBlocksPerGroup;

    uint32_t th[kGroups][4];

    static __device__ __forceinline__ uint64_t group(uint64_t tile, int g)
    {
        return tile * kThreads + uint32_t(g * kLanes) + threadIdx.x;
    }

    // full: the tile lies wholly inside its tensor (every tile but a tensor's
    // last): no per-lane bounds, and each access is the tile's (uniform) base
    // address plus a 32-bit lane offset. Otherwise a group that runs past the
    // tensor's end is read element by element, missing ones as zero.
    __device__ __forceinline__ void load(uint64_t src, uint64_t numel, uint64_t tile, bool full)
    {
        if (full) {
            const gu32x4_t* base = reinterpret_cast<const gu32x4_t*>(src) + tile * kThreads;
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const u32x4_t v = __builtin_nontemporal_load(base + (uint32_t(g * kLanes) + threadIdx.x));
                th[g][0] = v.x;
                th[g][1] = v.y;
                th[g][2] = v.z;
                th[g][3] = v.w;
            }
            return;
        }
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const uint64_t grp = group(tile, g);
            if ((grp + 1) * kPer <= numel) {
                const uint4 v = load_stream(src + grp * 16);
                th[g][0] = v.x;
                th[g][1] = v.y;
                th[g][2] = v.z;
                th[g][3] = v.w;
            } else {
                const uint64_t e0 = grp * kPer;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (kDtype == kF32) {
                        const MEZO_GLOBAL uint32_t* in = reinterpret_cast<const MEZO_GLOBAL uint32_t*>(src);
                        th[g][j] = (e0 + j < numel) ? in[e0 + j] : 0u;
                    } else {
                        const gu16_t* in = reinterpret_cast<const gu16_t*>(src);
                        const uint32_t lo = (e0 + 2 * j < numel) ? uint32_t(in[e0 + 2 * j]) : 0u;
                        const uint32_t hi = (e0 + 2 * j + 1 < numel) ? uint32_t(in[e0 + 2 * j + 1]) : 0u;
                        th[g][j] = lo | (hi << 16);
                    }
                }
            }
        }
    }

    __device__ __forceinline__ void store(uint64_t dst, uint64_t numel, uint64_t tile, bool full) const
    {
        if (full) {
            // buffer stores over the tile's 4 KiB with the cache policy "sc1
            // nt" (paired against "nt" alone: the 125M fp32 sweep 1.9% faster,
            // the bf16 sweeps and the record loops unchanged)
            const __amdgpu_buffer_rsrc_t r = tile_rsrc(dst + tile * (kThreads * 16), kThreads * 16);
#pragma unroll
            for (int g = 0; g < kGroups; ++g)
                store_tile_b128(r, (uint32_t(g * kLanes) + threadIdx.x) * 16u,
                                make_uint4(th[g][0], th[g][1], th[g][2], th[g][3]));
            return;
        }
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const uint64_t grp = group(tile, g);
            if ((grp + 1) * kPer <= numel) {
                store_stream(dst + grp * 16, make_uint4(th[g][0], th[g][1], th[g][2], th[g][3]));
            } else {
                const uint64_t e0 = grp * kPer;
#pragma unroll
                for (int j = 0; j < int(kPer); ++j) {
                    if (e0 + j >= numel) continue;
                    if constexpr (kDtype == kF32)
                        reinterpret_cast<MEZO_GLOBAL uint32_t*>(dst)[e0 + j] = th[g][j];
                    else
                        reinterpret_cast<gu16_t*>(dst)[e0 + j] = uint16_t(th[g][j >> 1] >> (16 * (j & 1)));
                }
            }
        }
    }

    // The seed-independent products of the lane's blocks, numbered within the
    // logical tensor (first: the shard's first element).
    __device__ __forceinline__ void blocks(uint64_t first, uint64_t tile, BlockPre (&pre)[kBlocks]) const
    {
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const uint64_t blk = (first >> 2) + kBlocksPerGroup * group(tile, g);
#pragma unroll
            for (int h = 0; h < kBlocksPerGroup; ++h) pre[g * kBlocksPerGroup + h] = block_pre(uint32_t(blk + h));
        }
    }

    // The end of a step: theta = round(theta + acc). bf16 theta stays packed:
    // after every step it is a bf16 value again, so the packed pairs lose
    // nothing.
    __device__ __forceinline__ void step_end(const float (&acc)[kBlocks][4])
    {
#pragma unroll
        for (int g = 0; g < kGroups; ++g)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (kDtype == kF32) {
                    th[g][j] = __float_as_uint(__uint_as_float(th[g][j]) + acc[g][j]);
                } else {
                    const int b = 2 * g + (j >> 1);
                    th[g][j] = pack_bf16(bf16_lo(th[g][j]) + acc[b][2 * (j & 1)],
                                         bf16_hi(th[g][j]) + acc[b][2 * (j & 1) + 1]);
                }
            }
    }
};

// The tile a workgroup handles: its tensor, where it reads and writes, and
// whether it lies wholly inside the tensor (uniform).
struct TileJob {
    TensorDesc d;
    uint64_t src, local;
    bool full;
};

template <uint32_t kDtype>
__device__ __forceinline__ TileJob tile_job(const EngineArgs& a)
{
    TileJob t;
    const uint64_t tile = blockIdx.x;  // the grid is exactly the tiles of this table
    const uint32_t ti = a.tile_tensor[tile];
    t.d = a.tensors[ti];
    // out of place: read tensor ti of the source set (same layout), write d
    t.src = a.src_tensors ? a.src_tensors[ti].data : t.d.data;
    t.local = tile - t.d.tile_begin;
    constexpr uint64_t kTileElems = kThreads * Layout<kDtype>::kPerGroup;
    t.full = (t.local + 1) * kTileElems <= t.d.numel;
    return t;
}

// Calls whose steps each hold one record (a perturbation, or a restore and
// the next perturbation in one pass), fast mode: each record's noise assigns
// the accumulators instead of being added to cleared ones. No records: a copy
// (out of place with nothing to apply). A kernel for each count: the record's
// words are then read beside the tile's descriptor and not after a branch on
// the count, which costs every wave's start as much again (launches in a graph,
// count read, compiled: bf16 60 thousand elements 2.87, 2.58 us, 1M 3.57, 3.21,
// 16M 12.25, 11.82; two records 1M 3.87, 3.54; fp32 60 thousand 2.53, 2.35).
template <uint32_t kDtype, int kRecs>
__global__ __launch_bounds__(kThreads) void engine_sweep_kernel(EngineArgs a)
{
    using Tile = LaneTile<kDtype, kThreads>;
    const TileJob t = tile_job<kDtype>(a);
    Tile tile;
    tile.load(t.src, t.d.numel, t.local, t.full);
    if constexpr (kRecs > 0) {
        BlockPre pre[Tile::kBlocks];
        tile.blocks(t.d.first, t.local, pre);
        const auto step = [&](const SeedRec& rec) {
            const SeedUniform u = seed_uniform(rec, t.d.tensor_id);
            float acc[Tile::kBlocks][4];
            noise_fast<Tile::kBlocks, true>(u, rec.coef, pre, acc);
            tile.step_end(acc);
        };
        step(a.inl[0]);
        if constexpr (kRecs == 2) step(a.inl[1]);
    }
    tile.store(t.d.data, t.d.numel, t.local, t.full);
}

// Any record list of one record or more, kLanes lanes per tile. Without issue
// phases (launch_list) each record's words are read while the one before is
// worked on; with them other waves hide the read, and reading early costs (12M
// bf16 elements, portable, K = 64: 448 -> 475 us).
template <bool kInline, uint32_t kDtype, bool kPortable, int kLanes, bool kPhases>
__global__ __launch_bounds__(kLanes) void engine_kernel(EngineArgs a)
{
    using Tile = LaneTile<kDtype, kLanes>;
    constexpr int kBlocks = Tile::kBlocks;
    const TileJob t = tile_job<kDtype>(a);
    Tile tile;
    tile.load(t.src, t.d.numel, t.local, t.full);
    BlockPre pre[kBlocks];
    tile.blocks(t.d.first, t.local, pre);
    float acc[kBlocks][4];
    const auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < kBlocks; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = 0.0f;
    };
    const auto accumulate = [&](const SeedRec& rec) {
        const SeedUniform u = seed_uniform(rec, t.d.tensor_id);
        if constexpr (kPortable)
            noise_portable<kBlocks, false>(u, rec.coef, pre, acc);
        else
            noise_fast<kBlocks, false, kPhases>(u, rec.coef, pre, acc);
    };
    clear();
    // the last record ends the call's last step: peeled off the loop, it
    // needs no reset of acc afterwards
    if constexpr (kPhases) {
        for (uint32_t r = 0; r + 1 < a.n_rec; ++r) {
            accumulate(rec_at<kInline>(a, r));
            if (rec_at<kInline>(a, r).last) {
                tile.step_end(acc);
                clear();
            }
        }
        if (a.n_rec > 0) {
            accumulate(rec_at<kInline>(a, a.n_rec - 1));
            tile.step_end(acc);
        }
    } else {
        SeedRec rec = rec_at<kInline>(a, 0);
        for (uint32_t r = 1; r < a.n_rec; ++r) {
            const SeedRec next = rec_at<kInline>(a, r);
            accumulate(rec);
            if (rec.last) {
                tile.step_end(acc);
                clear();
            }
            rec = next;
        }
        accumulate(rec);
        tile.step_end(acc);
    }
    tile.store(t.d.data, t.d.numel, t.local, t.full);
}

namespace {
template <uint32_t kDtype>
hipError_t launch_sweep(const EngineArgs& args, uint32_t tiles, hipStream_t stream)
{
    if (args.n_rec == 0) return launch1(engine_sweep_kernel<kDtype, 0>, tiles, kThreads, stream, args, args.done);
    if (args.n_rec == 1) return launch1(engine_sweep_kernel<kDtype, 1>, tiles, kThreads, stream, args, args.done);
    return launch1(engine_sweep_kernel<kDtype, 2>, tiles, kThreads, stream, args, args.done);
}

template <bool kInline, uint32_t kDtype, bool kPortable, int kBlocks, bool kPhases = true>
hipError_t launch_blocks(const EngineArgs& args, uint32_t tiles, hipStream_t stream)
{
    constexpr int kLanes = int(kThreads * Layout<kDtype>::kPerGroup / 4) / kBlocks;
    return launch1(engine_kernel<kInline, kDtype, kPortable, kLanes, kPhases>, tiles, kLanes, stream, args,
                   args.done);
}

// How many Philox blocks a lane of a list launch takes. More blocks make
// longer issue phases, fewer make more waves, which fill the chip's 1024 SIMDs
// evenly and hide the loads; so it goes by the tiles there are. Update times
// against one group per lane without phases (K = 8; fp32 with 1, 2, 4 blocks):
// 16M elements 62.6 -> 59.3, 59.3, 63.7 us; 32M 117.9 -> 112.9, 112.1, 118.5;
// 64M 230.9 -> 220.4, 217.7, 224.6; 128M 458.6 -> 445.5, 431.7, 425.7 (K = 64
// on 16M: 452 -> 426, 432, 453). bf16 with 2, 4: 8M 35.1 -> 33.0, 34.1; 16M
// 62.1 -> 58.4, 58.5; 32M 116.1 -> 109.1, 107.6; 64M 224.1 -> 210.8, 205.3.
// Portable, fp32 with 1, 2: 16M 113.2 -> 89.2, 96.7; 128M 864 -> 680, 670;
// bf16 gains from 2 at every size (4: 4-7% slower). One portable record on fp32
// is bound by memory too and keeps 1 at every size: one group per lane without
// phases, 1, 2: 130M 169.9, 165.9, 169.4 us; 300M 383.5, 378.3, 390.0; 520M
// 662, 654, 683 (two records: 520M 1039, 878, 839).
// Fast mode on up to 256 tiles, a workgroup per CU and a wave per SIMD, goes
// without phases: nothing pairs there, and the phases only keep the wave's own
// instructions apart. As above (no phases, one group per lane), with phases,
// without them and with the next record read early: 300 thousand bf16 elements
// K = 16 12.8, 13.6, 12.4 us, K = 32 20.5, 22.0, 19.9, K = 64 47.0, 47.6, 45.3;
// 255 thousand fp32 K = 32 18.1, 18.3, 16.1. From 257 tiles on two waves share
// a SIMD: 600 thousand bf16 K = 32 23.9, 22.4, 23.3.
constexpr uint32_t kTilesPhased = 257;
constexpr uint32_t kTilesF32For2 = 24u << 10, kTilesF32For4 = 96u << 10, kTilesBF16For4 = 8u << 10;
constexpr uint32_t kTilesF32PortableFor2 = 64u << 10;

template <bool kInline, bool kPortable>
hipError_t launch_list(const EngineArgs& args, uint32_t dtype, uint32_t tiles, hipStream_t stream)
{
    if (dtype == kF32) {
        if constexpr (kPortable) {
            if (tiles < kTilesF32PortableFor2 || args.n_rec == 1)
                return launch_blocks<kInline, kF32, true, 1>(args, tiles, stream);
            return launch_blocks<kInline, kF32, true, 2>(args, tiles, stream);
        } else {
            if (tiles < kTilesPhased) return launch_blocks<kInline, kF32, false, 1, false>(args, tiles, stream);
            if (tiles < kTilesF32For2) return launch_blocks<kInline, kF32, false, 1>(args, tiles, stream);
            if (tiles < kTilesF32For4) return launch_blocks<kInline, kF32, false, 2>(args, tiles, stream);
            return launch_blocks<kInline, kF32, false, 4>(args, tiles, stream);
        }
    }
    if constexpr (!kPortable) {
        if (tiles < kTilesPhased) return launch_blocks<kInline, kBF16, false, 2, false>(args, tiles, stream);
        if (tiles >= kTilesBF16For4) return launch_blocks<kInline, kBF16, false, 4>(args, tiles, stream);
    }
    return launch_blocks<kInline, kBF16, kPortable, 2>(args, tiles, stream);
}
}  // namespace

hipError_t launch_engine_dense(const EngineArgs& args, uint32_t dtype, bool portable, hipStream_t stream)
{
    if (args.total_tiles == 0) return hipSuccess;
    if (args.total_tiles > uint64_t(0x7FFFFFFF) || (dtype != kF32 && dtype != kBF16)) return hipErrorInvalidValue;
    const uint32_t tiles = uint32_t(args.total_tiles);
    // at most two records, each a step of its own (or none): the sweep kernel
    const bool sweep = args.n_rec <= 1 || (args.n_rec == 2 && args.inl[0].last);
    if (sweep && (!portable || args.n_rec == 0))
        return dtype == kF32 ? launch_sweep<kF32>(args, tiles, stream) : launch_sweep<kBF16>(args, tiles, stream);
    if (args.n_rec <= kInlineRecs)
        return portable ? launch_list<true, true>(args, dtype, tiles, stream)
                        : launch_list<true, false>(args, dtype, tiles, stream);
    return portable ? launch_list<false, true>(args, dtype, tiles, stream)
                    : launch_list<false, false>(args, dtype, tiles, stream);
}

}  // namespace mezo
