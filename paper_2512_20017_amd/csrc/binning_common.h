// Device code shared by the binning kernels of the 3D-Gaussian and the 2D-surfel variants: the block of 256 consecutive
// points that compacts its visible points, writes their raster records and puts their (tile, point) pairs into the tiles'
// lists.
#pragma once
#include "pbdr_internal.h"
#include "pair_reduce.h"
#include "wave_ops.h"

namespace pbdr {

// Pair counts are summed with saturation at 2^31 - 1: a degenerate state (many screen-filling splats) cannot wrap the
// 32-bit prefix sums; everything at or beyond the capacity (< 2^30) is dropped and reported as overflow.
constexpr uint32_t kPairSat = 0x7fffffffu;
__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b)      // a, b <= kPairSat
{
    return min(a + b, kPairSat);
}
struct OpSatAdd { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return sat_add(a, b); } };

// What the binning kernels keep per block of 256 points, per tile and per pair (device pointers into the workspace).
// Blocks of points per workgroup of k_count_visible, as a power of two: 16, one a wavefront, or 128 where that still makes 512
// workgroups. Every block with a listed point adds up the sums of all workgroups before its own, which grows as the square of the number
// of points (binning of 100M points, a tenth of them seen: 1,061 us with 16, 945 with 128; of 32M 319 and 317).
inline uint32_t super_shift(int n) { return n > 1 << 24 ? 7u : 4u; }
struct BinArrays {
    uint32_t* touched;           // [n] tiles per point, 0 = not listed
    uint2* blk;                  // [blocks] listed points and their pairs (saturating)
    uint2* sup;                  // [blocks >> super_shift] the same per 2^super_shift blocks
    uint2* blk_at;               // [blocks] listed points and pairs in the blocks before this one (of blocks with a listed point)
    uint4* blk_cells;            // [blocks] {tiles the block's pairs lie on or kDirect, x | y << 16 of its rectangle of tiles, its width, -}
    uint2* cells;                // [cap] those tiles, from blk_at.y on: {x | y << 16, pairs of the blocks that counted the tile before}
    uint32_t* ranges;            // [tiles][2] {0, pairs} from k_tile_count, {start, end} from k_tile_lists on
    uint32_t* order;             // [n] listed points in index order ("rank" -> point)
    uint32_t* offsets;           // [n + 1] first pair of each rank; offsets[listed] = pair total
    uint32_t* slot_base;         // [n] first pair of each listed point, by point index
    uint32_t* depth_bits;        // [n] bit pattern of the depth, by point index
    uint2* pairs;                // [cap] {depth bits, point index}, tile by tile
    uint32_t* chunk_rank;        // rank owning the first pair of every chunk (pair_reduce.h)
    uint32_t super_shift;
    uint32_t cap;
    uint32_t* status;
};

// ---- the pairs of a block of 256 points, spread over the kThreads threads of its workgroup --------------------------------------------------
// A pair's slot is its place in the order by point, then row by row over the point's tile rectangle; slots at or beyond the
// capacity are dropped. Points of fewer than kWidePairs pairs are walked together, 64 pairs per wavefront and step, whatever
// the mix of sizes: their pairs are numbered by a prefix sum, and the owner of a number is the last point whose range
// starts at or before it. The points whose range starts inside a step leave their number at that place in LDS, and a
// running maximum over the lanes (DPP) hands every lane its owner; the owner of the step's first pair is counted from the
// starts, four per lane. The wavefronts take the steps in turn, so a block with thousands of pairs keeps all of them busy.
// Wider points are walked by the whole workgroup one after the other, kThreads pairs per trip of a few additions (one splat over
// the whole image would keep a wavefront at its steps of 64 when all others have ended).
constexpr uint32_t kWidePairs = 256;

template <int kThreads>
struct PairLds {
    static constexpr int kWaves = kThreads / 64;
    uint32_t start[256];      // first number of the point's pairs among those walked together, ~0 if it has none
    uint32_t at[256];         // slot of its first pair
    uint32_t xy[256];         // its rectangle: x | y << 16 of the first tile (a grid has at most 4096 x 4096 tiles)
    uint32_t size[256];       // width | height << 16
    uint32_t mark[kWaves][64];
    uint16_t wide[256];       // the wide points
    uint32_t sums[3][4];
    uint4 box[4];             // (k_tile_count)
    uint32_t num_wide;
};

struct PointPairs {           // this thread's point of the block
    uint32_t cnt;             // pairs (tiles touched), 0 = not listed
    uint32_t slot_rank;       // listed points before it
    uint32_t at;              // pairs before it (saturating)
    int x0, y0, x1, y1;
};

// What of point i says where its pairs lie (nothing for a point that is culled). Asked for at once: reading the count of tiles that
// k_count_visible left, and then the rest for the points that have any, would be two round trips in a row.
struct PointExtent { int radius; float mx, my; };
__device__ __forceinline__ PointExtent point_extent(const BinInput& in, int i)      // (a block's points are its first 256 threads')
{
    if (threadIdx.x >= 256u || i >= in.n) return PointExtent{0, 0.f, 0.f};
    return PointExtent{in.radius[i], in.mean2d[i], in.mean2d[(size_t)in.n + i]};
}

// Its pairs (slot_rank and at are lay_out_pairs()'s).
__device__ __forceinline__ PointPairs point_pairs(const CamDev& cam, const PointExtent& e)
{
    PointPairs P;
    P.cnt = 0u;
    P.x0 = P.y0 = P.x1 = P.y1 = 0;
    if (e.radius > 0) {
        tile_rect(cam, e.mx, e.my, e.radius, P.x0, P.y0, P.x1, P.y1);
        P.cnt = (uint32_t)(max(P.x1 - P.x0, 0) * max(P.y1 - P.y0, 0));
    }
    return P;
}

// Lays the block's points out for walk_pairs(). before: listed points and pairs of the blocks before this one. Returns the
// number of pairs that are walked together. Every thread of the workgroup calls it; it ends with the LDS written and visible.
template <int kThreads>
__device__ __forceinline__ uint32_t lay_out_pairs(PairLds<kThreads>& S, uint2 before, PointPairs& P)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool vis = P.cnt > 0u;
    const bool wide = P.cnt >= kWidePairs;
    const uint32_t narrow = wide ? 0u : P.cnt;
    const unsigned long long vm = __ballot(vis);
    const uint32_t inc = wave_inclusive_scan(P.cnt, OpSatAdd{});
    const uint32_t ninc = wave_inclusive_scan(narrow, OpAdd{});      // (at most 255 * 256 in all)
    if (threadIdx.x == 0) S.num_wide = 0u;
    if (lane == 63 && wave < 4) { S.sums[0][wave] = (uint32_t)__popcll(vm); S.sums[1][wave] = inc; S.sums[2][wave] = ninc; }
    __syncthreads();
    const uint32_t below = __shfl_up(inc, 1, 64);            // exclusive = the lane below's inclusive sum
    P.slot_rank = before.x + (uint32_t)__popcll(vm & ((1ull << lane) - 1ull));
    P.at = sat_add(before.y, lane == 0 ? 0u : below);
    uint32_t nat = ninc - narrow, total = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) { P.slot_rank += S.sums[0][w]; P.at = sat_add(P.at, S.sums[1][w]); nat += S.sums[2][w]; }
        total += S.sums[2][w];
    }
    if (kThreads == 256 || threadIdx.x < 256u) {
        S.start[threadIdx.x] = narrow ? nat : 0xffffffffu;
        S.at[threadIdx.x] = P.at;
        S.xy[threadIdx.x] = (uint32_t)P.x0 | (uint32_t)P.y0 << 16;
        S.size[threadIdx.x] = (uint32_t)(P.x1 - P.x0) | (uint32_t)(P.y1 - P.y0) << 16;
    }
    if (wide) S.wide[atomicAdd(&S.num_wide, 1u)] = (uint16_t)threadIdx.x;
    __syncthreads();
    return total;
}

// For every pair of the block whose slot lies below the capacity: done(pair(x, y, slot), slot, place of its point in the block).
// Between the two lie up to four other pairs of the thread, so that what pair() fetches has time to arrive.
template <int kThreads, class Pair, class Done>
__device__ __forceinline__ void walk_pairs(PairLds<kThreads>& S, uint32_t total, uint32_t cap, Pair pair, Done done)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t st[4];
#pragma unroll
    for (uint32_t q = 0; q < 4u; ++q) st[q] = S.start[q * 64u + lane];
    for (uint32_t base = wave * 64u; base < total; base += (uint32_t)kThreads) {
        uint32_t first = 0u;      // owner of the step's first pair
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q) {
            const unsigned long long m = __ballot(st[q] <= base);
            if (m) first = q * 64u + 63u - (uint32_t)__builtin_clzll(m);
        }
        S.mark[wave][lane] = first;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (uint32_t q = 0; q < 4u; ++q)
            if (st[q] - base < 64u) S.mark[wave][st[q] - base] = q * 64u + lane;      // (a start before base wraps past 64)
        __builtin_amdgcn_wave_barrier();
        int own = (int)S.mark[wave][lane];
        __builtin_amdgcn_wave_barrier();
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x111, 0xf, 0xf, false));      // row_shr:1
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x112, 0xf, 0xf, false));      // row_shr:2
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x114, 0xf, 0xf, false));      // row_shr:4
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x118, 0xf, 0xf, false));      // row_shr:8
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x142, 0xa, 0xf, false));      // row_bcast:15 into rows 1 and 3
        own = max(own, __builtin_amdgcn_update_dpp(-1, own, 0x143, 0xc, 0xf, false));      // row_bcast:31 into rows 2 and 3
        const uint32_t e = base + lane;
        if (e < total) {
            const uint32_t t = e - S.start[own], w = S.size[own] & 0xffffu, xy = S.xy[own];
            if (S.at[own] + t < cap) {
                // t / w for t, w < 256: the quotient of t + 1/2 stays 1 / (2 w) away from any whole number
                const uint32_t row = (uint32_t)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)w));
                done(pair((xy & 0xffffu) + t - row * w, (xy >> 16) + row, S.at[own] + t), S.at[own] + t, (uint32_t)own);
            }
        }
    }
    const uint32_t num_wide = __builtin_amdgcn_readfirstlane(S.num_wide);
    for (uint32_t k = 0; k < num_wide; ++k) {
        const uint32_t own = S.wide[k], at = S.at[own], xy = S.xy[own], w = S.size[own] & 0xffffu, h = S.size[own] >> 16;
        const uint32_t dy = (uint32_t)kThreads / w, dx = (uint32_t)kThreads - dy * w;      // a step: rows and columns
        uint32_t ty = threadIdx.x / w, tx = threadIdx.x - ty * w;
        for (uint32_t t0 = threadIdx.x; t0 < w * h && at + t0 < cap; t0 += 4u * (uint32_t)kThreads) {
            decltype(pair(0u, 0u, 0u)) p[4];
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t t = t0 + q * (uint32_t)kThreads;
                if (t < w * h && at + t < cap) p[q] = pair((xy & 0xffffu) + tx, (xy >> 16) + ty, at + t);
                tx += dx; ty += dy;
                if (tx >= w) { tx -= w; ++ty; }
            }
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t t = t0 + q * (uint32_t)kThreads;
                if (t < w * h && at + t < cap) done(p[q], at + t, own);
            }
        }
    }
}

// A block's pairs are counted per tile in a table of its rectangle of tiles in LDS. Points in Z-order make that rectangle small: a
// dozen tiles by a dozen on the benchmark's views. The pairs of a block with a larger rectangle than the table (points beside the
// camera, whose splats cover much of a 4K image; points in no spatial order) are counted one by one in memory instead, and the rank
// each gets there is kept for k_pack: its tiles are many and have few pairs each, so the table would save little. (Taking the
// rectangle in bands of the table's size walks all pairs once per band: one 4K street view of 8M points, counting 258 us and
// packing 433; in memory 62 and 181.)
constexpr uint32_t kTableCells = 4096;
constexpr uint32_t kDirect = 0xffffffffu;      // blk_cells.x of such a block

// Threads per block of 256 points, in k_tile_count and the packing kernels. A block's pairs may be thousands, and where the blocks
// do not fill the chip the largest one is the launch: 1,024 threads (30k points at 1031x517, counting / packing 13.9 / 14.8 us with 256,
// 8.7 / 9.2 with 1,024; 200k at 1280x720 28.3 / 32.6 and 24.6 / 25.3 for two views). Where they do, 256 (1M points, 256 / 1,024:
// 20.6 / 29.8 and 32.4 / 31.9).
inline int block_threads(int n) { return (n + 255) / 256 <= 1024 ? 1024 : 256; }

// One block of 256 consecutive points. A listed point gets its rank among the listed points (index order), its raster
// record (store(i, load(i, its extent)), supplied by the variant), and the slots [at, at + count) of its pairs, where the backward
// pass leaves their partial sums. Its pairs go into the tiles' lists: k_tile_count has reserved room in each list for all pairs of
// the block, and here every pair takes the next place of its tile's room (an LDS counter per tile of the block). So a list holds its
// pairs in no particular order; k_tile_depth_sort orders them by depth bits and, among equals, by point index.
// A chain of round trips to memory per block, so what can be asked for early is: the record's parts before the block is laid out,
// the tiles' starts before the record is written.
template <int kThreads, class Load, class Store>
__device__ __forceinline__ void pack_block(const BinInput& in, const CamDev& cam, const BinArrays& A, const float* __restrict__ depth, Load load, Store store)
{
    __shared__ PairLds<kThreads> S;
    __shared__ uint32_t sNext[kTableCells];      // where the next pair of each tile goes
    __shared__ uint32_t sDepth[256];
    const uint32_t blk = blockIdx.x;
    const int i = (int)(blk * 256u + threadIdx.x);
    const uint2 before = A.blk_at[blk];
    const uint4 box = A.blk_cells[blk];
    const int chunk_bits = gather_chunk_bits(min(A.status[kStNumDup], A.cap));
    // a block none of whose points is listed has nothing to write (most blocks, when the view sees a tenth of a large cloud)
    if (A.blk[blk].x == 0u) return;
    const PointExtent extent = point_extent(in, i);
    PointPairs P = point_pairs(cam, extent);
    const bool listed = P.cnt > 0u;
    decltype(load(i, extent)) rec;
    uint32_t bits = 0u;
    if (listed) { rec = load(i, extent); bits = __float_as_uint(depth[i]); }
    // 1,024 of the block's tiles; more are fetched where they are used
    constexpr uint32_t kPer = 1024u / (uint32_t)kThreads;
    uint2 cell[kPer];
    uint32_t start[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t j = k * (uint32_t)kThreads + threadIdx.x;
        cell[k] = make_uint2(0u, 0u);
        if (j < box.x && box.x != kDirect) cell[k] = A.cells[before.y + j];
    }
    const auto tile_of = [&](const uint2& c) { return (c.x >> 16) * (uint32_t)cam.TX + (c.x & 0xffffu); };
    const uint32_t total = lay_out_pairs(S, before, P);
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        start[k] = 0u;
        if (k * (uint32_t)kThreads + threadIdx.x < box.x && box.x != kDirect) start[k] = A.ranges[2u * tile_of(cell[k])];
    }
    if (listed) {
        sDepth[threadIdx.x] = bits;
        A.order[P.slot_rank] = (uint32_t)i;
        A.offsets[P.slot_rank] = P.at;
        A.slot_base[i] = P.at;
        A.depth_bits[i] = bits;
        store(i, rec);
        // which rank owns the first pair of every chunk (for the pair-balanced gather of the backward pass)
        const uint32_t end = min(P.at + P.cnt, A.cap);
        for (uint32_t c = (P.at + (1u << chunk_bits) - 1u) >> chunk_bits; (uint64_t)c << chunk_bits < end; ++c) A.chunk_rank[c] = P.slot_rank;
    }
    if (box.x == 0u) return;                     // every pair lies beyond the capacity
    const auto place = [&](uint32_t pos, uint32_t own) {
        if (pos < A.cap) A.pairs[pos] = make_uint2(sDepth[own], blk * 256u + own);      // (always, for consistent inputs)
    };
    if (box.x == kDirect) {
        __syncthreads();                         // (the depths)
        const uint32_t* const rank = reinterpret_cast<const uint32_t*>(A.cells) + before.y;
        walk_pairs(S, total, A.cap, [&](uint32_t x, uint32_t y, uint32_t at) { return make_uint2(rank[at], A.ranges[2u * (y * (uint32_t)cam.TX + x)]); },
                   [&](const uint2& p, uint32_t, uint32_t own) { place(p.x + p.y, own); });
        return;
    }
    const uint32_t bx = box.y & 0xffffu, by = box.y >> 16, bw = box.z;
    const auto put = [&](const uint2& c, uint32_t at) { sNext[((c.x >> 16) - by) * bw + (c.x & 0xffffu) - bx] = at + c.y; };
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (k * (uint32_t)kThreads + threadIdx.x < box.x) put(cell[k], start[k]);
    for (uint32_t j = 1024u + threadIdx.x; j < box.x; j += (uint32_t)kThreads) {
        const uint2 c = A.cells[before.y + j];
        put(c, A.ranges[2u * tile_of(c)]);
    }
    __syncthreads();
    walk_pairs(S, total, A.cap, [&](uint32_t x, uint32_t y, uint32_t) { return atomicAdd(&sNext[(y - by) * bw + x - bx], 1u); },
               [&](uint32_t pos, uint32_t, uint32_t own) { place(pos, own); });
}

}  // namespace pbdr
