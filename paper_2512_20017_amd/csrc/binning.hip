// Tile binning: per-splat tile count + raster record, device prefix sums, per-tile pair counts, the (tile, point) pairs put
// into their tiles' lists, tile ranges and order, depth order inside each tile's list. These are the steps between
// pts_splatting and the per-pixel blend that realise "sorts these view-dependent splats by their distance to the camera
// plane" (paper Sec. 2.1) per 16x16 tile.  All HBM- or latency-bound integer work.
//
// The tile lists are ordered by the 64-bit key (tile << 32 | depth bits), ties by point index. The tile half is a counting
// sort without a pass over the pairs: a block of 256 points, which in Z-order lie on a few dozen tiles, counts its pairs per
// tile in LDS and reserves its room in each of those tiles' lists with one atomic add, and once the lists' starts are known
// every pair is written to its place. The lists come out in no particular order; each is then sorted by depth bits and, among
// equal ones, by point index (k_tile_depth_sort, depth_sort.hip), so the result is the same on every run.
// Five launches where a stable two-pass radix sort of the pairs by tile id took eleven; with the depth sort as it is now, us
// before and now, in turn on one card: 1M points at 1920x1080 472 -> 438 a step, 225 -> 195 an evaluation; 30k at 1031x517 156 -> 129 a
// step; 12,000 at 400x300 79 -> 48 an evaluation. The order of points matters more than before: where a block's points lie all
// over the image, its pairs are on as many tiles, and each costs an atomic add, 26 G/s wherever they go (1M points at 1920x1080, an
// evaluation: in Z-order 213 -> 178 us, in random order 242 -> 300, a tenth of them in random order 214 -> 183). Counting sixteen such blocks
// together in LDS is no faster (k_tile_count 104 -> 145 us): they have one or two pairs a tile, so the adds hardly become fewer.
#include "pbdr_internal.h"
#include "binning_common.h"

namespace pbdr {

// Tiles touched by every point (0 for culled points) and, per block of 256 consecutive points and per 2^super_shift of them,
// the number of points that touch at least one tile - those are the points binning lists ("visible" below) - and the number of
// their pairs. A state made by the preprocessing calls has radius == 0 for every point without a tile; a caller-made state with
// radius > 0 and an empty tile rectangle is treated as culled here, so every listed point owns at least one pair.
// Four consecutive points per thread (one 16-byte load of the radii, one 16-byte store of the counts: with one point
// per thread the launch did not keep enough bytes in flight, 2 TB/s at eight million points: 32 -> 21 us there), so a
// wavefront covers exactly one block of 256 points and its two sums need no LDS and no barrier.
template <uint32_t kSuper>
__global__ __launch_bounds__(1024) void k_count_visible(BinInput in, CamDev cam, BinArrays A, uint32_t nranges)
{
    __shared__ uint2 sBlk[16];
    const uint32_t gid = blockIdx.x * 1024u + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // first launch of a binning call: the status words and the tile ranges, which hold the tiles' pair counts first, start at zero
    // (every later kernel of the call comes after this one on the stream)
    if (gid < (uint32_t)kStCleared) A.status[gid] = 0u;
    for (uint32_t k = gid; k < nranges; k += gridDim.x * 1024u) A.ranges[k] = 0u;
    const size_t n = (size_t)in.n;
    uint2 sum = make_uint2(0u, 0u);      // of the wavefront's blocks
#pragma unroll 1
    for (uint32_t q = 0; q < kSuper / 16u; ++q) {
        const size_t blk = (size_t)blockIdx.x * kSuper + q * 16u + wave;      // the wavefront's 256 points
        if (kSuper > 16u && blk * 256u >= n) break;
        const size_t i0 = blk * 256u + (size_t)lane * 4u;
        int r[4] = {0, 0, 0, 0};
        if (i0 + 4u <= n && (reinterpret_cast<uintptr_t>(in.radius) & 15u) == 0u) {
            const int4 v = *reinterpret_cast<const int4*>(in.radius + i0);
            r[0] = v.x; r[1] = v.y; r[2] = v.z; r[3] = v.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) if (i0 + k < n) r[k] = in.radius[i0 + k];
        }
        uint32_t t[4];
        uint32_t vis = 0u, pairs = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            t[k] = 0u;
            if (r[k] > 0) {      // (r[k] is 0 past the end)
                int x0, y0, x1, y1;
                tile_rect(cam, in.mean2d[i0 + k], in.mean2d[n + i0 + k], r[k], x0, y0, x1, y1);
                t[k] = (uint32_t)(max(x1 - x0, 0) * max(y1 - y0, 0));       // <= 2^24: the grid has at most 4096 x 4096 tiles
            }
            vis += t[k] > 0u ? 1u : 0u;
            pairs = sat_add(pairs, t[k]);
        }
        if (i0 + 4u <= n) {
            *reinterpret_cast<uint4*>(A.touched + i0) = make_uint4(t[0], t[1], t[2], t[3]);      // (the array starts on a 256-byte boundary)
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) if (i0 + k < n) A.touched[i0 + k] = t[k];
        }
        vis = wave_reduce(vis, OpAdd{});
        pairs = wave_reduce(pairs, OpSatAdd{});
        if (lane == 0 && blk * 256u < n) A.blk[blk] = make_uint2(vis, pairs);
        sum.x += vis; sum.y = sat_add(sum.y, pairs);
    }
    if (lane == 0) sBlk[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint2 s = make_uint2(0u, 0u);
#pragma unroll
        for (uint32_t w = 0; w < 16u; ++w) { s.x += sBlk[w].x; s.y = sat_add(s.y, sBlk[w].y); }
        A.sup[blockIdx.x] = s;
    }
}

// Listed points and pairs of the blocks before block b.
template <int kThreads>
__device__ __forceinline__ uint2 blocks_before(const BinArrays& A, uint32_t b, uint2* sSum)
{
    const uint32_t s = b >> A.super_shift;
    uint32_t v = 0u, p = 0u;
    for (uint32_t i0 = 0; i0 < s; i0 += 4u * (uint32_t)kThreads) {      // four loads in flight
        uint2 x[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t i = i0 + k * (uint32_t)kThreads + threadIdx.x;
            x[k] = i < s ? A.sup[i] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) { v += x[k].x; p = sat_add(p, x[k].y); }
    }
    const uint32_t i = (s << A.super_shift) + threadIdx.x;      // (at most 128 blocks in a part, and a workgroup has 256 threads)
    if (i < b) {
        const uint2 x = A.blk[i];
        v += x.x; p = sat_add(p, x.y);
    }
    v = wave_reduce(v, OpAdd{});
    p = wave_reduce(p, OpSatAdd{});
    if ((threadIdx.x & 63u) == 0u) sSum[threadIdx.x >> 6] = make_uint2(v, p);
    __syncthreads();
    uint2 r = make_uint2(0u, 0u);
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) { r.x += sSum[w].x; r.y = sat_add(r.y, sSum[w].y); }
    return r;
}

// Pairs per tile, and every block's room in the tiles' lists: the block's pairs are counted per tile in LDS, one atomic add per
// tile then says how many pairs of other blocks counted so far (the order of the blocks in a list varies from run to run; the
// depth sort does not depend on it). What precedes a block of points it adds up by itself from the counts, so no workgroup
// waits for another. The last block leaves the totals.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_tile_count(BinInput in, CamDev cam, BinArrays A, uint32_t nb)
{
    __shared__ PairLds<kThreads> S;
    __shared__ uint32_t sCount[kTableCells / 2];      // two to a word: a block has at most 256 pairs on a tile
    __shared__ uint2 sSum[kThreads / 64];
    __shared__ uint16_t sList[kTableCells];               // the cells of the table that are not zero
    __shared__ uint32_t sListed;
    const uint32_t blk = blockIdx.x;
    const uint2 mine = A.blk[blk];
    if (mine.x == 0u && blk + 1u != nb) return;
    const int i = (int)(blk * 256u + threadIdx.x);
    const PointExtent extent = point_extent(in, i);
    if (threadIdx.x == 0) sListed = 0u;
    const uint2 before = blocks_before<kThreads>(A, blk, sSum);
    PointPairs P = point_pairs(cam, extent);
    if (blk + 1u == nb && threadIdx.x == 0) {
        const uint32_t listed = min(before.x + mine.x, (uint32_t)in.n), pairs = sat_add(before.y, mine.y);
        A.status[kStNumVis] = listed;
        A.status[kStNumDup] = pairs;
        A.status[kStOverflow] = pairs > A.cap ? 1u : 0u;
        A.offsets[listed] = pairs;
    }
    if (threadIdx.x == 0) A.blk_at[blk] = before;
    if (mine.x == 0u || before.y >= A.cap) {
        if (threadIdx.x == 0) A.blk_cells[blk] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const uint32_t total = lay_out_pairs(S, before, P);
    {   // the rectangle of tiles that holds the block's
        // (the lower edges as their distance from 65,535, so that all four are maxima)
        const uint32_t lo_x = wave_reduce(P.cnt ? 0xffffu - (uint32_t)P.x0 : 0u, OpMax{}), lo_y = wave_reduce(P.cnt ? 0xffffu - (uint32_t)P.y0 : 0u, OpMax{});
        const uint32_t hi_x = wave_reduce(P.cnt ? (uint32_t)P.x1 : 0u, OpMax{}), hi_y = wave_reduce(P.cnt ? (uint32_t)P.y1 : 0u, OpMax{});
        if ((threadIdx.x & 63u) == 0u && threadIdx.x < 256u) S.box[threadIdx.x >> 6] = make_uint4(lo_x, lo_y, hi_x, hi_y);
        __syncthreads();
    }
    const uint4 q0 = S.box[0], q1 = S.box[1], q2 = S.box[2], q3 = S.box[3];
    const uint32_t bx = 0xffffu - __builtin_amdgcn_readfirstlane(max(max(q0.x, q1.x), max(q2.x, q3.x)));
    const uint32_t by = 0xffffu - __builtin_amdgcn_readfirstlane(max(max(q0.y, q1.y), max(q2.y, q3.y)));
    const uint32_t bw = __builtin_amdgcn_readfirstlane(max(max(q0.z, q1.z), max(q2.z, q3.z))) - bx;
    const uint32_t bh = __builtin_amdgcn_readfirstlane(max(max(q0.w, q1.w), max(q2.w, q3.w))) - by;
    if (bw * bh > kTableCells) {
        uint32_t* const rank = reinterpret_cast<uint32_t*>(A.cells) + before.y;      // (its pairs' slots hold two words each)
        walk_pairs(S, total, A.cap, [&](uint32_t x, uint32_t y, uint32_t) { return atomicAdd(&A.ranges[2u * (y * (uint32_t)cam.TX + x) + 1u], 1u); },
                   [&](uint32_t r, uint32_t at, uint32_t) { rank[at] = r; });
        if (threadIdx.x == 0) A.blk_cells[blk] = make_uint4(kDirect, 0u, 0u, 0u);
        return;
    }
    const uint32_t cells = bw * bh;
    for (uint32_t c = threadIdx.x; 2u * c < cells; c += (uint32_t)kThreads) sCount[c] = 0u;
    __syncthreads();
    walk_pairs(S, total, A.cap, [&](uint32_t x, uint32_t y, uint32_t) {
        const uint32_t c = (y - by) * bw + x - bx;
        return atomicAdd(&sCount[c >> 1], 1u << ((c & 1u) << 4));
    }, [](uint32_t, uint32_t, uint32_t) {});
    __syncthreads();
    // (the cells are listed first: an atomic add of a cell as the search comes to it would be a round trip to memory each)
    const auto count_of = [&](uint32_t c) { return (sCount[c >> 1] >> ((c & 1u) << 4)) & 0xffffu; };
    for (uint32_t c = threadIdx.x; c < cells; c += (uint32_t)kThreads)
        if (count_of(c)) sList[atomicAdd(&sListed, 1u)] = (uint16_t)c;
    __syncthreads();
    const uint32_t listed = __builtin_amdgcn_readfirstlane(sListed);
    for (uint32_t j0 = 0; j0 < listed; j0 += 4u * (uint32_t)kThreads) {      // four adds in flight
        uint32_t at[4], xy[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t j = j0 + k * (uint32_t)kThreads + threadIdx.x;
            if (j < listed) {
                const uint32_t c = sList[j], row = c / bw, x = bx + c - row * bw, y = by + row;
                xy[k] = x | y << 16;
                at[k] = atomicAdd(&A.ranges[2u * (y * (uint32_t)cam.TX + x) + 1u], count_of(c));
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t j = j0 + k * (uint32_t)kThreads + threadIdx.x;
            if (j < listed) A.cells[before.y + j] = make_uint2(xy[k], at[k]);      // (fewer tiles than pairs below the capacity)
        }
    }
    if (threadIdx.x == 0) A.blk_cells[blk] = make_uint4(listed, bx | by << 16, bw, 0u);
}

// 3D Gaussians: the raster record (64 bytes) of a listed point (see binning_common.h for the rest of the block's work).
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_pack(SplatsDev sp, CamDev cam, BinArrays A, Packed* __restrict__ packed)
{
    const size_t N = (size_t)sp.n;
    struct Parts { float qa, qb, qc, o, red, green, blue, mx, my; int radius; };
    pack_block<kThreads>(BinInput{sp.n, sp.mean2d, sp.radius}, cam, A, sp.depth,
        [&](int i, const PointExtent& e) {
            return Parts{sp.conic[i], sp.conic[N + i], sp.conic[2 * N + i], sp.opacity[i], sp.color[i], sp.color[N + i], sp.color[2 * N + i],
                         e.mx, e.my, e.radius};
        },
        [&](int i, const Parts& p) {
            float4* dst = reinterpret_cast<float4*>(packed + i);
            const float A = 0.5f * kLog2e * p.qa, B = kLog2e * p.qb, C = 0.5f * kLog2e * p.qc, o = p.o;
            const float L = o < 0.f ? -__builtin_inff() : __log2f(o);      // below zero: blends nowhere, as zero does (NaN stays NaN)
            const bool safe = safely_definite(A, B, C);
            dst[0] = make_float4(p.mx, p.my, A, B);
            dst[1] = make_float4(C, L, p.red, p.green);
            dst[2] = make_float4(p.blue, __int_as_float(p.radius), o, __uint_as_float(!safe ? 0u : o <= 0.98f ? kSplatPlain : kSplatDefinite));
            dst[3] = splat_ellipse(A, B, C, L);
        });
}

__global__ __launch_bounds__(256) void k_bin_begin(uint32_t* __restrict__ status, uint32_t* __restrict__ ranges, size_t nranges,
                                                   uint32_t* __restrict__ tile_order)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < (size_t)kStCleared) status[i] = 0u;
    if (i < nranges) ranges[i] = 0u;
    if (2 * i < nranges) tile_order[i] = (uint32_t)i;      // no lists: any order will do
}

// Where every tile's list starts and ends, and the order in which the compositing kernels take the tiles: longest lists
// first. Workgroups start in index order and a tile's cost grows with its list, so in image order a launch ends on whatever long
// tiles happen to come late, with most of the chip idle. Tiles are put in classes of list length, two per octave (class 0 =
// longest); within a class they keep the image order, so neighbours in the order are still neighbours in the image and share
// splat records in L2. That is a stable counting sort on the class: a thread takes a tile, and a lane finds the lanes of its
// class from six ballots, one per bit of the class, with no loop over the classes present.
constexpr int kOrderClasses = 40;           // < 63; class 63 stands for "no tile"
constexpr uint32_t kOrderChunk = 1024;      // tiles per workgroup, one per thread (eight per thread: 12.0 us instead of 5.5 for 8,160 tiles)
__device__ __forceinline__ uint32_t order_class(uint32_t len)
{
    const uint32_t x = len + 1u;
    const int e = 31 - __clz((int)x);
    const uint32_t half = e > 0 ? (x >> (e - 1)) & 1u : 0u;
    return (uint32_t)(kOrderClasses - 1) - min(2u * (uint32_t)e + half, (uint32_t)(kOrderClasses - 1));
}

// the lanes of the wavefront whose class equals this lane's
__device__ __forceinline__ uint64_t lanes_of_my_class(uint32_t cls)
{
    uint64_t same = ~0ull;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const bool bit = ((cls >> b) & 1u) != 0u;
        const uint64_t set = __ballot(bit);
        same &= bit ? set : ~set;
    }
    return same;
}

// Workgroup g takes the kOrderChunk tiles from g * kOrderChunk on. Where they go also depends on the other workgroups' tiles:
// how many of each class lie in earlier chunks, and in later ones, and how many pairs in earlier ones. Every workgroup counts
// those for itself, so none waits for another. A tile's entry is {0, pairs} until its workgroup makes it {start, end}, in one store of
// eight bytes; whichever of the two another workgroup finds there in one load, the difference is the number of pairs.
template <bool kMulti>                      // more than one chunk
__global__ __launch_bounds__(1024) void k_tile_lists(uint64_t* ranges, uint32_t ntiles, uint32_t* __restrict__ tile_order, uint32_t* __restrict__ status,
                                                     int long_code)
{
    const auto entry = [&](uint32_t t) { return __hip_atomic_load(ranges + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    const auto pairs_of = [](uint64_t r) { return (uint32_t)(r >> 32) - (uint32_t)r; };
    // per class: (earlier chunks,) the 16 wavefronts of this one(, later chunks)
    constexpr uint32_t kOrderSlots = kMulti ? 18u : 16u, kFirst = kMulti ? 1u : 0u;
    constexpr int kPer = (kOrderClasses * kOrderSlots + 63) / 64;
    __shared__ uint32_t count[64 * kOrderSlots];      // [class][slot]: tiles, then where the next tile of (class, slot) goes (class 63: unused, in bounds)
    __shared__ uint32_t other[kMulti ? 2 * kOrderClasses * 16 : 1];      // [earlier, later chunks][class][lane % 16]
    __shared__ uint32_t sPairs[2][16];                // per wavefront: pairs of its tiles, and of its share of the earlier chunks
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    const uint32_t c0 = blockIdx.x * kOrderChunk, c1 = min(ntiles, c0 + kOrderChunk);
    const uint32_t t = c0 + threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t len = t < c1 ? pairs_of(entry(t)) : 0u;
    for (uint32_t i = threadIdx.x; i < 64u * kOrderSlots; i += 1024u) count[i] = 0u;
    if (kMulti)
        for (uint32_t i = threadIdx.x; i < 2u * kOrderClasses * 16u; i += 1024u) other[i] = 0u;
    __syncthreads();
    const uint32_t cls = t < c1 ? order_class(len) : 63u;
    const uint64_t same = lanes_of_my_class(cls);
    if ((same & below) == 0ull && cls != 63u) count[cls * kOrderSlots + kFirst + w] = (uint32_t)__popcll(same);      // first lane of its class
    uint32_t earlier = 0u;
    if (kMulti) {      // the tiles of the other chunks, by class
        // (one of 16 counters per side and class, by lane: a wavefront's tiles are mostly of one class, and additions to
        // one LDS address take their turns)
        for (uint32_t ib = threadIdx.x; ib < ntiles; ib += 4u * 1024u) {
            uint64_t r[4];
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                r[k] = entry(min(ib + k * 1024u, ntiles - 1u));
            }
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) {
                const uint32_t i = ib + k * 1024u;
                if (i < c0) earlier += pairs_of(r[k]);      // (all lists together stay below the capacity, 2^30)
                if (i < ntiles && (i < c0 || i >= c1))
                    atomicAdd(&other[((i < c0 ? 0u : (uint32_t)kOrderClasses) + order_class(pairs_of(r[k]))) * 16u + (lane & 15u)], 1u);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) earlier += (uint32_t)__shfl_xor((int)earlier, d, 64);
        if (lane == 0u) sPairs[1][w] = earlier;
        __syncthreads();
        if (threadIdx.x < 2u * kOrderClasses) {
            uint32_t sum = 0;
#pragma unroll
            for (uint32_t k = 0; k < 16u; ++k) sum += other[threadIdx.x * 16u + k];
            const uint32_t c = threadIdx.x < (uint32_t)kOrderClasses ? threadIdx.x : threadIdx.x - (uint32_t)kOrderClasses;
            count[c * kOrderSlots + (threadIdx.x < (uint32_t)kOrderClasses ? 0u : kOrderSlots - 1u)] = sum;
        }
    }
    // where this thread's list starts
    uint32_t inc = len;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(inc, d);
        if (lane >= (uint32_t)d) inc += up;
    }
    if (lane == 63u) sPairs[0][w] = inc;
    __syncthreads();
    if (w == 0) {      // exclusive prefix sums over (class, slot), classes 0 .. kOrderClasses - 1: kPer consecutive entries per lane
        uint32_t v[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) { v[k] = count[lane * kPer + k]; sum += v[k]; }
        uint32_t incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t up = __shfl_up(incl, d);
            if (lane >= (uint32_t)d) incl += up;
        }
        uint32_t at = incl - sum;
#pragma unroll
        for (int k = 0; k < kPer; ++k) { count[lane * kPer + k] = at; at += v[k]; }
    }
    uint32_t start = inc - len;
#pragma unroll
    for (uint32_t k = 0; k < 16u; ++k) {
        if (k < w) start += sPairs[0][k];
        if (kMulti) start += sPairs[1][k];
    }
    if (t < c1 && len) __hip_atomic_store(ranges + t, (uint64_t)(start + len) << 32 | start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (an empty one stays {0, 0})
    __syncthreads();
    // how many tiles hold 2^(long_code / 2) - 1 entries (1.5 times that if odd) or more: they come first in the order, and the depth sort gives each a whole
    // workgroup (where a class starts)
    if (threadIdx.x == 0 && blockIdx.x == 0) status[kStNumBig] = count[((uint32_t)kOrderClasses - (uint32_t)long_code) * kOrderSlots];
    if (cls != 63u) tile_order[count[cls * kOrderSlots + kFirst + w] + (uint32_t)__popcll(same & below)] = t;
}

// Inspection only: the 64-bit keys (tile << 32 | depth bits) of the sorted pairs, rebuilt from the tile ranges, the
// sorted point indices and the per-point depth bits. One workgroup per tile.
__global__ __launch_bounds__(256) void k_make_keys64(const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tvals,
                                                     const uint32_t* __restrict__ depth_bits, uint32_t cap, uint64_t* __restrict__ keys64)
{
    const uint32_t tile = blockIdx.x;
    const uint32_t s = ranges[2 * tile], e = min(ranges[2 * tile + 1], cap);
    for (uint32_t i = s + threadIdx.x; i < e; i += 256u) keys64[i] = ((uint64_t)tile << 32) | depth_bits[tvals[i]];
}

hipError_t launch_make_keys64(const Layout& L, char* ws, hipStream_t s)
{
    const uint32_t* tv = reinterpret_cast<const uint32_t*>(ws + L.off_vals);
    hipLaunchKernelGGL(k_make_keys64, dim3((unsigned)L.tiles), dim3(256), 0, s, reinterpret_cast<const uint32_t*>(ws + L.off_ranges), tv,
                       reinterpret_cast<const uint32_t*>(ws + L.off_depth_bits), L.cap, reinterpret_cast<uint64_t*>(ws + L.off_pairs));
    return hipGetLastError();
}

hipError_t launch_bin_begin(const Layout& L, char* ws, hipStream_t s)
{
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + L.off_status);
    uint32_t* ranges = reinterpret_cast<uint32_t*>(ws + L.off_ranges);
    // status words and tile ranges start at zero (one launch)
    ProfScope prof(kKFill, s);
    hipLaunchKernelGGL(k_bin_begin, dim3((unsigned)((2 * (size_t)L.tiles + 255) / 256)), dim3(256), 0, s, status, ranges,
                       2 * (size_t)L.tiles, reinterpret_cast<uint32_t*>(ws + L.off_tile_order));
    return hipGetLastError();
}

BinArrays bin_arrays(const Layout& L, char* ws)
{
    const auto u32 = [&](size_t off) { return reinterpret_cast<uint32_t*>(ws + off); };
    BinArrays A;
    A.touched = u32(L.off_touched);
    A.blk = reinterpret_cast<uint2*>(ws + L.off_blk);
    A.sup = reinterpret_cast<uint2*>(ws + L.off_sup);
    A.blk_at = reinterpret_cast<uint2*>(ws + L.off_blk_at);
    A.blk_cells = reinterpret_cast<uint4*>(ws + L.off_blk_cells);
    A.cells = reinterpret_cast<uint2*>(ws + L.off_spare);
    A.ranges = u32(L.off_ranges);
    A.order = u32(L.off_order);
    A.offsets = u32(L.off_offsets);
    A.slot_base = u32(L.off_slot_base);
    A.depth_bits = u32(L.off_depth_bits);
    A.pairs = reinterpret_cast<uint2*>(ws + L.off_pairs);
    A.chunk_rank = u32(L.off_chunk_rank);
    A.super_shift = super_shift(L.n);
    A.cap = L.cap;
    A.status = u32(L.off_status);
    return A;
}

// Everything up to the tiles' lists having their places: tiles per point, listed points and pairs per block of 256 points, pairs
// per tile, the ranges and the order of the tiles. Also the call's first launch: clears the status words and the tile ranges.
hipError_t launch_bin_count(const BinInput& in, const CamDev& cam, const Layout& L, char* ws, hipStream_t s)
{
    if (in.n == 0) return hipSuccess;
    const BinArrays A = bin_arrays(L, ws);
    const unsigned nb = (unsigned)((in.n + 255) / 256);
    const uint32_t ntiles = (uint32_t)(cam.TX * cam.TY);      // the call's tile grid (a patch covers fewer tiles than the image the workspace is sized for)
    {
        ProfScope prof(kKCountVisible, s);
        const dim3 grid(((nb - 1u) >> A.super_shift) + 1u);
        const uint32_t nranges = (uint32_t)(2 * (size_t)L.tiles);
        if (A.super_shift == 4u) hipLaunchKernelGGL(k_count_visible<16>, grid, dim3(1024), 0, s, in, cam, A, nranges);
        else hipLaunchKernelGGL(k_count_visible<128>, grid, dim3(1024), 0, s, in, cam, A, nranges);
    }
    {
        ProfScope prof(kKTileCount, s);
        if (block_threads(in.n) == 256) hipLaunchKernelGGL(k_tile_count<256>, dim3(nb), dim3(256), 0, s, in, cam, A, nb);
        else hipLaunchKernelGGL(k_tile_count<1024>, dim3(nb), dim3(1024), 0, s, in, cam, A, nb);
    }
    ProfScope prof(kKTileLists, s);
    uint64_t* ranges = reinterpret_cast<uint64_t*>(ws + L.off_ranges);
    uint32_t* tile_order = reinterpret_cast<uint32_t*>(ws + L.off_tile_order);
    if (ntiles <= kOrderChunk) hipLaunchKernelGGL(k_tile_lists<false>, dim3(1), dim3(1024), 0, s, ranges, ntiles, tile_order, A.status, long_list_code(ntiles));
    else hipLaunchKernelGGL(k_tile_lists<true>, dim3((ntiles + kOrderChunk - 1u) / kOrderChunk), dim3(1024), 0, s, ranges, ntiles, tile_order, A.status, long_list_code(ntiles));
    return hipGetLastError();
}

hipError_t launch_bin_sort(const SplatsDev& sp, const CamDev& cam, const Layout& L, char* ws, hipStream_t s)
{
    if (sp.n == 0) return launch_bin_begin(L, ws, s);      // nothing to count: only the cleared status words and ranges
    hipError_t e = launch_bin_count(BinInput{sp.n, sp.mean2d, sp.radius}, cam, L, ws, s);
    if (e != hipSuccess) return e;
    {
        ProfScope prof(kKPack, s);
        const unsigned nb = (unsigned)((sp.n + 255) / 256);
        Packed* packed = reinterpret_cast<Packed*>(ws + L.off_packed);
        if (block_threads(sp.n) == 256) hipLaunchKernelGGL(k_pack<256>, dim3(nb), dim3(256), 0, s, sp, cam, bin_arrays(L, ws), packed);
        else hipLaunchKernelGGL(k_pack<1024>, dim3(nb), dim3(1024), 0, s, sp, cam, bin_arrays(L, ws), packed);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_tile_depth_sort(cam, L, ws, s);
}

}  // namespace pbdr
