// Device code shared by the binning kernels of the 3D-Gaussian and the 2D-surfel variants: the block of 256 consecutive
// points that compacts its visible points, writes their raster records and emits their (tile, point) pairs.
#pragma once
#include "pbdr_internal.h"
#include "pair_reduce.h"

namespace pbdr {

// Pair counts are summed with saturation at 2^31 - 1: a degenerate state (many screen-filling splats) cannot wrap the
// 32-bit prefix sums; everything at or beyond the capacity (< 2^30) is dropped and reported as overflow.
constexpr uint32_t kPairSat = 0x7fffffffu;
__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b)      // a, b <= kPairSat
{
    return min(a + b, kPairSat);
}

__device__ __forceinline__ uint32_t wave_inclusive_scan_sat(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v = sat_add(v, t);
    }
    return v;
}

// What the pair emission reads and writes (device pointers into the workspace).
struct BinArrays {
    const uint32_t* touched;     // [n] tiles per point, 0 = not listed
    const uint32_t* blk_vis;     // [blocks] listed points in the blocks before this one
    const uint32_t* blk_pairs;   // [blocks] pairs of the blocks before this one (saturating)
    const uint32_t* blk_order;   // [blocks] the block of points each workgroup takes: those with the most pairs first
    const uint32_t* blk_count;   // [blocks] listed points of each block
    uint32_t* order;             // [n] listed points in index order ("rank" -> point)
    uint32_t* offsets;           // [n + 1] first pair of each rank; offsets[listed] = pair total (written by the block scan)
    uint32_t* slot_base;         // [n] first pair of each listed point, by point index
    uint32_t* depth_bits;        // [n] bit pattern of the depth, by point index
    uint32_t* tkeys;             // [cap] tile id of each pair, in emission order
    uint32_t* tvals;             // [cap] point index of each pair
    uint32_t* chunk_rank;        // rank owning every 256th pair (pair_reduce.h)
    uint32_t cap;
    uint32_t* status;
};

// One block of 256 consecutive points. A listed point gets its rank among the listed points (index order), its raster
// record (pack(i), supplied by the variant), and the slots [at, at + count) of the pair list, where its pairs go in
// row-major order over its tile rectangle. Every (tile, point) pair of a wavefront's 64 consecutive points is written
// by whichever lane comes next, so the work is balanced whatever the mix of small and large splats: the pairs of those
// 64 points occupy one contiguous range (the slots are a prefix sum); lane l writes slots B + l, B + l + 64, ... and
// finds the owning point of a slot from the range starts (see the loop). Points are emitted in index
// order: the depth order of each tile's list is made afterwards, tile by tile (k_tile_depth_sort).
// In a block that holds a point with kWideBlock pairs or more, the points with kWidePairs or more are left out of that loop
// and written by the whole workgroup, 256 slots per trip of two stores and four additions: a step of 64 slots is a chain of
// LDS and cross-lane reads, and one splat over the whole image kept one wavefront at it when all others had ended. 1M disks
// at 1920x1080, three of eight scenes with such a splat: this kernel 76 -> 23 us, step 785 -> 727, 749 -> 725 and 831 -> 810 us;
// scenes without one as before (within 0.1 %).
// A trip is a step that four wavefronts share, so it pays from somewhat over 256 slots: all lists of 300 points at 1920x1080,
// without / with, 119.4 / 120.6 us at 289 tiles a point, 123.2 / 121.5 at 306, 140.5 / 123.3 at 380, 1033 / 307 over the image.
// And doing both after one another costs more than either (points on 225 to 256 tiles, half of them left out: 105.1 / 114.1),
// so a block of points below kWideBlock leaves out none (105.1). A wavefront without such a point takes the loop without the
// test that steps over their slots (points on 210 tiles: 105.3 -> 101.2).
constexpr uint32_t kWidePairs = 256, kWideBlock = 320;

template <class Pack>
__device__ __forceinline__ void pack_dup_block(const BinInput& in, const CamDev& cam, const BinArrays& A,
                                               const float* __restrict__ depth, Pack pack)
{
    __shared__ uint32_t sMark[4][64];      // per wavefront: which lane's range starts at each slot of the current step
    __shared__ uint32_t sVis[4], sPairs[4], sLarge[4];
    __shared__ uint4 sWide[256];           // the block's wide points: first slot; pairs; x0, y0; width of the rectangle, place in the block
    __shared__ uint32_t sNumWide;
    // the blocks with many pairs are started first: their wavefronts run longest (64 slots per step), and in index order
    // the launch ended on the few that happened to come late
    const uint32_t blk = A.blk_order[blockIdx.x];
    // a block none of whose points is listed has nothing to write (most blocks, when the view sees a tenth of a large cloud)
    if (A.blk_count[blk] == 0u) return;
    const int i = (int)(blk * 256u + threadIdx.x);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t cnt = (i < in.n) ? A.touched[i] : 0u;
    const bool vis = cnt > 0u;
    const unsigned long long vm = __ballot(vis);
    const uint32_t inc = wave_inclusive_scan_sat(cnt);
    const bool large = __ballot(cnt >= kWideBlock) != 0ull;
    if (lane == 63) { sVis[wave] = (uint32_t)__popcll(vm); sPairs[wave] = inc; sLarge[wave] = large ? 1u : 0u; }
    if (threadIdx.x == 0) sNumWide = 0u;
    __syncthreads();
    uint32_t slot = A.blk_vis[blk] + (uint32_t)__popcll(vm & ((1ull << lane) - 1ull));
    const uint32_t below = __shfl_up(inc, 1, 64);                    // exclusive = the lane below's inclusive sum
    uint32_t at = sat_add(A.blk_pairs[blk], lane == 0 ? 0u : below);
#pragma unroll
    for (int w = 0; w < 3; ++w)
        if (w < wave) { slot += sVis[w]; at = sat_add(at, sPairs[w]); }
    int x0 = 0, y0 = 0, x1 = 0, y1 = 0;
    if (vis) {
        const float mx = in.mean2d[i], my = in.mean2d[(size_t)in.n + i];
        tile_rect(cam, mx, my, in.radius[i], x0, y0, x1, y1);
        A.order[slot] = (uint32_t)i;
        A.offsets[slot] = at;
        A.slot_base[i] = at;
        A.depth_bits[i] = __float_as_uint(depth[i]);
        pack(i);
        // which rank owns every 256th pair (for the pair-balanced gather of the backward pass)
        const uint32_t end = min(at + cnt, A.cap);
        for (uint32_t c = (at + kChunkPairs - 1) / kChunkPairs; (uint64_t)c * kChunkPairs < end; ++c) A.chunk_rank[c] = slot;
    }
    const bool wide = cnt >= kWidePairs && (sLarge[0] | sLarge[1] | sLarge[2] | sLarge[3]) != 0u;
    const unsigned long long wide_lanes = __ballot(wide);
    if (wide) {
        const uint32_t pairs = at < A.cap ? min(cnt, A.cap - at) : 0u;      // (a grid has at most 4096 x 4096 tiles)
        sWide[atomicAdd(&sNumWide, 1u)] = make_uint4(at, pairs, (uint32_t)x0 | (uint32_t)y0 << 16, (uint32_t)(x1 - x0) | threadIdx.x << 16);
    }
    const int w = wide ? 0 : x1 - x0;      // 0: no slot of this point is written by the wavefront's loop
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)at, 0);
    const uint32_t last_raw = (uint32_t)__builtin_amdgcn_readlane((int)(at + cnt), 63);
    const uint32_t last = min(last_raw, A.cap);        // slots at or beyond the capacity are dropped
    __builtin_amdgcn_wave_barrier();
    // Uniform trip count: every lane takes part in the cross-lane reads of each step, only lanes with a slot store.
    // The owner of slot u is the last lane whose range starts at or before u (the ranges are a prefix sum: no gaps, and
    // the ranges of listed points start at distinct slots). Per step of 64 slots: the lanes whose range starts inside
    // the step leave their number at that slot's place in LDS, and a running maximum over the lanes (DPP), carried from
    // step to step, hands every slot its owner - one LDS round trip per step where a binary search over the 64 range
    // ends took six in a row, which is what the wavefronts with thousands of pairs, the last to finish, were made of.
    int carry = -1;
    const auto step = [&](uint32_t base) {
        const uint32_t u = base + lane;
        sMark[wave][lane] = 0xffffffffu;
        if (vis && at - base < 64u) sMark[wave][at - base] = (uint32_t)lane;      // at >= base or the difference wraps past 64
        __builtin_amdgcn_wave_barrier();
        int lo = (int)sMark[wave][lane];                  // -1 where no range starts
        __builtin_amdgcn_wave_barrier();
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x111, 0xf, 0xf, false));      // row_shr:1
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x112, 0xf, 0xf, false));      // row_shr:2
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x114, 0xf, 0xf, false));      // row_shr:4
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x118, 0xf, 0xf, false));      // row_shr:8
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x142, 0xa, 0xf, false));      // row_bcast:15 into rows 1 and 3
        lo = max(lo, __builtin_amdgcn_update_dpp(-1, lo, 0x143, 0xc, 0xf, false));      // row_bcast:31 into rows 2 and 3
        lo = max(lo, carry);
        carry = __builtin_amdgcn_readlane(lo, 63);
        const int src = max(lo, 0);
        const int ox0 = __shfl(x0, src, 64), oy0 = __shfl(y0, src, 64), ow = __shfl(w, src, 64);
        const uint32_t oat = (uint32_t)__shfl((int)at, src, 64);
        const uint32_t oid = blk * 256u + (uint32_t)(wave * 64 + src);
        if (u < last && lo >= 0 && ow > 0) {
            const int t = (int)(u - oat);
            const int ty = oy0 + t / ow, tx = ox0 + t - (t / ow) * ow;
            A.tkeys[u] = (uint32_t)(ty * cam.TX + tx);
            A.tvals[u] = oid;
        }
    };
    if (wide_lanes == 0ull) {
        for (uint32_t base = first; base < last; base += 64) step(base);
    } else {
        for (uint32_t base = first; base < last;) {
            step(base);
            base += 64u;
            if (carry >= 0 && ((wide_lanes >> carry) & 1ull) != 0ull) {      // on to the step in which a wide point's range ends
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)(at + cnt), carry);
                if (end > base) base += (end - base) & ~63u;
            }
        }
    }
    __syncthreads();
    const uint32_t num_wide = __builtin_amdgcn_readfirstlane(sNumWide);
    for (uint32_t k = 0; k < num_wide; ++k) {
        const uint4 e = sWide[k];
        const uint32_t ow = e.w & 0xffffu, id = blk * 256u + (e.w >> 16);
        const uint32_t dy = 256u / ow, dx = 256u - dy * ow;      // a step of 256 slots: rows and columns
        uint32_t ty = threadIdx.x / ow, tx = threadIdx.x - ty * ow;
        uint32_t key = ((e.z >> 16) + ty) * (uint32_t)cam.TX + (e.z & 0xffffu) + tx;
        const uint32_t dkey = dy * (uint32_t)cam.TX + dx, wrap = (uint32_t)cam.TX - ow;
        for (uint32_t t = threadIdx.x; t < e.y; t += 256u) {
            A.tkeys[e.x + t] = key;
            A.tvals[e.x + t] = id;
            tx += dx;
            key += dkey;
            if (tx >= ow) { tx -= ow; key += wrap; }
        }
    }
    if (lane == 0 && last_raw > A.cap) A.status[kStOverflow] = 1u;
}

}  // namespace pbdr
