// Device helpers shared by the compositing kernels of the 3D-Gaussian and the 2D-surfel variants.
#pragma once
#include "pbdr_internal.h"

namespace pbdr {

constexpr int kBatch = 256;

struct TileCtx {
    int px, py;       // this lane's pixel (image coordinates)
    int tx0, ty0;     // tile origin in pixels (image coordinates)
    int tix, tiy;     // tile coordinates within the call's tile grid
    bool inside;      // the pixel belongs to the rendered patch
    uint32_t pix;     // its index in the output buffers
    uint32_t start, end;
};

// Workgroup b takes tile tile_order[b]: the hardware starts workgroups in index order, and the order array lists the
// tiles with the longest lists first (k_tile_lists), so the launch does not end on a few long tiles with the chip idle.
__device__ __forceinline__ TileCtx tile_ctx(const CamDev& cam, const uint32_t* __restrict__ ranges,
                                            const uint32_t* __restrict__ tile_order)
{
    TileCtx c;
    const int tile = (int)tile_order[blockIdx.x];
    const int ty = tile / cam.TX, tx = tile - ty * cam.TX;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    c.tix = tx; c.tiy = ty;
    c.tx0 = (cam.otx + tx) * kTile; c.ty0 = (cam.oty + ty) * kTile;
    c.px = c.tx0 + (wave & 1) * 8 + (lane & 7);
    c.py = c.ty0 + (wave >> 1) * 8 + (lane >> 3);
    c.inside = c.px >= cam.rx0 && c.px < cam.rx1 && c.py >= cam.ry0 && c.py < cam.ry1;
    c.pix = (uint32_t)(c.py - cam.ry0) * (uint32_t)cam.W + (uint32_t)(c.px - cam.rx0);
    c.start = ranges[2 * tile];
    c.end = ranges[2 * tile + 1];
    return c;
}

// Asks for 16 bytes per active lane, from src to the wavefront's 16 * lane bytes behind dst (uniform) in LDS, without a
// register in between. The issuing wavefront waits with wait_loads() before anybody reads them. (The builtin for this
// instruction makes the compiler wait for the load before the next LDS read, whatever that reads.)
__device__ __forceinline__ void load_to_lds16(const void* src, void* dst)
{
    const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)dst);
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0" : "=&s"(m0) : "s"(at), "v"(src) : "memory");
}
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, false));
}

// Sums eight values over each quad of lanes: lane r of the quad is left with the sums of values 2 r and 2 r + 1.
__device__ __forceinline__ void quad_sum8(const float (&v)[8], int quad_lane, float2& out)
{
    const bool hi = (quad_lane & 2) != 0, odd = (quad_lane & 1) != 0;
    float a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float keep = hi ? v[k + 4] : v[k], send = hi ? v[k] : v[k + 4];
        a[k] = keep + dpp_move<0x4E>(send);        // quad_perm:[2,3,0,1]
    }
    const float k0 = odd ? a[2] : a[0], s0 = odd ? a[0] : a[2], k1 = odd ? a[3] : a[1], s1 = odd ? a[1] : a[3];
    out.x = k0 + dpp_move<0xB1>(s0);               // quad_perm:[1,0,3,2]
    out.y = k1 + dpp_move<0xB1>(s1);
}

// sum over each quad of lanes, in all of them
__device__ __forceinline__ float quad_sum(float v)
{
    asm volatile("" : "+v"(v));   // keeps a product that feeds v from being fused into the first add (which would cost the DPP form)
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    return v;
}

// The cells of half a tile, bit 4 r + c for row r and column c of its two rows of four, in the order the kernels keep them: four
// bits per quadrant, its cells in row order.
__device__ __forceinline__ uint32_t by_quadrant(uint32_t m)
{
    return (m & 3u) | ((m >> 2) & 12u) | ((m << 2) & 0x30u) | (m & 0xc0u);
}

// One blend in list order. ok: lanes whose alpha counts; live: lanes whose pixel is still open, which is updated by the
// stop rule. Returns whether this lane blends. (A lane that is not live may set its bit of "stops": it is not live anyway.)
__device__ __forceinline__ bool blend_decision(unsigned long long& live, bool ok, float Tn)
{
    const unsigned long long m = __ballot(ok);
    live &= ~(m & __ballot(Tn < kTStop));
    return __builtin_amdgcn_inverse_ballot_w64(live & m);
}

}  // namespace pbdr
