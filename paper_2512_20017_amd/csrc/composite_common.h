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

__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
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

// Sums eight values over each row of 16 lanes at once by recursive halving: at each of three exchange steps a lane
// keeps half of its values and adds its partner's copy of that half, then one more pairing finishes.
//   step 1: partner lane ^ 8 (row_ror:8);           lanes with bit 3 clear keep values 0..3, the others 4..7
//   step 2: partner lane ^ 7 (row_half_mirror);     lanes with bit 2 clear keep the first two of those, the others the rest
//   step 3: partner lane ^ 3 (quad_perm [3,2,1,0]); lanes with bit 1 clear keep the first of those two
//   last  : partner lane ^ 1 (quad_perm [1,0,3,2]); plain add
// Each partner differs from the lane in exactly the bit that decides the step and in none of the bits that decided
// earlier steps, so both hold the same values. Bits 3 and 2 are the quad a lane sits in, which is what a DPP bank
// mask selects: steps 1 and 2 are two masked adds per output and no select (written as assembly because the compiler
// has no form for a masked DPP write; the s_nop's cover the VALU-write -> DPP-read wait states inside and on both
// sides of the block). 16 VALU instructions instead of 8 x 4. Every lane of the wavefront must be active.
// On return the lane holds the row sum of value number (lane >> 1) & 7; lanes 2k and 2k+1 hold the same number.
__device__ __forceinline__ float row_sum8(const float v[8], bool bit1)
{
    float a[4], c[2];
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %9, %9 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %0, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %4, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %5, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %4, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %5, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "s_nop 1"
        : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(c[0]), "=&v"(c[1])
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
    const float keep = bit1 ? c[1] : c[0], send = bit1 ? c[0] : c[1];
    float d = keep + dpp_move<0x1B>(send);         // quad_perm:[3,2,1,0]
    d += dpp_move<0xB1>(d);                        // quad_perm:[1,0,3,2]
    return d;
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

// ---- bookkeeping of the walks ----------------------------------------------------------------------------------------
// The walks are bound by issue, scalar instructions included, so a visit's bookkeeping is spelled out: which pixels are still
// open is a scalar lane mask and, in the surfel walks, the splats left in a wavefront's batch are a 64-bit scalar mask that
// gives up one bit in one instruction (the 3D walks read lists, see composite.hip).

// the lowest splat left in the mask, taken out of it (m != 0)
__device__ __forceinline__ int take_lowest(unsigned long long& m)
{
    const int j = __builtin_ctzll(m);
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(j));
    return j;
}

// the highest splat left in the mask, taken out of it (m != 0)
__device__ __forceinline__ int take_highest(unsigned long long& m)
{
    const int j = 63 - __builtin_clzll(m);
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(j));
    return j;
}

// One blend in list order. ok: lanes whose alpha counts; live: lanes whose pixel is still open, which is updated by the
// stop rule. Returns whether this lane blends. (A lane that is not live may set its bit of "stops": it is not live anyway.)
__device__ __forceinline__ bool blend_decision(unsigned long long& live, bool ok, float Tn)
{
    const unsigned long long m = __ballot(ok);
    live &= ~(m & __ballot(Tn < kTStop));
    return __builtin_amdgcn_inverse_ballot_w64(live & m);
}

// Byte offset of a staged record, as a vector value: the address of the visit's LDS reads, and what a lane that blends
// keeps as its last record (turned into a list position once a batch). Scalar multiply, one vector move; left to itself
// the compiler forms the address with a 64-bit vector multiply-add, four times the issue slots.
__device__ __forceinline__ uint32_t staged_offset(uint32_t wave_base, int j, uint32_t stride)
{
    uint32_t off = wave_base + (uint32_t)j * stride;
    asm("" : "+s"(off));
    uint32_t v;
    asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(off));
    return v;
}

}  // namespace pbdr
