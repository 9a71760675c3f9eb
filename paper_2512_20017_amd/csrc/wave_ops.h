// Scans and reductions over a wavefront.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbdr {

// Reductions and scans over a wavefront with DPP moves (an exchange through the LDS crossbar, what a shuffle is, has ten times
// their latency, and these stand in a row). kOp(a, b); 0 is the neutral element.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_or0(uint32_t v)      // lanes without a source read 0
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRows, 0xf, true);
}
template <class Op>
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, Op op)
{
    v = op(v, dpp_or0<0x111, 0xf>(v));      // row_shr:1
    v = op(v, dpp_or0<0x112, 0xf>(v));      // row_shr:2
    v = op(v, dpp_or0<0x114, 0xf>(v));      // row_shr:4
    v = op(v, dpp_or0<0x118, 0xf>(v));      // row_shr:8
    v = op(v, dpp_or0<0x142, 0xa>(v));      // row_bcast:15 into rows 1 and 3
    v = op(v, dpp_or0<0x143, 0xc>(v));      // row_bcast:31 into rows 2 and 3
    return v;
}
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, Op op)      // uniform
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(v, op), 63);
}
struct OpAdd { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };

}  // namespace pbdr
