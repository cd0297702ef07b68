// Reductions over a 64-lane wave without LDS traffic: lane exchanges inside
// rows of 16 by DPP, across rows by the swap instructions of gfx950.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hsim {

// v of the lane given by a DPP control word (every lane has a source).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// op(v, v of the partner group) for groups of 16 (ROW) or 32 lanes whose
// lanes all hold the same value: the swap leaves the even group's value in
// one result and the odd group's in the other, in every lane.
template <int GROUP, typename OP>
__device__ __forceinline__ double swap_op(double v, OP op)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t l = (uint32_t)b, h = (uint32_t)(b >> 32);
    if constexpr (GROUP == 16) {
        const auto sl = __builtin_amdgcn_permlane16_swap(l, l, false, false);
        const auto sh = __builtin_amdgcn_permlane16_swap(h, h, false, false);
        return op(__builtin_bit_cast(double, ((uint64_t)(uint32_t)sh[0] << 32) | (uint32_t)sl[0]),
                  __builtin_bit_cast(double, ((uint64_t)(uint32_t)sh[1] << 32) | (uint32_t)sl[1]));
    } else {
        const auto sl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
        const auto sh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
        return op(__builtin_bit_cast(double, ((uint64_t)(uint32_t)sh[0] << 32) | (uint32_t)sl[0]),
                  __builtin_bit_cast(double, ((uint64_t)(uint32_t)sh[1] << 32) | (uint32_t)sl[1]));
    }
}

// op over groups of 16 lanes; every lane of a group gets the result.
template <typename OP>
__device__ __forceinline__ double row_all(double v, OP op)
{
    v = op(v, dpp_move<0xB1>(v));    // quad_perm [1,0,3,2]
    v = op(v, dpp_move<0x4E>(v));    // quad_perm [2,3,0,1]
    v = op(v, dpp_move<0x141>(v));   // row_half_mirror: the other quad of eight
    return op(v, dpp_move<0x140>(v));// row_mirror: the other eight of sixteen
}

// op over the wave; every lane gets the result.
template <typename OP>
__device__ __forceinline__ double wave_all(double v, OP op)
{
    return swap_op<32>(swap_op<16>(row_all(v, op), op), op);
}

// op over the 16 lanes with the same lane number modulo 4; each gets the
// result.
template <typename OP>
__device__ __forceinline__ double quarter_all(double v, OP op)
{
    v = op(v, dpp_move<0x124>(v));   // row_ror:4
    v = op(v, dpp_move<0x128>(v));   // row_ror:8
    return swap_op<32>(swap_op<16>(v, op), op);
}

struct OpAdd {
    __device__ __forceinline__ double operator()(double a, double b) const { return a + b; }
};
struct OpMax {
    __device__ __forceinline__ double operator()(double a, double b) const { return fmax(a, b); }
};

}  // namespace hsim
