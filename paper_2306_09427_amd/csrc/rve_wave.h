// Cross-lane reductions of a 64-lane wavefront (device code, gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace rve {

// Cross-lane moves on the vector ALU.  The partner of a butterfly stage is
// fetched by a lane swap (stages 32 and 16) or a DPP move (8, 4, 2, 1) instead
// of ds_bpermute, whose LDS round trip a sum of six dependent stages pays six
// times.  Stages run from 32 down to 1, so before stage 4 the values of a row
// of 16 lanes repeat with period 8 and a rotation by 4 fetches lane i ^ 4; the
// additions are those of a __shfl_xor butterfly, bit for bit.
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppRor4 = 0x124, kDppRor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ unsigned dpp_mov(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v)
{
    return __hiloint2double((int)dpp_mov<CTRL>((unsigned)__double2hiint(v)),
                            (int)dpp_mov<CTRL>((unsigned)__double2loint(v)));
}
// v(i) + v(i ^ 32) and v(i) + v(i ^ 16) in every lane
__device__ __forceinline__ double add_xor32(double v)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double add_xor16(double v)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// a(i) + a(i ^ 32) in the lanes below 32, b(i) + b(i ^ 32) in those above
__device__ __forceinline__ double halves_xor32(double a, double b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = add_xor32(v);
    v = add_xor16(v);
    v += dpp_mov<kDppRor8>(v);
    v += dpp_mov<kDppRor4>(v);
    v += dpp_mov<kDppXor2>(v);
    v += dpp_mov<kDppXor1>(v);
    return v;
}

// Maximum over the 64 lanes of a non-negative number (bit patterns of
// non-negative numbers order like unsigned integers), by DPP butterflies
// inside each row of 16 lanes and row broadcasts across rows: complete in
// lane 63 (wave_max_lane63), or from there in a scalar register.  Lanes a move does not reach read
// zero, the identity, so every step is one v_max_u32 with a DPP operand.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_max_step(unsigned v)
{
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
    return o > v ? o : v;
}
__device__ __forceinline__ float wave_max_lane63(float x)
{
    unsigned v = __float_as_uint(x);
    v = dpp_max_step<kDppXor1, 0xf>(v);
    v = dpp_max_step<kDppXor2, 0xf>(v);
    v = dpp_max_step<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_max_step<0x140, 0xf>(v);   // row_mirror
    v = dpp_max_step<0x142, 0xa>(v);   // row_bcast:15
    v = dpp_max_step<0x143, 0xc>(v);   // row_bcast:31
    return __uint_as_float(v);
}
__device__ __forceinline__ float wave_max_nonneg(float x)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wave_max_lane63(x)), 63));
}
__device__ __forceinline__ double wave_max(double v)
{
    v = fmax(v, dpp_mov<kDppXor1>(v));
    v = fmax(v, dpp_mov<kDppXor2>(v));
    v = fmax(v, dpp_mov<0x141>(v));    // row_half_mirror
    v = fmax(v, dpp_mov<0x140>(v));    // row_mirror
    const auto l16 = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h16 = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = fmax(__hiloint2double((int)h16[0], (int)l16[0]), __hiloint2double((int)h16[1], (int)l16[1]));
    const auto l32 = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h32 = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    return fmax(__hiloint2double((int)h32[0], (int)l32[0]), __hiloint2double((int)h32[1], (int)l32[1]));
}
__device__ __forceinline__ double wave_max_lane63(double v) { return wave_max(v); }

}  // namespace rve
