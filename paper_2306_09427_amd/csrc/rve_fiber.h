// FP32 fiber law in the scaled form, shared by the register-resident and the
// spread relaxation kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace rve {

// One fiber evaluated at u = dh / L0: e = D + u (the current vector over L0),
// g = T L0 / l, so that the force on end j is g e, and b = max(k_t, |g|), so
// that its Gershgorin term is b / L0.
struct FiberState {
    float ex, ey, ez, g, b;
};

// One v_max_f32 each: fmax would quiet its operands first.
__device__ __forceinline__ float max0(float x)
{
    float y;
    asm("v_max_f32 %0, 0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ __forceinline__ float max_abs(float a, float b)   // max(a, |b|)
{
    float y;
    asm("v_max_f32 %0, %1, |%2|" : "=v"(y) : "v"(a), "v"(b));
    return y;
}

// Hardware reciprocal square root, reciprocal and exp2 (about 1 ulp each).
// Every rounding is spelled out (products contracted where an fma stands,
// nowhere else), so the kernels agree bit for bit whatever the surrounding
// code.  Compression needs no second branch for k_t: the clamped argument
// gives T_e = 0 and k_t = EA.
__device__ __forceinline__ FiberState fiber_state(bool linear, float EA, float B, float EAoB, float Dx, float Dy,
                                                  float Dz, float Qn, float iL, float dhx, float dhy, float dhz)
{
#pragma clang fp contract(off)
    const float ux = iL * dhx, uy = iL * dhy, uz = iL * dhz;
    const float du = fmaf(Dz, uz, fmaf(Dx, ux, Dy * uy));
    const float uu = fmaf(uz, uz, fmaf(ux, ux, uy * uy));
    const float qn = Qn + fmaf(2.f, du, uu);
    const float m = 1.f + qn;
    const float rs = __builtin_amdgcn_rsqf(m);
    const float eps = qn * __builtin_amdgcn_rcpf(fmaf(m, rs, 1.f));
    float T = EA * eps, kt = EA;
    if (!linear) {
        // e^x - 1 for x >= 0: below 1/4 the Taylor series to x^6 (truncation
        // under half an ulp), above it the hardware exp2 minus one
        const float x = B * max0(eps);
        float t = fmaf(x, 1.f / 720.f, 1.f / 120.f);
        t = fmaf(x, t, 1.f / 24.f);
        t = fmaf(x, t, 1.f / 6.f);
        t = fmaf(x, t, 0.5f);
        t = fmaf(x, t, 1.f);
        // (both, and one select: a ballot around the exp2, which the compiler
        // turned into two selects, took 261 instead of 259 ms on 4096 RVEs of 200
        // to 400 seeds and 96 instead of 94 on 64 of 2000; a real branch 259 to
        // 265 and 97: most waves hold a fiber beyond 1/4)
        const float big = __builtin_amdgcn_exp2f(x * 1.44269504088896341f) - 1.f;
        const float em1 = x < 0.25f ? x * t : big;
        const float Te = EAoB * em1;
        kt = fmaf(B, Te, EA);
        T = eps >= 0.f ? Te : T;
    }
    const float g = T * rs;
    return {Dx + ux, Dy + uy, Dz + uz, g, max_abs(kt, g)};
}

}  // namespace rve
