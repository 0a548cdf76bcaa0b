// Device helpers shared by the relaxation kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rve_internal.h"
#include "rve_wave.h"

namespace rve {

constexpr int kLawLinear = 0;
constexpr int kMassScaled = 1;
constexpr int kInitWarm = 2;

constexpr int ST_CONVERGED = 0, ST_MAXITER = 1, ST_NONFINITE = 2, ST_BAD_F = 3, ST_STAGNATED = 8;

// Stagnation stop, evaluated at a convergence test that did not converge
// (floor_tol_rel > 0): Rref is the residual of the start, replaced by R
// whenever R falls below half of it, and stall counts the tests since (it
// saturates at stall_checks).  The run stops once stall_checks tests have
// passed without a halving while R and the damping-force norm D are both
// within floor_tol_rel |f_bnd|.
template <typename Args>
__device__ __forceinline__ bool stagnated(const Args& A, double R, double D, double B, double& Rref,
                                          int& stall)
{
    if (!(A.floor_tol_rel > 0.0)) return false;
    if (R < 0.5 * Rref) {
        Rref = R;
        stall = 0;
        return false;
    }
    if (stall < A.stall_checks) ++stall;
    const double ftol = A.floor_tol_rel * B;
    return stall >= A.stall_checks && R <= ftol && D <= ftol;
}

// Whether the convergence test can pass: squares compared first, with a
// margin far above their rounding, so the three dependent FP64 square roots
// are taken only on the last few tests (and on every test of a run with the
// stagnation stop).
template <typename Args>
__device__ __forceinline__ bool test_in_reach(const Args& A, double R2, double B2)
{
    const double lim = fmax(A.tol_abs * A.tol_abs, A.tol_rel * A.tol_rel * B2);
    return A.floor_tol_rel > 0.0 || !(R2 > lim * (1.0 + 1e-9) + 1e-300);
}

// The thread id as a value the compiler cannot see through: indices derived
// from it are recomputed where used instead of being hoisted and kept live.
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Broadcast helpers: values every lane holds identically (read back from LDS
// after a barrier) are moved to scalar registers.
__device__ __forceinline__ double uniform(double x)
{
    int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
    int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float uniform(float x)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}
__device__ __forceinline__ int uniform32(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform64(int64_t x)
{
    const int lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const int hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ inline double det3(const double* F)
{
    return F[0] * (F[4] * F[8] - F[5] * F[7]) - F[1] * (F[3] * F[8] - F[5] * F[6]) +
           F[2] * (F[3] * F[7] - F[4] * F[6]);
}

__device__ __forceinline__ double readlane_d(double x, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
    return __hiloint2double(hi, lo);
}

// Error-free sum of two doubles: s + e == a + b exactly (Knuth's two-sum;
// symmetric in a and b).
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e)
{
    s = a + b;
    const double z = s - a;
    e = (a - (s - z)) + (b - z);
}

// One butterfly stage on (sum, error) pairs.
template <int CTRL>
__device__ __forceinline__ void combine_pairs(double& s, double& c)
{
    const double so = dpp_mov<CTRL>(s), co = dpp_mov<CTRL>(c);
    double t, e;
    two_sum(s, so, t, e);
    s = t;
    c = (c + co) + e;
}

// A kernel's argument struct read through an opaque pointer: what only a rare
// path or one phase needs is loaded there (a scalar load) instead of being held
// in scalar registers, and spilled, across the kernel.
template <typename Args>
using KernArgsT = const __attribute__((address_space(4))) Args;
template <typename Args>
__device__ __forceinline__ KernArgsT<Args>* kernel_args()
{
    auto* p = (KernArgsT<Args>*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

}  // namespace rve
