// Register-resident relaxation kernels for gfx950 (MI355X): one workgroup
// relaxes one RVE, its fibers and free nodes dealt round-robin to the threads
// and kept in VGPRs for the whole solve; LDS holds the positions, the fiber
// forces and two small tables, all at compile-time offsets (ResLayout).
//
// What bounds it.  With two or more RVEs on a CU the FP32 builds issue a VALU
// instruction in nearly every cycle, so the instructions per fiber and node
// are the time; with one RVE on a CU an iteration is a chain of LDS round
// trips, dependent arithmetic and three barriers.  Both ask for the same:
//   - no exec masks: lanes past the last fiber or node hold neutral slots
//     (1/L0 = 0, no incidence) whose force and motion are zero, and a wave
//     skips a slot only when it holds no fiber or node of the RVE at all;
//   - no address arithmetic: fiber ends and incidences are stored as LDS byte
//     offsets, two per register, and the array bases are instruction offsets;
//   - nothing read from global memory inside the loop: the incidences beyond
//     a node's four register-held ones, and the fibers at the boundary nodes,
//     are 16-bit tables in LDS (a dependent pair of global loads in every
//     iteration, and three more on a test, took a third of a small RVE's time);
//   - each node's position and inverse mass in its thread's registers, the LDS
//     copy being written only for the others;
//   - one LDS round trip for the time-step maximum (per-wave slots read back
//     by the lanes of a row and combined by DPP).
// Measured, us per iteration (convergence test every 8), against the kernel
// before, which kept the node's position and inverse mass in LDS, masked every
// slot and read the rest of the incidences from global memory: one RVE of 60
// seeds 1.60 -> 1.17, of 300 seeds 3.08 -> 2.25, of 400 seeds 3.35 -> 2.74; 1024
// RVEs of 300 seeds (two per CU) 8.2 -> 7.0.  FP64: 60 seeds 2.34 -> 1.73, 300 seeds
// 5.74 -> 4.60, 400 seeds (until then beyond the FP64 builds) 20.3 -> 6.2.  A test in
// every iteration costs 0.8 more at 100 seeds in FP64 (2.30 -> 3.07; linear law 1.99
// -> 2.76): the norms with a division per node, three wave sums, four dependent
// two-sums and the boundary loop.  Counters of 2048 RVEs of 300 seeds, two per CU:
// 472 VALU instructions per wave and iteration, in 0.95 of the busy cycles, LDS
// busy 0.72 of the time, 0.45 of that in bank conflicts.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "rve_fiber.h"
#include "rve_internal.h"
#include "rve_relax.h"
#include "rve_wave.h"

namespace rve {

namespace {

typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ fiber law
// Force on end j and Gershgorin term of one fiber in the scaled form
// (fiber_eval_scaled in rve_kernels.hip): u = dh / L0,
// qn = (l^2 - L0^2) / L0^2 = Qn + 2 D.u + u.u, l / L0 = sqrt(1 + qn),
// eps = qn / (1 + l/L0), force = (T L0 / l) (D + u).
// A neutral slot (iL = Qn = 0) gives exact zeros.
template <typename Real>
struct Fiber {
    Real x, y, z, b;
};

__device__ __forceinline__ Fiber<float> fiber_force(bool linear, float EA, float B, float EAoB, float Dx, float Dy,
                                                    float Dz, float Qn, float iL, float dhx, float dhy, float dhz)
{
#pragma clang fp contract(off)
    const FiberState f = fiber_state(linear, EA, B, EAoB, Dx, Dy, Dz, Qn, iL, dhx, dhy, dhz);
    return {f.g * f.ex, f.g * f.ey, f.g * f.ez, iL * f.b};
}

// FP64: the same chain with the library's sqrt, division and expm1 replaced
// by branch-free sequences of about their accuracy (1 ulp against at most 1):
// sqrt and 1/sqrt by Goldschmidt's coupled iteration from the hardware
// estimate with a residual correction each, the quotient by Newton's
// reciprocal with a residual correction, e^x - 1 by the Taylor series of the
// argument reduced by a multiple of ln 2 (Cody and Waite's two-part ln 2).
// x >= 0; beyond the largest double the result is infinite, as the library's:
// the scale 2^k is applied as 2 * 2^(k - 1), which stays finite up to the
// argument 710, where larger ones are cut (e^710 overflows).
__device__ __forceinline__ double exp_minus_one(double x)
{
    x = fmin(x, 710.0);
    const double k = __builtin_rint(x * 1.4426950408889634);
    const double r = fma(-k, 1.90821492927058770002e-10, fma(-k, 6.93147180369123816490e-01, x));
    double p = 1.0 / 87178291200.0;   // 1/14!
    p = fma(p, r, 1.0 / 6227020800.0);
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p * r, r, r);
    const double s = __builtin_amdgcn_ldexp(0.5, (int)k);
    return 2.0 * fma(s, p, s - 0.5);
}
__device__ __forceinline__ Fiber<double> fiber_force(bool linear, double EA, double B, double EAoB, double Dx,
                                                     double Dy, double Dz, double Qn, double iL, double dhx,
                                                     double dhy, double dhz)
{
    const double ux = iL * dhx, uy = iL * dhy, uz = iL * dhz;
    const double qn = Qn + (2.0 * (Dx * ux + Dy * uy + Dz * uz) + (ux * ux + uy * uy + uz * uz));
    const double m = 1.0 + qn;
    const double y = __builtin_amdgcn_rsq(m);
    double s = m * y, h = 0.5 * y;
    const double e0 = fma(-h, s, 0.5);
    s = fma(s, e0, s);
    h = fma(h, e0, h);
    s = fma(fma(-s, s, m), h, s);        // l / L0
    double rs = h + h;
    rs = fma(fma(-s, rs, 1.0), rs, rs);  // L0 / l
    const double t = s + 1.0;
    double yt = __builtin_amdgcn_rcp(t);
    yt = fma(fma(-t, yt, 1.0), yt, yt);
    double eps = qn * yt;
    eps = fma(fma(-t, eps, qn), yt, eps);
    double T = EA * eps, kt = EA;
    if (!linear) {
        const double Te = EAoB * exp_minus_one(B * fmax(eps, 0.0));
        kt = fma(B, Te, EA);
        T = eps >= 0.0 ? Te : T;
    }
    const double g = T * rs;
    return {g * (Dx + ux), g * (Dy + uy), g * (Dz + uz), iL * fmax(kt, fabs(g))};
}

__device__ __forceinline__ float signed_one(uint32_t sign, float) { return __uint_as_float(sign | 0x3f800000u); }
__device__ __forceinline__ double signed_one(uint32_t sign, double) { return __hiloint2double((int)(sign | 0x3ff00000u), 0); }
__device__ __forceinline__ float fma_r(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float rcp_r(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_r(double x) { return 1.0 / x; }

// ------------------------------------------------------------------ LDS access
// Byte offsets `o` are chip_ends / chip_offset values (multiples of the unit).
template <typename Real, int T, int SF, int SN>
struct Chip {
    static constexpr bool F64 = sizeof(Real) == 8;
    static constexpr ResLayout L = res_layout(F64, T, SF, SN);
    static constexpr int FV0 = res_pos_bytes(F64, L), ARR = res_arr_bytes(F64, L);
    static constexpr int BCAP = res_bcap(T), XCAP = res_xcap(T);
    static constexpr int BYTES = ARR + 2 * (BCAP + XCAP);
    static constexpr int PS = 8 * (L.NP + 1), FS = 8 * L.NF;   // FP64 component strides

    static __device__ __forceinline__ void get_h(const char* S, uint32_t o, Real& x, Real& y, Real& z)
    {
        if constexpr (F64) {
            x = *(const double*)(S + o);
            y = *(const double*)(S + PS + o);
            z = *(const double*)(S + 2 * PS + o);
        } else {
            const f32x3 v = *(const f32x3*)(S + o);
            x = v.x; y = v.y; z = v.z;
        }
    }
    static __device__ __forceinline__ void put_h(char* S, uint32_t o, Real x, Real y, Real z)
    {
        if constexpr (F64) {
            *(double*)(S + o) = x;
            *(double*)(S + PS + o) = y;
            *(double*)(S + 2 * PS + o) = z;
        } else {
            *(f32x3*)(S + o) = f32x3{x, y, z};
        }
    }
    static __device__ __forceinline__ void put_f(char* S, uint32_t o, const Fiber<Real>& f)
    {
        if constexpr (F64) {
            *(double*)(S + FV0 + o) = f.x;
            *(double*)(S + FV0 + FS + o) = f.y;
            *(double*)(S + FV0 + 2 * FS + o) = f.z;
            *(float*)(S + FV0 + 3 * FS + (o >> 1)) = (float)f.b;
        } else {
            *(f32x4*)(S + FV0 + o) = f32x4{f.x, f.y, f.z, f.b};
        }
    }
    static __device__ __forceinline__ Fiber<Real> get_f(const char* S, uint32_t o)
    {
        if constexpr (F64) {
            return {*(const double*)(S + FV0 + o), *(const double*)(S + FV0 + FS + o),
                    *(const double*)(S + FV0 + 2 * FS + o), (double)*(const float*)(S + FV0 + 3 * FS + (o >> 1))};
        } else {
            const f32x4 v = *(const f32x4*)(S + FV0 + o);
            return {v.x, v.y, v.z, v.w};
        }
    }
    static __device__ __forceinline__ uint16_t* bcodes(char* S) { return (uint16_t*)(S + ARR); }
    static __device__ __forceinline__ uint2* xcodes(char* S) { return (uint2*)((uint16_t*)(S + ARR) + BCAP); }
};

// Reduction slots: per-wave partial sums of |f_free|^2, |c M v|^2, |f_bnd|^2
// and the kinetic energy, and the per-wave time-step maxima (alternating).
template <typename Real>
struct ChipRed {
    double v[4][16];
    Real g[2][16];
    int task, x4, xd;
};

__device__ __forceinline__ float row_max(float x)
{
    unsigned v = __float_as_uint(x);
    v = dpp_max_step<kDppXor1, 0xf>(v);
    v = dpp_max_step<kDppXor2, 0xf>(v);
    v = dpp_max_step<0x141, 0xf>(v);
    v = dpp_max_step<0x140, 0xf>(v);
    return __uint_as_float(__builtin_amdgcn_readfirstlane(v));
}
__device__ __forceinline__ double row_max(double v)
{
    v = fmax(v, dpp_mov<kDppXor1>(v));
    v = fmax(v, dpp_mov<kDppXor2>(v));
    v = fmax(v, dpp_mov<0x141>(v));
    return uniform(fmax(v, dpp_mov<0x140>(v)));
}

typedef KernArgsT<SolveArgs> KernArgs;

// fn(0), fn(1), ... while slot s of this wave holds an element (the slots a wave
// uses are a prefix).  Nested, so a wave leaves the unused ones by one branch.
template <int T, int N, int S0 = 0, typename Fn>
__device__ __forceinline__ void each_slot(int wave64, int count, Fn&& fn)
{
    if constexpr (S0 < N) {
        if (S0 * T + wave64 < count) {
            fn(std::integral_constant<int, S0>{});
            __builtin_amdgcn_sched_barrier(0);
            each_slot<T, N, S0 + 1>(wave64, count, fn);
        }
    }
}

// ------------------------------------------------------------------ one RVE
// Fiber k lives in slot k / T of thread k % T, free node a in slot a / T of
// thread a % T (replayed on the host by rve_check_indexing).
template <typename Real, int T, int SF, int SN, bool KIN>
__device__ __forceinline__ void chip_solve(KernArgs& A, int r, char* S, ChipRed<Real>& red)
{
    using C = Chip<Real, T, SF, SN>;
    constexpr bool F64 = C::F64;
    constexpr ResLayout L = C::L;
    constexpr int NW = T / 64;
    constexpr uint32_t ZH = (uint32_t)(L.NP * L.unit);   // zero position slot
    // incidences gathered per batch of LDS reads, and fiber slots whose chains
    // are interleaved (as the register budget allows)
    constexpr int GB = F64 && SN > 3 ? 1 : (F64 || SF + SN > 6 ? 2 : kResIncRegs);
    // positions in registers, except where that exceeds the register budget
    constexpr bool HREG = F64 ? SN < 4 : !(KIN && SN > 2);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave64 = uniform32(tid & ~63);
    auto& net = A.net;
    const int64_t f0 = uniform64(net.fib_off[r]), a0 = uniform64(net.free_off[r]), b0 = uniform64(net.bnd_off[r]);
    const int nfib = uniform32((int)(net.fib_off[r + 1] - f0));
    const int nf = uniform32((int)(net.free_off[r + 1] - a0));
    const int nb = uniform32((int)(net.bnd_off[r + 1] - b0));
    const int64_t* incoffb = net.inc_off + a0;
    const uint32_t zk = (uint32_t)nfib;   // zero force slot

    double F[9];
    bool finite = true;
    for (int k = 0; k < 9; ++k) {
        F[k] = A.F[9 * r + k];
        finite = finite && isfinite(F[k]);
    }
    const double J = det3(F);
    if (!finite || !(J > 0.0)) {
        if (tid == 0) {
            int64_t zero = 0;   // opaque, as the NaN: not held across RVEs
            double nanv = NAN;
            asm volatile("" : "+v"(zero), "+v"(nanv));
            A.status[r] = ST_BAD_F;
            A.iters[r] = zero;
            A.Rres[r] = nanv; A.Dres[r] = nanv; A.Bres[r] = nanv;
            for (int k = 0; k < 9; ++k) A.sigma[9 * r + k] = nanv;
        }
        return;
    }
    const bool linear = A.law == kLawLinear;
    const Real EA = uniform((Real)A.EA), Bc = uniform((Real)A.B), EAoB = uniform((Real)(A.EA / A.B));
    // kinetic damping: no viscous force (c = 0); velocities are zeroed at
    // kinetic-energy peaks below
    const double cr = uniform(A.c[r]);
    const Real c = KIN ? Real(0) : uniform((Real)cr);
    const Real cg = uniform((Real)cr);   // scale of the damping-force test

    if (tid == 0) {
        red.x4 = nf;
        red.xd = kResIncRegs;
    }
    __syncthreads();
    // ---- fibers into registers
    Real Dx[SF], Dy[SF], Dz[SF], Qn[SF], iL[SF];
    uint32_t E[SF];
#pragma unroll
    for (int s = 0; s < SF; ++s) {
        const int k = s * T + tid;
        Dx[s] = Dy[s] = Dz[s] = Qn[s] = iL[s] = Real(0);
        E[s] = ZH | ZH << 16;
        if (k < nfib) {
            const double* d0 = net.d0 + 3 * (f0 + k);
            const double L0 = net.L0[f0 + k], il = 1.0 / L0;
            const double Dxd = F[0] * d0[0] + F[1] * d0[1] + F[2] * d0[2];
            const double Dyd = F[3] * d0[0] + F[4] * d0[1] + F[5] * d0[2];
            const double Dzd = F[6] * d0[0] + F[7] * d0[1] + F[8] * d0[2];
            Dx[s] = (Real)(Dxd * il); Dy[s] = (Real)(Dyd * il); Dz[s] = (Real)(Dzd * il);
            Qn[s] = (Real)((((Dxd * Dxd + Dyd * Dyd + Dzd * Dzd) - L0 * L0) * il) * il);
            iL[s] = (Real)il;
            E[s] = chip_ends(net.ends[f0 + k], (uint32_t)nf, L);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // ---- free nodes: velocity, acceleration, position, inverse mass and the
    // first four incidences in registers
    Real vx[SN], vy[SN], vz[SN], ax[SN], ay[SN], az[SN], im[SN];
    Real hx[HREG ? SN : 1], hy[HREG ? SN : 1], hz[HREG ? SN : 1];
    uint32_t inc[SN][kResIncRegs / 2];
    int degw[SN];   // largest degree in this wave's node slot (scalar)
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        const int a = s * T + tid;
        vx[s] = vy[s] = vz[s] = ax[s] = ay[s] = az[s] = im[s] = Real(0);
        Real x = Real(0), y = Real(0), z = Real(0);
        int deg = 0;
        uint32_t k[kResIncRegs], neg[kResIncRegs];
#pragma unroll
        for (int q = 0; q < kResIncRegs; ++q) {
            k[q] = zk;
            neg[q] = 0;
        }
        if (a < nf) {
            im[s] = (Real)(1.0 / (net.mass[a0 + a] * A.rhoA));
            const int64_t e0 = incoffb[a];
            deg = (int)(incoffb[a + 1] - e0);
#pragma unroll
            for (int q = 0; q < kResIncRegs; ++q)
                if (q < deg) {
                    const uint32_t w = net.inc[e0 + q];
                    k[q] = w & 0x7fffffffu;
                    neg[q] = w >> 31;
                }
            if (A.init == kInitWarm) {
                const double* h = A.h_state + 3 * (a0 + a);
                x = (Real)h[0]; y = (Real)h[1]; z = (Real)h[2];
            }
            if (deg > kResIncRegs) {
                atomicMin(&red.x4, a);
                atomicMax(&red.xd, deg);
            }
        }
#pragma unroll
        for (int q = 0; q < kResIncRegs / 2; ++q)
            inc[s][q] = chip_codes(k[2 * q], neg[2 * q], k[2 * q + 1], neg[2 * q + 1], L);
        if constexpr (HREG) {
            hx[s] = x; hy[s] = y; hz[s] = z;
        }
        if (a < L.NP) C::put_h(S, (uint32_t)(a * L.unit), x, y, z);
        degw[s] = uniform32((int)__float_as_uint(wave_max_nonneg(__uint_as_float((unsigned)deg))));
        __builtin_amdgcn_sched_barrier(0);
    }
    // an opaque zero: no zero vector is held in registers across RVEs for it
    Real z0 = Real(0);
    asm volatile("" : "+v"(z0));
    if (tid < 32) (&red.g[0][0])[tid] = z0;
    if (tid == 0) {
        C::put_h(S, ZH, z0, z0, z0);
        C::put_f(S, zk * (uint32_t)L.unit, Fiber<Real>{z0, z0, z0, z0});
    }
    __syncthreads();
    // ---- tables: the incidences beyond the first four of the nodes x4 .. nf
    // (the packing puts the nodes of degree above 4 last), four per 8-byte
    // word, row j of the words for incidences 4 + 4 j ..; and the fiber of every
    // boundary node of degree 1 (0xffff: the node's incidence list is read
    // from global memory)
    const int x4 = uniform32(red.x4), nx = nf - x4;
    const int xrows = (uniform32(red.xd) - 1) / 4;   // rows of words
    const bool xtab = 4 * xrows * nx <= C::XCAP, btab = nb <= C::BCAP;
    if (xtab) {
        for (int e = tid; e < xrows * nx; e += T) {
            const int j = e / nx, a = x4 + (e - j * nx);
            const int64_t e0 = incoffb[a] + kResIncRegs + 4 * j, e1 = incoffb[a + 1];
            uint32_t k[4], neg[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t w = e0 + q < e1 ? net.inc[e0 + q] : zk;
                k[q] = w & 0x7fffffffu;
                neg[q] = w >> 31;
            }
            C::xcodes(S)[e] = make_uint2(chip_codes(k[0], neg[0], k[1], neg[1], L), chip_codes(k[2], neg[2], k[3], neg[3], L));
        }
    }
    if (btab) {
        for (int q = tid; q < nb; q += T) {
            const int64_t e = net.binc_off[b0 + q];
            C::bcodes(S)[q] = net.binc_off[b0 + q + 1] - e == 1 ? (uint16_t)(net.binc[e] & 0x7fffffffu) : (uint16_t)0xffffu;
        }
    }
    __syncthreads();

    auto fiber_one = [&](int s, int t) __attribute__((always_inline)) {
        Real ix, iy, iz, jx, jy, jz;
        C::get_h(S, E[s] & 0xffffu, ix, iy, iz);
        C::get_h(S, E[s] >> 16, jx, jy, jz);
        C::put_f(S, (uint32_t)((s * T + t) * L.unit),
                 fiber_force(linear, EA, Bc, EAoB, Dx[s], Dy[s], Dz[s], Qn[s], iL[s], jx - ix, jy - iy, jz - iz));
    };
    auto fiber_pass = [&](int t) __attribute__((always_inline)) {
        each_slot<T, SF>(wave64, nfib, [&](auto s) __attribute__((always_inline)) { fiber_one(s, t); });
    };
    // internal force and Gershgorin sum of the node in slot s
    auto gather = [&](int s, int t, Real& fx, Real& fy, Real& fz, Real& G) __attribute__((always_inline)) {
        fx = fy = fz = G = Real(0);
        auto add = [&](const Fiber<Real>& f, uint32_t sign) __attribute__((always_inline)) {
            const Real sg = signed_one(sign, Real(0));
            fx = fma_r(sg, f.x, fx); fy = fma_r(sg, f.y, fy); fz = fma_r(sg, f.z, fz);
            G += f.b;
        };
        // four incidences of two words, GB at a time
        auto add4 = [&](uint32_t w0, uint32_t w1) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 4; h += GB) {
                Fiber<Real> f[GB];
#pragma unroll
                for (int u = 0; u < GB; ++u) f[u] = C::get_f(S, chip_offset(h + u < 2 ? w0 : w1, (h + u) & 1, L));
#pragma unroll
                for (int u = 0; u < GB; ++u) add(f[u], chip_sign(h + u < 2 ? w0 : w1, (h + u) & 1, L));
            }
        };
        const bool more = degw[s] > kResIncRegs;   // wave-uniform
        const int a = s * T + t, i = a - x4;
        const bool mine = i >= 0 && a < nf;
        const uint32_t zz = chip_codes(zk, 0, zk, 0, L);
        uint2 xw = make_uint2(zz, zz);
        if (more && xtab && mine) xw = C::xcodes(S)[i];   // in flight during the first four
        add4(inc[s][0], inc[s][1]);
        if (more) {
            if (xtab) {
                add4(xw.x, xw.y);
#pragma unroll 1
                for (int j = 1; 4 * j + kResIncRegs < degw[s]; ++j)
                    if (mine) {
                        const uint2 w = C::xcodes(S)[j * nx + i];
                        add4(w.x, w.y);
                    }
            } else if (mine) {
                KernArgs* K = kernel_args<SolveArgs>();
                const int64_t* io = K->net.inc_off + K->net.free_off[r] + a;
                const int64_t e1 = io[1];
#pragma unroll 1
                for (int64_t e = io[0] + kResIncRegs; e < e1; ++e) {
                    const uint32_t w = K->net.inc[e];
                    add(C::get_f(S, (w & 0x7fffffffu) * (uint32_t)L.unit), w & 0x80000000u);
                }
            }
        }
        G += G;
    };
    // boundary reaction norm^2 partial of this thread (test iterations only)
    auto boundary_norm2 = [&](int t) __attribute__((always_inline)) -> double {
        double acc = 0.0;
#pragma unroll 1
        for (int q = t; q < nb; q += T) {
            const uint32_t k = btab ? (uint32_t)C::bcodes(S)[q] : 0xffffu;
            double x = 0.0, y = 0.0, z = 0.0;
            if (k != 0xffffu) {
                const Fiber<Real> f = C::get_f(S, k * (uint32_t)L.unit);
                x = (double)f.x; y = (double)f.y; z = (double)f.z;
            } else {
                KernArgs* K = kernel_args<SolveArgs>();
                const int64_t* bo = K->net.binc_off + K->net.bnd_off[r] + q;
                const int64_t e1 = bo[1];
#pragma unroll 1
                for (int64_t e = bo[0]; e < e1; ++e) {
                    const uint32_t w = K->net.binc[e];
                    const Fiber<Real> f = C::get_f(S, (w & 0x7fffffffu) * (uint32_t)L.unit);
                    const double sg = (w >> 31) ? -1.0 : 1.0;
                    x += sg * (double)f.x; y += sg * (double)f.y; z += sg * (double)f.z;
                }
            }
            acc += x * x + y * y + z * z;
        }
        return acc;
    };
    // Workgroup maximum of g (>= 0) every call, the three norms when `full`,
    // the kinetic energy in the kinetic builds.  One barrier.  The maxima
    // alternate with `parity`; the sums are read at least two barriers before
    // they are written again.  Sums: pairwise in a wave, then over the waves
    // with an exact two-sum (row p of a wave combines quantity p), so every
    // wave ends with the same totals.
    auto reduce = [&](int t, int parity, Real g, double r2, double d2, double b2, double ke, bool full, Real& gmax,
                      double& R2, double& D2, double& B2, double& KE) __attribute__((always_inline)) {
        const int lane = t & 63, wave = t >> 6;
        g = wave_max_lane63(g);
        if (lane == 63) red.g[parity][wave] = g;
        if constexpr (KIN) ke = wave_sum(ke);
        if (full) {
            r2 = wave_sum(r2);
            d2 = wave_sum(d2);
            b2 = wave_sum(b2);
        }
        if ((full || KIN) && lane == 0) {
            if constexpr (KIN) red.v[3][wave] = ke;
            if (full) {
                red.v[0][wave] = r2;
                red.v[1][wave] = d2;
                red.v[2][wave] = b2;
            }
        }
        __syncthreads();
        gmax = row_max(red.g[parity][lane & 15]);
        if (full || KIN) {
            const int p = lane >> 4, w = lane & 15;
            const bool use = w < NW && (p == 3 ? KIN : full);
            double s = use ? red.v[p][w] : 0.0, e = 0.0;
            combine_pairs<kDppRor8>(s, e);
            combine_pairs<kDppRor4>(s, e);
            combine_pairs<kDppXor2>(s, e);
            combine_pairs<kDppXor1>(s, e);
            const double tot = s + e;
            if (full) {
                R2 = readlane_d(tot, 0);
                D2 = readlane_d(tot, 16);
                B2 = readlane_d(tot, 32);
            }
            if constexpr (KIN) KE = readlane_d(tot, 48);
        }
    };

    // ---- initial force, residual and (optionally) stiffness-scaled mass
    fiber_pass(tid);
    __syncthreads();
    Real gpart = Real(0);
    double r2p = 0.0;
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        if (s * T + wave64 < nf) {
            const int a = s * T + tid;
            Real fx, fy, fz, G;
            gather(s, tid, fx, fy, fz, G);
            if (A.mass_mode == kMassScaled && a < nf) im[s] = G > Real(0) ? Real(4) / G : Real(1);
            ax[s] = -fx * im[s];
            ay[s] = -fy * im[s];
            az[s] = -fz * im[s];
            gpart = fmax(gpart, G * im[s]);
            r2p += (double)fx * fx + (double)fy * fy + (double)fz * fz;
        }
    }
    Real gmax;
    double R2 = 0.0, D2 = 0.0, B2 = 0.0, ke = 0.0;
    int parity = 0;
    reduce(tid, parity, gpart, r2p, 0.0, boundary_norm2(tid), 0.0, true, gmax, R2, D2, B2, ke);

    int64_t n = 0;
    int status = ST_CONVERGED;
    const int ce = A.check_every > 0 ? A.check_every : 1;
    bool done = sqrt(R2) <= fmax(A.tol_abs, A.tol_rel * sqrt(B2));   // v = 0: damping norm is 0
    double Rref = uniform(sqrt(R2));   // stagnation stop: reference residual
    int stall = 0;                     // stagnation stop: tests since R last halved
    if (!isfinite(R2)) {
        status = ST_NONFINITE;
        done = true;
    }
    if (!done && n >= A.n_max) {
        status = ST_MAXITER;
        done = true;
    }
    // iterations to the next event: a convergence test, or n_max
    int cd = uniform32((int)(A.n_max < ce ? A.n_max : ce));
    bool ev_test = cd == ce;
    const Real two_alpha = uniform((Real)(2.0 * A.alpha));
    double ke_prev = 0.0;   // kinetic damping: kinetic energy at the previous full step
    int evn = cd;           // iterations of the current stretch

    while (!done) {
        int t = tid;
        asm volatile("" : "+v"(t));
        // Keep the packed fiber ends and incidences packed: without this the
        // compiler unpacks them before the loop, which doubles the registers
        // they occupy.
#pragma unroll
        for (int s = 0; s < SF; ++s) asm volatile("" : "+v"(E[s]));
#pragma unroll
        for (int s = 0; s < SN; ++s) {
#pragma unroll
            for (int q = 0; q < kResIncRegs / 2; ++q) asm volatile("" : "+v"(inc[s][q]));
        }
        // half-step velocity and position update with the time step of this
        // state (FP32: hardware rsqrt; the state it advances is FP32 anyway)
        Real rdt;
        if constexpr (F64)
            rdt = uniform(two_alpha / sqrt(gmax));
        else
            rdt = uniform(two_alpha * __builtin_amdgcn_rsqf(gmax));
        const Real hdt = Real(0.5) * rdt;
        each_slot<T, SN>(wave64, nf, [&](auto s) __attribute__((always_inline)) {
            const uint32_t o = (uint32_t)((s * T + t) * L.unit);
            vx[s] = fma_r(ax[s], hdt, vx[s]); vy[s] = fma_r(ay[s], hdt, vy[s]); vz[s] = fma_r(az[s], hdt, vz[s]);
            if constexpr (HREG) {
                hx[s] = fma_r(vx[s], rdt, hx[s]); hy[s] = fma_r(vy[s], rdt, hy[s]); hz[s] = fma_r(vz[s], rdt, hz[s]);
                C::put_h(S, o, hx[s], hy[s], hz[s]);
            } else {
                Real x, y, z;
                C::get_h(S, o, x, y, z);
                C::put_h(S, o, fma_r(vx[s], rdt, x), fma_r(vy[s], rdt, y), fma_r(vz[s], rdt, z));
            }
        });
        __syncthreads();
        fiber_pass(t);
        __syncthreads();
        --cd;
        const bool check = cd == 0 && ev_test;
        gpart = Real(0);
        r2p = 0.0;
        double d2p = 0.0, b2p = 0.0, kep = 0.0;
        each_slot<T, SN>(wave64, nf, [&](auto s) __attribute__((always_inline)) {
            Real fx, fy, fz, G;
            gather(s, t, fx, fy, fz, G);
            // damped acceleration with the half-step velocity, then second half step
            ax[s] = fma_r(im[s], -fx, -(c * vx[s]));
            ay[s] = fma_r(im[s], -fy, -(c * vy[s]));
            az[s] = fma_r(im[s], -fz, -(c * vz[s]));
            vx[s] = fma_r(ax[s], hdt, vx[s]); vy[s] = fma_r(ay[s], hdt, vy[s]); vz[s] = fma_r(az[s], hdt, vz[s]);
            gpart = fmax(gpart, G * im[s]);
            const bool real = s * T + t < nf;   // neutral slots have im = 0
            if constexpr (KIN) {
                const Real k2 = fma_r(vz[s], vz[s], fma_r(vx[s], vx[s], vy[s] * vy[s])) * rcp_r(im[s]);
                kep += real ? 0.5 * (double)k2 : 0.0;
            }
            if (check) {
                r2p += (double)fx * fx + (double)fy * fy + (double)fz * fz;
                // damping-force norm c |M v| of this node (kinetic damping
                // applies no viscous force but keeps c as the test's scale)
                const Real cm = cg * rcp_r(im[s]);
                const double px = (double)(cm * vx[s]), py = (double)(cm * vy[s]), pz = (double)(cm * vz[s]);
                d2p += real ? px * px + py * py + pz * pz : 0.0;
            }
        });
        if (check) b2p = boundary_norm2(t);
        parity ^= 1;
        double r2n = R2, d2n = D2, b2n = B2;
        reduce(t, parity, gpart, r2p, d2p, b2p, kep, check, gmax, r2n, d2n, b2n, ke);
        if constexpr (KIN) {
            // a kinetic-energy peak was passed: restart every node from rest
            // (the acceleration is already -f/M)
            if (ke < ke_prev) {
#pragma unroll
                for (int s = 0; s < SN; ++s) vx[s] = vy[s] = vz[s] = Real(0);
                ke = 0.0;
                if (check) d2n = 0.0;
            }
            ke_prev = ke;
        }
        if (check) {
            R2 = r2n;
            D2 = d2n;
            B2 = b2n;
            if (!isfinite(R2) || !isfinite(D2)) {
                status = ST_NONFINITE;
                break;
            }
            KernArgs* K = kernel_args<SolveArgs>();
            if (test_in_reach(*K, R2, B2)) {
                const double Rn = sqrt(R2), Dn = sqrt(D2), Bn = sqrt(B2);
                const double tol = fmax(K->tol_abs, K->tol_rel * Bn);
                if (Rn <= tol && Dn <= tol) break;
                if (stagnated(*K, Rn, Dn, Bn, Rref, stall)) {
                    status = ST_STAGNATED;
                    break;
                }
                Rref = uniform(Rref);
            }
        }
        if (!(gmax > Real(0)) || !isfinite(gmax)) {
            status = ST_NONFINITE;
            break;
        }
        if (cd == 0) {
            n += evn;
            const int64_t left = kernel_args<SolveArgs>()->n_max - n;
            if (left <= 0) {
                status = ST_MAXITER;
                evn = 0;
                break;
            }
            evn = cd = uniform32((int)(left < ce ? left : ce));
            ev_test = cd == ce;
        }
    }
    n += evn - cd;   // the stretch the loop was left in

    // ---- fluctuation state for warm starts, positions and the tangent
    int te = tid;
    asm volatile("" : "+v"(te));
    KernArgs* K = kernel_args<SolveArgs>();
    double* hsb = K->h_state + 3 * K->net.free_off[r];
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        const int a = s * T + te;
        if (a < nf) {
            Real x, y, z;
            C::get_h(S, (uint32_t)(a * L.unit), x, y, z);
            double* h = hsb + 3 * a;
            h[0] = (double)x; h[1] = (double)y; h[2] = (double)z;
        }
    }
    if (te == 0) {
        K->status[r] = status;
        K->iters[r] = n;
        K->Rres[r] = sqrt(R2);
        K->Dres[r] = sqrt(D2);
        K->Bres[r] = sqrt(B2);
    }
    __syncthreads();
}

// Register budget (waves per SIMD the build must allow): 128 VGPRs for FP32
// (four waves per SIMD, so two 512-thread or four 256-thread workgroups share a
// CU) and for 1024 threads, 168 for 768 threads, 256 for the other FP64
// builds.  A build that does not fit its budget without private memory is
// never launched (the host checks every build before the first launch).
template <typename Real, int T>
constexpr int chip_waves_per_eu()
{
    return T == 1024 ? 4 : (T == 768 ? 3 : (sizeof(Real) == 8 ? 2 : 4));
}

template <typename Real, int T, int SF, int SN, bool KIN>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(chip_waves_per_eu<Real, T>())))
void dr_chip_kernel(SolveArgs)
{
    __shared__ __attribute__((aligned(16))) char S[Chip<Real, T, SF, SN>::BYTES];
    __shared__ ChipRed<Real> red;
    static_assert(sizeof(S) + sizeof(red) + 64 <= (size_t)res_lds_total(sizeof(Real) == 8, T, SF, SN), "LDS account");
    static_assert(res_lds_total(sizeof(Real) == 8, T, SF, SN) <= 160 * 1024, "LDS of a CU");
    for (;;) {
        KernArgs& A = *kernel_args<SolveArgs>();
        if (threadIdx.x == 0) red.task = atomicAdd(A.queue, 1);
        __syncthreads();
        // the task id is the same for every lane: keep everything derived from it in SGPRs
        const int t = __builtin_amdgcn_readfirstlane(red.task);
        __syncthreads();
        if (t >= A.n_list) break;
        chip_solve<Real, T, SF, SN, KIN>(A, __builtin_amdgcn_readfirstlane(A.list[t]), S, red);
    }
}

const void* chip_kernel(int variant, bool fp64, bool kin)
{
#define RVE_CHIP(R, T, SF, SN) \
    (kin ? (const void*)dr_chip_kernel<R, T, SF, SN, true> : (const void*)dr_chip_kernel<R, T, SF, SN, false>)
    if (fp64) switch (variant) {
        case 0: return RVE_CHIP(double, 256, 4, 2);
        case 1: return RVE_CHIP(double, 512, 4, 2);
        case 3: return RVE_CHIP(double, 512, 6, 3);
        case 6: return RVE_CHIP(double, 512, 8, 4);
        default: return nullptr;
    }
    switch (variant) {
    case 0: return RVE_CHIP(float, 256, 4, 2);
    case 1: return RVE_CHIP(float, 512, 4, 2);
    case 2: return RVE_CHIP(float, 768, 4, 2);
    case 3: return RVE_CHIP(float, 512, 6, 3);
    case 4: return RVE_CHIP(float, 1024, 4, 2);
    case 5: return RVE_CHIP(float, 1024, 6, 3);
    default: return nullptr;
    }
#undef RVE_CHIP
}

}  // namespace

hipError_t launch_resident(int variant, bool fp64, const SolveArgs& a, size_t lds_pad, int grid, hipStream_t s)
{
    const void* k = chip_kernel(variant, fp64, a.kinetic != 0);
    if (!k) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_pad);
    if (e != hipSuccess) return e;
    void* args[] = {const_cast<SolveArgs*>(&a)};
    return hipLaunchKernel(k, dim3(grid), dim3(kResident[variant].threads), args, lds_pad, s);
}

hipError_t max_resident_blocks(int variant, bool fp64, bool kin, size_t lds_pad, int* blocks)
{
    const void* k = chip_kernel(variant, fp64, kin);
    if (!k) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_pad);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k, kResident[variant].threads, lds_pad);
}

hipError_t resident_scratch_bytes(int variant, bool fp64, bool kin, size_t* bytes)
{
    const void* k = chip_kernel(variant, fp64, kin);
    if (!k) return resident_wide_scratch_bytes(variant, fp64, kin, bytes);
    return max_private_bytes({k}, bytes);
}

}  // namespace rve
