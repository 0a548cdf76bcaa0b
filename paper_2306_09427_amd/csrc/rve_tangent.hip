// Material tangent dsigma/dF and its vector-Jacobian product on the state of
// the last relaxation, by matrix-free conjugate gradients on the free-node
// stiffness K_ff (the paper differentiates the stress by finite differences
// of extra relaxations, Section 3.2; here the same linearisation is solved
// directly at the converged network).
//
// Per fiber, K contributes B_f = a n n^T + g (I - n n^T) with n = d/l,
// a = k_t/L0, g = T/l, so (K u)_a = sum_{fibers at a} B_f (u_a - u_other).
//
// Tangent (one right-hand side per F_kl): the boundary moves by E Xm_b,
// E = e_k e_l, so K_ff dx = -[K (E Xm)]_f with [K (E Xm)]_a =
// sum s_af B_f (E d0_f); then df_b = sum s_bf B_f (E d0_f + dx_j - dx_i) and
// dsigma = (sum_b df_b x_b^T + f_b (E Xm_b)^T) / (J V0) - sigma (F^-1)_lk.
//
// VJP (one right-hand side): with y_b = G x_b on boundary nodes (G = dL/dsigma)
// and u = [0; y], solve K_ff lambda = (K u)_f, then z_b = (K [-lambda; y])_b
// and dL/dF_kl = sum_b (z_b + G^T f_b)_k Xm_b,l / (J V0) - (G:sigma) F^-T_kl.
//
// Work decomposition: one wavefront per (RVE, right-hand side) task, pulled
// from a work counter in longest-first order of the RVEs, so the nine solves
// of one RVE's tangent run as nine independent wavefronts with no workgroup
// synchronisation.  A first kernel
// forms, once per call, the fiber operators (FP64 per fiber, FP32 per
// incidence record) and the block-Jacobi preconditioner.  The incidence of
// the free nodes is stored in ELL chunks of 64 nodes (record s of the chunk's
// lane-th node at s*64 + lane), so the lanes of a wavefront read their
// records with unit stride.
//
// Precision: iterative refinement.  The outer loop keeps the solution, the
// right-hand side and the residual r = b - K x in FP64 (FP64 fiber
// operators); each inner solve K d = r is conjugate gradients preconditioned
// by the inverse 3x3 diagonal blocks of K_ff, with FP32 products and FP64 dot
// products, stopped after a 1e-6 reduction of its residual; x += d.  Plain
// FP32 CG stalls near eps_32 cond(K_ff), about 1e-3 on these networks, which
// refinement removes.  The final assembly is FP64.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rve_exchange.h"
#include "rve_internal.h"
#include "rve_relax.h"
#include "rve_wave.h"

namespace rve {

namespace {

typedef KernArgsT<TangentArgs> TanArgs;
typedef float f32x3 __attribute__((ext_vector_type(3)));
constexpr int ST_NO_STATE = 4, ST_CG_MAXITER = 5, ST_CG_INDEFINITE = 6;
constexpr int kOpsThreads = 256;

// ------------------------------------------------------------------ static records
// Fills (fiber, other end) of every ELL record of RVE blockIdx.x from the CSR
// incidence; padding records are (-1, nf).
__global__ __launch_bounds__(kOpsThreads) void ell_build_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    const int r = blockIdx.x;
    auto& net = A.net;
    const int64_t f0 = net.fib_off[r];
    const int64_t a0 = net.free_off[r], nf = net.free_off[r + 1] - a0;
    const int64_t cf = A.chunk_first[r], nch = A.chunk_first[r + 1] - cf;
#pragma unroll 1
    for (int64_t a = threadIdx.x; a < 64 * nch; a += kOpsThreads) {
        const int64_t c = cf + (a >> 6);
        const int64_t base = A.chunk_rec[c] + (a & 63), w = (A.chunk_rec[c + 1] - A.chunk_rec[c]) >> 6;
        const int64_t e0 = a < nf ? net.inc_off[a0 + a] : 0, deg = a < nf ? net.inc_off[a0 + a + 1] - e0 : 0;
#pragma unroll 1
        for (int64_t s = 0; s < w; ++s) {
            int2 v = make_int2(-1, (int)nf);
            if (s < deg) {
                const uint32_t e = net.inc[e0 + s];
                const int64_t k = e & 0x7fffffffu;
                const uint32_t en = net.ends[f0 + k];
                const int64_t o = (e >> 31) ? (int64_t)(en >> 16) : (int64_t)(en & 0xffff);
                v = make_int2((int)k, (int)(o < nf ? o : nf));
            }
            A.rec_static[base + 64 * s] = v;
        }
    }
}

// ------------------------------------------------------------------ fiber operators
// One workgroup per RVE: n, a = k_t/L0, g = T/l and T of every fiber at the
// last solve's state (FP64), then the FP32 record operators and the inverse
// diagonal blocks of K_ff.
__global__ __launch_bounds__(kOpsThreads) void fiber_ops_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    const int r = blockIdx.x;
    if (A.solve_status[r] != 0) return;
    auto& net = A.net;
    const int64_t f0 = net.fib_off[r], nfib = net.fib_off[r + 1] - f0;
    const int64_t a0 = net.free_off[r], nf = net.free_off[r + 1] - a0;
    double F[9];
    for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
#pragma unroll 1
    for (int64_t k = threadIdx.x; k < nfib; k += kOpsThreads) {
        const double* d0 = net.d0 + 3 * (f0 + k);
        const double L0 = net.L0[f0 + k];
        uint32_t e = net.ends[f0 + k];
        int i = e & 0xffff, j = e >> 16;
        double D[3], dh[3] = {0, 0, 0};
        for (int p = 0; p < 3; ++p) D[p] = F[3 * p] * d0[0] + F[3 * p + 1] * d0[1] + F[3 * p + 2] * d0[2];
        for (int p = 0; p < 3; ++p) {
            if (j < nf) dh[p] += A.h_state[3 * (a0 + j) + p];
            if (i < nf) dh[p] -= A.h_state[3 * (a0 + i) + p];
        }
        double q0 = (D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) - L0 * L0;
        double q = q0 + (2.0 * (D[0] * dh[0] + D[1] * dh[1] + D[2] * dh[2]) + (dh[0] * dh[0] + dh[1] * dh[1] + dh[2] * dh[2]));
        double l = sqrt(L0 * L0 + q);
        double eps = q / (L0 * (l + L0));
        double T, kt;
        if (A.law != 0 && eps >= 0.0) {
            double em1 = expm1(A.B * eps);
            T = A.EA * em1 / A.B;
            kt = A.EA * (em1 + 1.0);
        } else {
            T = A.EA * eps;
            kt = A.EA;
        }
        double* q64 = A.par64 + 6 * (f0 + k);
        q64[0] = (D[0] + dh[0]) / l;
        q64[1] = (D[1] + dh[1]) / l;
        q64[2] = (D[2] + dh[2]) / l;
        q64[3] = kt / L0;
        q64[4] = T / l;
        q64[5] = T;
    }
    __syncthreads();
    const double* par64 = A.par64 + 6 * f0;
    const int64_t cf = A.chunk_first[r], nch = A.chunk_first[r + 1] - cf;
#pragma unroll 1
    for (int64_t a = threadIdx.x; a < 64 * nch; a += kOpsThreads) {
        const int64_t c = cf + (a >> 6);
        const int64_t base = A.chunk_rec[c] + (a & 63), w = (A.chunk_rec[c + 1] - A.chunk_rec[c]) >> 6;
        double Dg[6] = {0, 0, 0, 0, 0, 0};   // 00 01 02 11 12 22
#pragma unroll 1
        for (int64_t s = 0; s < w; ++s) {
            const int2 st = A.rec_static[base + 64 * s];
            float4 ra = make_float4(0.f, 0.f, 0.f, 0.f);
            int2 rb = make_int2(st.y, 0);
            if (st.x >= 0) {
                const double* q = par64 + 6 * st.x;
                ra = make_float4((float)q[0], (float)q[1], (float)q[2], (float)q[3]);
                rb.y = __float_as_int((float)q[4]);
                const double c2 = q[3] - q[4];
                Dg[0] += q[4] + c2 * q[0] * q[0];
                Dg[1] += c2 * q[0] * q[1];
                Dg[2] += c2 * q[0] * q[2];
                Dg[3] += q[4] + c2 * q[1] * q[1];
                Dg[4] += c2 * q[1] * q[2];
                Dg[5] += q[4] + c2 * q[2] * q[2];
            }
            A.recA[base + 64 * s] = ra;
            A.recB[base + 64 * s] = rb;
        }
        if (a < nf) {
            // inverse by cofactors when the block is positive definite
            // (leading minors), else a scalar 1/max diagonal
            const double m1 = Dg[0], m2 = Dg[0] * Dg[3] - Dg[1] * Dg[1];
            const double c00 = Dg[3] * Dg[5] - Dg[4] * Dg[4], c01 = Dg[2] * Dg[4] - Dg[1] * Dg[5],
                         c02 = Dg[1] * Dg[4] - Dg[2] * Dg[3], c11 = Dg[0] * Dg[5] - Dg[2] * Dg[2],
                         c12 = Dg[1] * Dg[2] - Dg[0] * Dg[4], c22 = m2;
            const double det = Dg[0] * c00 + Dg[1] * c01 + Dg[2] * c02;
            const double tr = Dg[0] + Dg[3] + Dg[5];
            float4 p0, p1;
            if (m1 > 0.0 && m2 > 0.0 && det > 1e-9 * tr * tr * tr) {
                const double id = 1.0 / det;
                p0 = make_float4((float)(c00 * id), (float)(c01 * id), (float)(c02 * id), (float)(c11 * id));
                p1 = make_float4((float)(c12 * id), (float)(c22 * id), 0.f, 0.f);
            } else {
                const double dm = fmax(fmax(fabs(Dg[0]), fabs(Dg[3])), fabs(Dg[5]));
                const float s = dm > 0.0 ? (float)(1.0 / dm) : 1.f;
                p0 = make_float4(s, 0.f, 0.f, s);
                p1 = make_float4(0.f, s, 0.f, 0.f);
            }
            A.precond[2 * (a0 + a)] = p0;
            A.precond[2 * (a0 + a) + 1] = p1;
        }
    }
}

// ------------------------------------------------------------------ wave helpers
// Values the whole wavefront shares (loaded through vector memory) moved to
// scalar registers.
__device__ __forceinline__ int64_t uni64(int64_t x)
{
    int lo = __builtin_amdgcn_readfirstlane((int)(x & 0xffffffff));
    int hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

__device__ __forceinline__ double uniformd(double x)
{
    int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
    int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ void apply_B64(const double* q, double dx, double dy, double dz, double& wx, double& wy,
                                          double& wz)
{
    double dn = q[0] * dx + q[1] * dy + q[2] * dz;
    double c = (q[3] - q[4]) * dn;
    wx = q[4] * dx + c * q[0];
    wy = q[4] * dy + c * q[1];
    wz = q[4] * dz + c * q[2];
}

// z = P v with P the symmetric inverse block (00, 01, 02, 11), (12, 22, -, -)
__device__ __forceinline__ float4 precond_apply(const float4* P, float4 v)
{
    const float4 p0 = P[0], p1 = P[1];
    return make_float4(p0.x * v.x + p0.y * v.y + p0.z * v.z, p0.y * v.x + p0.w * v.y + p1.x * v.z,
                       p0.z * v.x + p1.x * v.y + p1.y * v.z, 0.f);
}

__device__ __forceinline__ double dot3(float4 a, float4 b)
{
    return (double)a.x * b.x + (double)a.y * b.y + (double)a.z * b.z;
}

// ------------------------------------------------------------------ per-RVE context
struct Ctx {
    int64_t f0, nfib, a0, nf, b0;
    const double* par64;
    const int64_t* incoff;
    const uint32_t* ends;
};

__device__ __forceinline__ Ctx make_ctx(TanArgs& A, int r)
{
    auto& net = A.net;
    Ctx c;
    c.f0 = uni64(net.fib_off[r]);
    c.nfib = uni64(net.fib_off[r + 1]) - c.f0;
    c.a0 = uni64(net.free_off[r]);
    c.nf = uni64(net.free_off[r + 1]) - c.a0;
    c.b0 = uni64(net.bnd_off[r]);
    c.par64 = A.par64 + 6 * c.f0;
    c.incoff = net.inc_off + c.a0;
    c.ends = net.ends + c.f0;
    return c;
}

// Outputs of a task whose RVE has no converged state.  tid: the caller's
// thread id (opaque in the persistent kernels); the NaN is produced at the
// store so that no constant is kept live across tasks.
template <bool TAN>
__device__ void no_state(TanArgs& A, int r, int col, int tid)
{
    if (tid == 0) {
        int code = ST_NO_STATE;
        asm volatile("" : "+v"(code));
        atomicMax(&A.status[r], code);
    }
    if (tid < 9) {
        double nanv = NAN;
        asm volatile("" : "+v"(nanv));
        if (TAN)
            A.out[(int64_t)r * 81 + 9 * tid + col] = nanv;
        else
            A.out[(int64_t)r * 9 + tid] = nanv;
    }
}

// Right-hand side at free node a (FP64).  Tangent: -sum s B_f (e_k d0_l),
// s = +1 at end j, -1 at end i.  VJP: (K u)_a with u = -G x_b on fixed ends.
template <bool TAN>
__device__ __forceinline__ void rhs_node(TanArgs& A, const Ctx& c, int64_t a, int kk, int ll,
                                         const double* F, const double* G, double* b)
{
    auto& net = A.net;
    b[0] = b[1] = b[2] = 0.0;
#pragma unroll 1
    for (int64_t e = c.incoff[a]; e < c.incoff[a + 1]; ++e) {
        const uint32_t w = net.inc[e];
        const int64_t k = w & 0x7fffffffu;
        const double* q = c.par64 + 6 * k;
        if (TAN) {
            const double s = ((w >> 31) ? 1.0 : -1.0) * net.d0[3 * (c.f0 + k) + ll];
            const double nk = kk == 0 ? q[0] : (kk == 1 ? q[1] : q[2]);
            const double cc = (q[3] - q[4]) * nk;
            for (int p = 0; p < 3; ++p) b[p] += s * (cc * q[p] + (p == kk ? q[4] : 0.0));
        } else {
            const uint32_t en = c.ends[k];
            const int64_t o = (w >> 31) ? (int64_t)(en >> 16) : (int64_t)(en & 0xffff);
            if (o >= c.nf) {
                const double* Xm = net.Xb + 3 * (c.b0 + (o - c.nf));
                double x[3], y[3];
                for (int p = 0; p < 3; ++p) x[p] = F[3 * p] * Xm[0] + F[3 * p + 1] * Xm[1] + F[3 * p + 2] * Xm[2];
                for (int p = 0; p < 3; ++p) y[p] = -(G[3 * p] * x[0] + G[3 * p + 1] * x[1] + G[3 * p + 2] * x[2]);
                double w3[3];
                apply_B64(q, y[0], y[1], y[2], w3[0], w3[1], w3[2]);
                for (int p = 0; p < 3; ++p) b[p] += w3[p];
            }
        }
    }
}

// FP64 residual b - K x at free node a; x64 holds the solution (entry nf = 0).
__device__ __forceinline__ void residual_node(TanArgs& A, const Ctx& c, int64_t a, const double* x64,
                                              const double* b64, bool first, double* ra)
{
    for (int p = 0; p < 3; ++p) ra[p] = b64[3 * a + p];
    if (first) return;
    const double xa[3] = {x64[3 * a], x64[3 * a + 1], x64[3 * a + 2]};
#pragma unroll 1
    for (int64_t e = c.incoff[a]; e < c.incoff[a + 1]; ++e) {
        const uint32_t w = A.net.inc[e];
        const uint32_t en = c.ends[w & 0x7fffffffu];
        int64_t o = (w >> 31) ? (int64_t)(en >> 16) : (int64_t)(en & 0xffff);
        o = o < c.nf ? o : c.nf;
        const double* xo = x64 + 3 * o;
        double w3[3];
        apply_B64(c.par64 + 6 * (w & 0x7fffffffu), xa[0] - xo[0], xa[1] - xo[1], xa[2] - xo[2], w3[0], w3[1], w3[2]);
        for (int p = 0; p < 3; ++p) ra[p] -= w3[p];
    }
}

// Partial sums of the assembly over fibers k0, k0 + stride, ... that have a
// fixed end (FP64).  acc[3p + c] collects sum_b df_b,p x_b,c + f_b,p (E Xm_b)_c
// (tangent) or sum_b (z_b + G^T f_b)_p Xm_b,c (VJP).
template <bool TAN>
__device__ __forceinline__ void assembly_partial(TanArgs& A, const Ctx& c, int r, int kk, int ll,
                                                 const double* x64, int64_t k0, int stride, double* acc)
{
    auto& net = A.net;
    double F[9], G[9];
    for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
    if (!TAN)
        for (int k = 0; k < 9; ++k) G[k] = A.gsigma[9 * r + k];
    double z0 = 0.0;   // opaque: no zeros are held in registers for it
    asm volatile("" : "+v"(z0));
#pragma unroll
    for (int p = 0; p < 9; ++p) acc[p] = z0;
#pragma unroll 1
    for (int64_t k = k0; k < c.nfib; k += stride) {
        const uint32_t en = c.ends[k];
        const int64_t i = en & 0xffff, j = en >> 16;
        if (i < c.nf && j < c.nf) continue;
        const double* q = c.par64 + 6 * k;
        double u[3] = {0.0, 0.0, 0.0};
        if (TAN) {
            const double d0l = net.d0[3 * (c.f0 + k) + ll];
            for (int p = 0; p < 3; ++p) {
                u[p] = p == kk ? d0l : 0.0;
                if (j < c.nf) u[p] += x64[3 * j + p];
                if (i < c.nf) u[p] -= x64[3 * i + p];
            }
        } else {
            // u = [-lambda; y] at the two ends, difference j - i
            for (int end = 0; end < 2; ++end) {
                const int64_t node = end ? j : i;
                const double s = end ? 1.0 : -1.0;
                if (node < c.nf) {
                    for (int p = 0; p < 3; ++p) u[p] -= s * x64[3 * node + p];
                } else {
                    const double* Xm = net.Xb + 3 * (c.b0 + (node - c.nf));
                    double x[3];
                    for (int p = 0; p < 3; ++p) x[p] = F[3 * p] * Xm[0] + F[3 * p + 1] * Xm[1] + F[3 * p + 2] * Xm[2];
                    for (int p = 0; p < 3; ++p) u[p] += s * (G[3 * p] * x[0] + G[3 * p + 1] * x[1] + G[3 * p + 2] * x[2]);
                }
            }
        }
        double w[3];
        apply_B64(q, u[0], u[1], u[2], w[0], w[1], w[2]);
        const double fv[3] = {q[5] * q[0], q[5] * q[1], q[5] * q[2]};
        for (int end = 0; end < 2; ++end) {
            const int64_t node = end ? j : i;
            if (node < c.nf) continue;
            const double s = end ? 1.0 : -1.0;
            const double* Xm = net.Xb + 3 * (c.b0 + (node - c.nf));
            if (TAN) {
                double x[3];
                for (int p = 0; p < 3; ++p) x[p] = F[3 * p] * Xm[0] + F[3 * p + 1] * Xm[1] + F[3 * p + 2] * Xm[2];
                const double xl = ll == 0 ? Xm[0] : (ll == 1 ? Xm[1] : Xm[2]);
                for (int p = 0; p < 3; ++p)
                    for (int cc = 0; cc < 3; ++cc) acc[3 * p + cc] += s * (w[p] * x[cc] + (cc == kk ? fv[p] * xl : 0.0));
            } else {
                double gtf[3];
                for (int p = 0; p < 3; ++p) gtf[p] = G[p] * fv[0] + G[3 + p] * fv[1] + G[6 + p] * fv[2];
                for (int p = 0; p < 3; ++p)
                    for (int cc = 0; cc < 3; ++cc) acc[3 * p + cc] += s * (w[p] + gtf[p]) * Xm[cc];
            }
        }
    }
}

// The same sums for one fixed end (0: i, 1: j) of fiber k; xo: x64 of the other
// end (zero where that is fixed too).
template <bool TAN>
__device__ __forceinline__ void assembly_end(TanArgs& A, const Ctx& c, const double* F, const double* G, int kk, int ll,
                                             int64_t k, int end, const double* xo, double* acc)
{
    auto& net = A.net;
    const uint32_t en = c.ends[k];
    const int64_t ends[2] = {(int64_t)(en & 0xffff), (int64_t)(en >> 16)};
    const double* q = c.par64 + 6 * k;
    const double s = end ? 1.0 : -1.0;
    const double* Xm = net.Xb + 3 * (c.b0 + (ends[end] - c.nf));
    double x[3], u[3], w[3];
    for (int p = 0; p < 3; ++p) x[p] = F[3 * p] * Xm[0] + F[3 * p + 1] * Xm[1] + F[3 * p + 2] * Xm[2];
    const double fv[3] = {q[5] * q[0], q[5] * q[1], q[5] * q[2]};
    if (TAN) {
        const double d0l = net.d0[3 * (c.f0 + k) + ll];
        for (int p = 0; p < 3; ++p) u[p] = (p == kk ? d0l : 0.0) - s * xo[p];
        apply_B64(q, u[0], u[1], u[2], w[0], w[1], w[2]);
        const double xl = ll == 0 ? Xm[0] : (ll == 1 ? Xm[1] : Xm[2]);
        for (int p = 0; p < 3; ++p)
            for (int cc = 0; cc < 3; ++cc) acc[3 * p + cc] += s * (w[p] * x[cc] + (cc == kk ? fv[p] * xl : 0.0));
    } else {
        // u = [-lambda; y] at the two ends, difference j - i
        for (int p = 0; p < 3; ++p) u[p] = s * xo[p] + s * (G[3 * p] * x[0] + G[3 * p + 1] * x[1] + G[3 * p + 2] * x[2]);
        if (ends[1 - end] >= c.nf) {
            const double* Xo = net.Xb + 3 * (c.b0 + (ends[1 - end] - c.nf));
            double y[3];
            for (int p = 0; p < 3; ++p) y[p] = F[3 * p] * Xo[0] + F[3 * p + 1] * Xo[1] + F[3 * p + 2] * Xo[2];
            for (int p = 0; p < 3; ++p) u[p] -= s * (G[3 * p] * y[0] + G[3 * p + 1] * y[1] + G[3 * p + 2] * y[2]);
        }
        apply_B64(q, u[0], u[1], u[2], w[0], w[1], w[2]);
        double gtf[3];
        for (int p = 0; p < 3; ++p) gtf[p] = G[p] * fv[0] + G[3 + p] * fv[1] + G[6 + p] * fv[2];
        for (int p = 0; p < 3; ++p)
            for (int cc = 0; cc < 3; ++cc) acc[3 * p + cc] += s * (w[p] + gtf[p]) * Xm[cc];
    }
}

// Final outputs of a task from the summed assembly (one thread).
template <bool TAN>
__device__ void assembly_write(TanArgs& A, int r, int col, const double* acc, int status, int64_t iters)
{
    double F[9];
    for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
    const double J = det3(F);
    const double V0 = A.net.V0[r];
    const double id = 1.0 / J;
    // F^-1 by cofactors
    const double Fi[9] = {(F[4] * F[8] - F[5] * F[7]) * id, (F[2] * F[7] - F[1] * F[8]) * id,
                          (F[1] * F[5] - F[2] * F[4]) * id, (F[5] * F[6] - F[3] * F[8]) * id,
                          (F[0] * F[8] - F[2] * F[6]) * id, (F[2] * F[3] - F[0] * F[5]) * id,
                          (F[3] * F[7] - F[4] * F[6]) * id, (F[1] * F[6] - F[0] * F[7]) * id,
                          (F[0] * F[4] - F[1] * F[3]) * id};
    if (TAN) {
        const int kk = col / 3, ll = col % 3;
        double fi = 0.0;   // (F^-1)_{l k}
        for (int m = 0; m < 9; ++m) fi = m == 3 * ll + kk ? Fi[m] : fi;
        for (int p = 0; p < 9; ++p)
            A.out[(int64_t)r * 81 + 9 * p + col] = acc[p] / (J * V0) - A.sigma[9 * r + p] * fi;
    } else {
        double gs = 0.0;
        for (int p = 0; p < 9; ++p) gs += A.gsigma[9 * r + p] * A.sigma[9 * r + p];
        for (int p = 0; p < 9; ++p) {
            const int k2 = p / 3, l2 = p % 3;
            A.out[(int64_t)r * 9 + p] = acc[p] / (J * V0) - gs * Fi[3 * l2 + k2];
        }
    }
    if (status != ST_CONVERGED) atomicMax(&A.status[r], status);
    atomicAdd(&A.iters[r], (unsigned long long)iters);
}

// ------------------------------------------------------------------ workgroup sums
struct CgRed {
    double s[2][3][16];   // per-wavefront partial sums, alternating buffers
};

// q[0] + ... + q[NW - 1] in order, the reads issued eight together (left to
// itself the compiler waits for each pair before the next: eight LDS latencies
// in a row; all sixteen at once spill).
template <int NW>
__device__ __forceinline__ double sum_in_order(const double* q)
{
    constexpr int U = NW < 8 ? NW : 8;
    double x = 0.0;
#pragma unroll
    for (int j = 0; j < NW; j += U) {
        double v[U];
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = q[j + i];
#pragma unroll
        for (int i = 0; i < U; ++i) asm volatile("" : "+v"(v[i]));
#pragma unroll
        for (int i = 0; i < U; ++i) x += v[i];
    }
    return x;
}

// Totals of N <= 3 values over the workgroup, in every thread: wave sums, then
// the waves in order.  One barrier; the buffers alternate with `parity`.
template <int NW, int N>
__device__ __forceinline__ void block_sums(CgRed& red, int parity, double (&v)[N])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] = wave_sum(v[q]);
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < N; ++q) red.s[parity][q][wave] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; ++q) {
        v[q] = uniformd(sum_in_order<NW>(red.s[parity][q]));
    }
}
template <int NW>
__device__ __forceinline__ void block_sum3(CgRed& red, int parity, double& a, double& b, double& c)
{
    double v[3] = {a, b, c};
    block_sums<NW, 3>(red, parity, v);
    a = v[0];
    b = v[1];
    c = v[2];
}
template <int NW>
__device__ __forceinline__ void block_sum2(CgRed& red, int parity, double& a, double& b)
{
    double v[2] = {a, b};
    block_sums<NW, 2>(red, parity, v);
    a = v[0];
    b = v[1];
}
template <int NW>
__device__ __forceinline__ void block_sum1(CgRed& red, int parity, double& a)
{
    double v[1] = {a};
    block_sums<NW, 1>(red, parity, v);
    a = v[0];
}

// ------------------------------------------------------------------ streamed tasks
// A task is (RVE r, right-hand side col): col = 3k + l for the tangent, 0 for
// the VJP.  One workgroup of T threads (T = 64: one wavefront); wavefront w
// takes ELL chunks w, w + T/64, ... and lane = node within its chunk.
// Solver vectors live in the workgroup's global slot (any RVE size).
template <bool TAN, int T>
__device__ void cg_stream_task(TanArgs& A, int r, int col, CgRed& red)
{
    constexpr int NW = T / 64;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int parity = 0;
    // sums over the workgroup (every thread gets the same totals)
    auto sum1 = [&](double& x) __attribute__((always_inline)) {
        if (T == 64) {
            x = uniformd(wave_sum(x));
        } else {
            block_sum1<NW>(red, parity, x);
            parity ^= 1;
        }
    };
    auto sum2 = [&](double& x, double& y) __attribute__((always_inline)) {
        if (T == 64) {
            x = uniformd(wave_sum(x));
            y = uniformd(wave_sum(y));
        } else {
            block_sum2<NW>(red, parity, x, y);
            parity ^= 1;
        }
    };
    if (__builtin_amdgcn_readfirstlane(A.solve_status[r]) != 0) {
        no_state<TAN>(A, r, col, tid);
        return;
    }
    const Ctx c = make_ctx(A, r);
    const int64_t nf = c.nf;
    const int kk = col / 3, ll = col % 3;
    const float4* Pc = A.precond + 2 * c.a0;
    const int64_t cf = uni64(A.chunk_first[r]), nch = uni64(A.chunk_first[r + 1]) - cf;
    const float4* recA = A.recA;
    const int2* recB = A.recB;

    // slot workspace: FP64 x and b (3 per node), FP32 p, q, r, d, z (float4
    // per node); entry nf of p and x is the zero vector of fixed ends
    const int64_t S = A.slot_nodes;
    double* x64 = A.slot_ws64 + (int64_t)blockIdx.x * 6 * S;
    double* b64 = x64 + 3 * S;
    float4* vp = A.slot_ws32 + (int64_t)blockIdx.x * 5 * S;
    float4* vq = vp + S;
    float4* vr = vq + S;
    float4* vd = vr + S;
    float4* vz = vd + S;
    if (tid == 0) vp[nf] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < 3) x64[3 * nf + tid] = 0.0;

    double bb = 0.0;
    {
        double F[9], G[9];
        for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
        if (!TAN)
            for (int k = 0; k < 9; ++k) G[k] = A.gsigma[9 * r + k];
#pragma unroll 1
        for (int64_t a = tid; a < nf; a += T) {
            double b[3];
            rhs_node<TAN>(A, c, a, kk, ll, F, G, b);
            for (int p = 0; p < 3; ++p) {
                b64[3 * a + p] = b[p];
                x64[3 * a + p] = 0.0;
            }
            bb += b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
        }
    }
    sum1(bb);
    __syncthreads();

    int status = ST_CONVERGED;
    const double tol2 = A.cg_tol * A.cg_tol;
    const int64_t maxit = A.cg_max > 0 ? A.cg_max : 6 * nf + 100;
    int64_t it_total = 0;
    bool done = !(bb > 0.0);
    for (int outer = 0; outer < 8 && !done; ++outer) {
        // FP64 residual r = b - K x of the FP64 solution; z = P r, p = z
        double rr = 0.0, rz = 0.0;
#pragma unroll 1
        for (int64_t a = tid; a < nf; a += T) {
            double ra[3];
            residual_node(A, c, a, x64, b64, outer == 0, ra);
            const float4 r4 = make_float4((float)ra[0], (float)ra[1], (float)ra[2], 0.f);
            const float4 z4 = precond_apply(Pc + 2 * a, r4);
            vr[a] = r4;
            vz[a] = z4;
            vp[a] = z4;
            vd[a] = make_float4(0.f, 0.f, 0.f, 0.f);
            rr += ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2];
            rz += dot3(r4, z4);
        }
        sum2(rr, rz);
        __syncthreads();
        if (rr <= tol2 * bb) {
            done = true;
            break;
        }
        if (it_total >= maxit) {
            status = ST_CG_MAXITER;
            break;
        }
        // inner preconditioned CG with FP32 products
        const double rr0 = rr;
        for (;;) {
            if (it_total >= maxit) break;
            ++it_total;
            // q = K p over the ELL records of each chunk
            double pq = 0.0;
#pragma unroll 1
            for (int64_t ch = wave; ch < nch; ch += NW) {
                const int64_t a = 64 * ch + lane;
                const int64_t c0 = uni64(A.chunk_rec[cf + ch]), w = (uni64(A.chunk_rec[cf + ch + 1]) - c0) >> 6;
                const int64_t rb = c0 + lane;
                if (a < nf) {
                    const float4 pa = vp[a];
                    float qx = 0.f, qy = 0.f, qz = 0.f;
                    // w is a multiple of 4: issue 4 records' loads, then their gathers
#pragma unroll 1
                    for (int64_t s0 = 0; s0 < w; s0 += 4) {
                        float4 nA[4];
                        int2 ob[4];
                        float4 po[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            nA[u] = recA[rb + 64 * (s0 + u)];
                            ob[u] = recB[rb + 64 * (s0 + u)];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) po[u] = vp[ob[u].x];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float g = __int_as_float(ob[u].y);
                            const float dx = pa.x - po[u].x, dy = pa.y - po[u].y, dz = pa.z - po[u].z;
                            const float cn = (nA[u].w - g) * (nA[u].x * dx + nA[u].y * dy + nA[u].z * dz);
                            qx += fmaf(g, dx, cn * nA[u].x);
                            qy += fmaf(g, dy, cn * nA[u].y);
                            qz += fmaf(g, dz, cn * nA[u].z);
                        }
                    }
                    vq[a] = make_float4(qx, qy, qz, 0.f);
                    pq += (double)pa.x * qx + (double)pa.y * qy + (double)pa.z * qz;
                }
            }
            sum1(pq);
            if (!(pq > 0.0)) {
                status = ST_CG_INDEFINITE;
                done = true;
                break;
            }
            const float alpha = (float)(rz / pq);
            double rn = 0.0, rzn = 0.0;
#pragma unroll 1
            for (int64_t a = tid; a < nf; a += T) {
                const float4 pa = vp[a], qa = vq[a];
                float4 da = vd[a], ra = vr[a];
                da.x = fmaf(alpha, pa.x, da.x);
                da.y = fmaf(alpha, pa.y, da.y);
                da.z = fmaf(alpha, pa.z, da.z);
                ra.x = fmaf(-alpha, qa.x, ra.x);
                ra.y = fmaf(-alpha, qa.y, ra.y);
                ra.z = fmaf(-alpha, qa.z, ra.z);
                const float4 za = precond_apply(Pc + 2 * a, ra);
                vd[a] = da;
                vr[a] = ra;
                vz[a] = za;
                rn += dot3(ra, ra);
                rzn += dot3(ra, za);
            }
            sum2(rn, rzn);
            if (rn <= 1e-6 * rr0 || rn <= 0.25 * tol2 * bb) break;
            const float beta = (float)(rzn / rz);
            rz = rzn;
#pragma unroll 1
            for (int64_t a = tid; a < nf; a += T) {
                const float4 za = vz[a];
                float4 pa = vp[a];
                pa.x = fmaf(beta, pa.x, za.x);
                pa.y = fmaf(beta, pa.y, za.y);
                pa.z = fmaf(beta, pa.z, za.z);
                vp[a] = pa;
            }
            __syncthreads();
        }
        // x += d
        __syncthreads();
#pragma unroll 1
        for (int64_t a = tid; a < nf; a += T) {
            const float4 da = vd[a];
            x64[3 * a] += (double)da.x;
            x64[3 * a + 1] += (double)da.y;
            x64[3 * a + 2] += (double)da.z;
        }
        __syncthreads();
        if (outer == 7 && !done && status == ST_CONVERGED) status = ST_CG_MAXITER;
    }

    double acc[9];
    assembly_partial<TAN>(A, c, r, kk, ll, x64, tid, T, acc);
    if (T == 64) {
#pragma unroll
        for (int p = 0; p < 9; ++p) acc[p] = wave_sum(acc[p]);
    } else {
#pragma unroll
        for (int p = 0; p < 9; p += 3) {
            block_sum3<NW>(red, parity, acc[p], acc[p + 1], acc[p + 2]);
            parity ^= 1;
        }
    }
    if (tid == 0) assembly_write<TAN>(A, r, col, acc, status, it_total);
    __syncthreads();
}

template <bool TAN, int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void cg_stream_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    __shared__ CgRed red;
    __shared__ int task;
    constexpr int per = TAN ? 9 : 1;
    const int64_t n_tasks = A.n_order * per;
    for (;;) {
        if (threadIdx.x == 0) task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(task);
        __syncthreads();
        if (t >= n_tasks) break;
        if (A.done && A.done[t]) continue;
        cg_stream_task<TAN, T>(A, __builtin_amdgcn_readfirstlane(A.order[t / per]), t % per, red);
    }
}

// ------------------------------------------------------------------ on-chip tasks
// Tasks of RVEs of at most 2048 free nodes: nothing but the workgroup's sums
// and one vector leaves the registers during the inner solve.  Thread tid owns
// free nodes tid + T k (k < SN); each node slot keeps its first four records
// (the chunks of nodes of degree <= 4 hold no more), its inverse block and its
// p, r, q and d in VGPRs; p is exchanged through LDS, where the records beyond
// four of the nodes x4 .. nf (the packing puts the degrees above 4 last) are
// held too.  Reading the records from L2 in every iteration (24 bytes each,
// about 250 iterations) took three quarters of an iteration.
//
// An iteration is bound by vector instruction issue (0.72 of the cycles) and by
// its serial chain: three barriers, two FP64 sums over the workgroup and two FP64
// quotients, which every wave works out for itself (r.r and r.z share one
// butterfly, put_pair).  From 1024 free nodes on these cost more than the
// latency that more waves hide: four nodes in 512 threads take 3.3 us per
// iteration at 1742 free nodes where two in 1024 took 3.7 (2.8 and 3.05 on a
// full chip); below, two nodes per thread are better (178 free nodes 1.55 us in
// 256 threads, 1.98 in 128; 791 2.35 in 512, 2.61 in 256).  Microseconds per
// iteration of one RVE, records from L2 -> here: 2.43 -> 1.55 at 178 free nodes,
// 3.78 -> 2.35 at 791, 6.16 -> 3.3 at 1742.
//
// The arithmetic, its rounding and the order of every sum are those of
// cg_res_task.
template <int N>
struct ChipExtra {
    static constexpr int XN = N / 8;   // rows of nodes: 4 records each
    float4 A[4 * XN];                  // (n, k_t/L0 - T/l)
    int2 B[4 * XN];                    // (LDS byte offset of the other end, bits of T/l)
    int x4, xd;
};

// s += B_f (p - po) of one record; c = k_t/L0 - T/l
__device__ __forceinline__ void add_record(float nx, float ny, float nz, float c, float g, const float* p, f32x3 po,
                                           float* s)
{
#pragma clang fp contract(off)
    const float dx = p[0] - po.x, dy = p[1] - po.y, dz = p[2] - po.z;
    const float cn = c * fmaf(nz, dz, fmaf(nx, dx, ny * dy));
    s[0] += fmaf(g, dx, cn * nx);
    s[1] += fmaf(g, dy, cn * ny);
    s[2] += fmaf(g, dz, cn * nz);
}
// z = P r, P = (00, 01, 02, 11, 12, 22)
__device__ __forceinline__ void apply_block(const float* P, const float* r, float* z)
{
#pragma clang fp contract(off)
    z[0] = fmaf(P[2], r[2], fmaf(P[1], r[1], P[0] * r[0]));
    z[1] = fmaf(P[4], r[2], fmaf(P[3], r[1], P[1] * r[0]));
    z[2] = fmaf(P[5], r[2], fmaf(P[2], r[0], P[4] * r[1]));
}

// Sums over the workgroup, in every thread.  H = 2: in the order of twice as many
// threads with half the nodes: the even slots' partial sum a[0] and the odd
// slots' a[1] of wave w are those of waves w and w + NW there.  put_pair: one
// butterfly for two sums; after the exchange of stage 32 the lower half of the
// wave holds v0's, the upper half v1's.
template <int NW>
__device__ __forceinline__ void put_pair(double* s0, double* s1, int tid, double v0, double v1)
{
    const int lane = tid & 63, wave = tid >> 6;
    double v = halves_xor32(v0, v1);
    v = add_xor16(v);
    v += dpp_mov<kDppRor8>(v);
    v += dpp_mov<kDppRor4>(v);
    v += dpp_mov<kDppXor2>(v);
    v += dpp_mov<kDppXor1>(v);
    if ((lane & 31) == 0) (lane ? s1 : s0)[wave] = v;
}
template <int NW, int H>
__device__ __forceinline__ double chip_sum(CgRed& red, int parity, int tid, const double* a)
{
    double* s = red.s[parity][0];
    if (H == 2) {
        put_pair<NW>(s, s + NW, tid, a[0], a[H - 1]);
    } else {
        const double v = wave_sum(a[0]);
        if ((tid & 63) == 0) s[tid >> 6] = v;
    }
    __syncthreads();
    return uniformd(sum_in_order<H * NW>(s));
}
// two sums; the halves of the wave add one each
template <int NW, int H>
__device__ __forceinline__ void chip_sum2(CgRed& red, int parity, int tid, double* a, double* b)
{
    double *sa = red.s[parity][0], *sb = red.s[parity][1];
    if (H == 2) {
        put_pair<NW>(sa, sa + NW, tid, a[0], a[H - 1]);
        put_pair<NW>(sb, sb + NW, tid, b[0], b[H - 1]);
    } else {
        put_pair<NW>(sa, sb, tid, a[0], b[0]);
    }
    __syncthreads();
    const double x = sum_in_order<H * NW>((tid & 32) ? sb : sa);
    a[0] = readlane_d(x, 0);
    b[0] = readlane_d(x, 32);
}

template <bool TAN, int T, int SN>
__device__ void cg_chip_task(TanArgs& A, int r, int col, float4* zl, ChipExtra<T * SN>& X, CgRed& red)
{
    constexpr int NW = T / 64, H = SN > 2 ? 2 : 1;   // H partial sums per thread (chip_sum)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (__builtin_amdgcn_readfirstlane(A.solve_status[r]) != 0) {
        no_state<TAN>(A, r, col, tid);
        return;
    }
    const Ctx c = make_ctx(A, r);
    const int nf = (int)c.nf;
    const int kk = col / 3, ll = col % 3;
    const int64_t cf = uni64(A.chunk_first[r]);
    const int64_t S = A.slot_nodes;
    double* x64 = A.slot_ws64 + (int64_t)blockIdx.x * 8 * S;   // x, b (3 S each)
    double* b64 = x64 + 3 * S;
    const int64_t rec0 = uni64(A.chunk_rec[cf]);
    const float4* recA = A.recA + rec0;
    const int2* recB = A.recB + rec0;
    int parity = 0;
    if (tid == 0) {
        int xd = 4;
        asm volatile("" : "+v"(xd));
        X.x4 = nf;
        X.xd = xd;
    }
    __syncthreads();

    // opaque zeros: no zero vectors are held in registers across tasks
    double b2[2] = {0.0, 0.0};
    float zf = 0.f;
    asm volatile("" : "+v"(b2[0]), "+v"(b2[1]), "+v"(zf));
    // right-hand side (FP64)
    {
        double F[9], G[9];
        for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
        if (!TAN)
            for (int k = 0; k < 9; ++k) G[k] = A.gsigma[9 * r + k];
#pragma unroll 1
        for (int k = 0; k < SN; ++k) {
            const int a = tid + T * k;
            if (a < nf) {
                double b[3];
                rhs_node<TAN>(A, c, a, kk, ll, F, G, b);
                double zx = 0.0;
                asm volatile("" : "+v"(zx));
                for (int p = 0; p < 3; ++p) {
                    b64[3 * a + p] = b[p];
                    x64[3 * a + p] = zx;
                }
                const double bn = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
                if (k % H)
                    b2[1] += bn;
                else
                    b2[0] += bn;
                const int deg = (int)(c.incoff[a + 1] - c.incoff[a]);
                if (deg > 4) {
                    atomicMin(&X.x4, a);
                    atomicMax(&X.xd, deg);
                }
            }
        }
        double zx = 0.0;
        asm volatile("" : "+v"(zx));
        if (tid < 3) x64[3 * nf + tid] = zx;
    }
    const double bb = chip_sum<NW, H>(red, parity, tid, b2);
    parity ^= 1;

    // records, blocks and extra records on chip (read once per task)
    const int x4 = __builtin_amdgcn_readfirstlane(X.x4), nx = nf - x4;
    const int xrows = (__builtin_amdgcn_readfirstlane(X.xd) - 1) / 4;
    const bool xtab = xrows * nx <= ChipExtra<T * SN>::XN;
    float rx[SN][4], ry[SN][4], rz_[SN][4], rc[SN][4], rg[SN][4];
    uint32_t ro[SN][2];   // LDS byte offsets of the other ends, two per word
    float Pb[SN][6];
    int rb[SN], wd[SN];   // first record and width of the slot's chunk (scalar width; 0 past the last node)
#pragma unroll
    for (int k = 0; k < SN; ++k) {
        const int ch = wave + NW * k, a = tid + T * k;
        rb[k] = 0;
        wd[k] = 0;
        float4 p0 = make_float4(zf, zf, zf, zf), p1 = p0;
        uint32_t o4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            rx[k][u] = ry[k][u] = rz_[k][u] = rc[k][u] = rg[k][u] = zf;
            o4[u] = 16u * (uint32_t)(T * SN);
        }
        if (64 * ch < nf) {
            const int64_t c0 = uni64(A.chunk_rec[cf + ch]);
            wd[k] = (int)((uni64(A.chunk_rec[cf + ch + 1]) - c0) >> 6);
            rb[k] = (int)(c0 - rec0) + (tid & 63);
            if (a < nf) {
                p0 = A.precond[2 * (c.a0 + a)];
                p1 = A.precond[2 * (c.a0 + a) + 1];
            }
            if (wd[k] > 0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 ra = recA[rb[k] + 64 * u];
                    const int2 ob = recB[rb[k] + 64 * u];
                    rx[k][u] = ra.x; ry[k][u] = ra.y; rz_[k][u] = ra.z;
                    rg[k][u] = __int_as_float(ob.y);
                    rc[k][u] = ra.w - rg[k][u];
                    o4[u] = 16u * (uint32_t)(ob.x < nf ? ob.x : T * SN);
                }
            }
            if (xtab && a >= x4 && a < nf) {
#pragma unroll 1
                for (int j = 0; j < 4 * xrows; ++j) {
                    float4 ra = make_float4(zf, zf, zf, zf);
                    int2 ob = make_int2(nf, 0);
                    if (4 + j < wd[k]) {
                        ra = recA[rb[k] + 64 * (4 + j)];
                        ob = recB[rb[k] + 64 * (4 + j)];
                    }
                    ra.w -= __int_as_float(ob.y);
                    ob.x = 16 * (ob.x < nf ? ob.x : T * SN);
                    X.A[j * nx + (a - x4)] = ra;
                    X.B[j * nx + (a - x4)] = ob;
                }
            }
        }
        ro[k][0] = o4[0] | o4[1] << 16;
        ro[k][1] = o4[2] | o4[3] << 16;
        Pb[k][0] = p0.x; Pb[k][1] = p0.y; Pb[k][2] = p0.z; Pb[k][3] = p0.w; Pb[k][4] = p1.x; Pb[k][5] = p1.y;
        __builtin_amdgcn_sched_barrier(0);
    }
    float P[SN][3], R[SN][3], Q[SN][3], D[SN][3];
    char* zb = reinterpret_cast<char*>(zl);

    int status = ST_CONVERGED;
    // per-task copy: a kernel-lifetime value would be kept live across tasks
    double cgt = A.cg_tol;
    asm volatile("" : "+v"(cgt));
    const double tol2 = uniformd(cgt * cgt);
    const int64_t maxit = A.cg_max > 0 ? A.cg_max : 6 * (int64_t)nf + 100;
    int64_t it_total = 0;
    bool done = !(bb > 0.0);
    for (int outer = 0; outer < 8 && !done; ++outer) {
        // thread id opaque per phase: no per-thread address is hoisted out of
        // the loops and kept live across them
        asm volatile("" : "+v"(tid));
        // FP64 residual of the FP64 solution (x64 complete: barrier above);
        // d = 0, p = z = P r
        double rr2[2] = {0.0, 0.0}, rz2[2] = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int a = tid + T * k;
            double z0 = 0.0;   // opaque: no zeros are held in registers for it
            asm volatile("" : "+v"(z0));
            double ra[3] = {z0, z0, z0};
            if (a < nf) residual_node(A, c, a, x64, b64, outer == 0, ra);
            for (int p = 0; p < 3; ++p) R[k][p] = (float)ra[p];
            rr2[k % H] += ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2];
            apply_block(Pb[k], R[k], P[k]);
            rz2[k % H] += (double)R[k][0] * P[k][0] + (double)R[k][1] * P[k][1] + (double)R[k][2] * P[k][2];
            __builtin_amdgcn_sched_barrier(0);
        }
        chip_sum2<NW, H>(red, parity, tid, rr2, rz2);
        parity ^= 1;
        const double rr = rr2[0];
        double rz = rz2[0];
        if (rr <= tol2 * bb) {
            done = true;
            break;
        }
        if (it_total >= maxit) {
            status = ST_CG_MAXITER;
            break;
        }
        // inner preconditioned CG (FP32 vectors, p exchanged through LDS):
        // q = K p, alpha = rz / p.q, d += alpha p, r -= alpha q, z = P r,
        // beta = r.z / rz, p = z + beta p
        double drop = 1e-6;
        asm volatile("" : "+s"(drop));
        const double rr0 = uniformd(drop * rr);
#pragma unroll
        for (int k = 0; k < SN; ++k)
            for (int p = 0; p < 3; ++p) D[k][p] = Q[k][p] = 0.f;
        for (;;) {
            if (it_total >= maxit) break;
            ++it_total;
            asm volatile("" : "+v"(tid));
            // the packed offsets stay packed
#pragma unroll
            for (int k = 0; k < SN; ++k) asm volatile("" : "+v"(ro[k][0]), "+v"(ro[k][1]));
#pragma unroll
            for (int k = 0; k < SN; ++k) *(f32x3*)&zl[tid + T * k] = f32x3{P[k][0], P[k][1], P[k][2]};
            __syncthreads();
            double pq2[2] = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < SN; ++k) {
                if (wd[k] > 0) {
                    f32x3 po[4];
                    float s[3] = {0.f, 0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        po[u] = *(const f32x3*)(zb + ((u & 1) ? ro[k][u >> 1] >> 16 : ro[k][u >> 1] & 0xffffu));
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        add_record(rx[k][u], ry[k][u], rz_[k][u], rc[k][u], rg[k][u], P[k], po[u], s);
                    if (wd[k] > 4) {
                        if (xtab) {
                            const int i = tid + T * k - x4;
                            if (i >= 0 && i < nx) {
#pragma unroll 1
                                for (int j = 0; j < wd[k] - 4; j += 2) {
                                    const float4 a0 = X.A[j * nx + i], a1 = X.A[(j + 1) * nx + i];
                                    const int2 b0 = X.B[j * nx + i], b1 = X.B[(j + 1) * nx + i];
                                    const f32x3 q0 = *(const f32x3*)(zb + b0.x), q1 = *(const f32x3*)(zb + b1.x);
                                    add_record(a0.x, a0.y, a0.z, a0.w, __int_as_float(b0.y), P[k], q0, s);
                                    add_record(a1.x, a1.y, a1.z, a1.w, __int_as_float(b1.y), P[k], q1, s);
                                }
                            }
                        } else {
#pragma unroll 1
                            for (int j = 4; j < wd[k]; ++j) {
                                const float4 ra = recA[rb[k] + 64 * j];
                                const int2 ob = recB[rb[k] + 64 * j];
                                const float g = __int_as_float(ob.y);
                                add_record(ra.x, ra.y, ra.z, ra.w - g, g, P[k], *(const f32x3*)&zl[ob.x < nf ? ob.x : T * SN], s);
                            }
                        }
                    }
                    for (int p = 0; p < 3; ++p) Q[k][p] = s[p];
                    pq2[k % H] += (double)P[k][0] * s[0] + (double)P[k][1] * s[1] + (double)P[k][2] * s[2];
                }
            }
            const double pq = chip_sum<NW, H>(red, parity, tid, pq2);
            parity ^= 1;
            if (!(pq > 0.0)) {
                status = ST_CG_INDEFINITE;
                done = true;
                break;
            }
            const float af = (float)(rz / pq);
            double rn2[2] = {0.0, 0.0}, rzn2[2] = {0.0, 0.0};
            float (&Z)[SN][3] = Q;   // (q is done with)
#pragma unroll
            for (int k = 0; k < SN; ++k)
                if (k == 0 || wd[k] > 0) {   // (nothing to do for a wave without nodes in the slot)
                    for (int p = 0; p < 3; ++p) {
                        D[k][p] = fmaf(af, P[k][p], D[k][p]);
                        R[k][p] = fmaf(-af, Q[k][p], R[k][p]);
                    }
                    apply_block(Pb[k], R[k], Z[k]);
                    rn2[k % H] += (double)R[k][0] * R[k][0] + (double)R[k][1] * R[k][1] + (double)R[k][2] * R[k][2];
                    rzn2[k % H] += (double)R[k][0] * Z[k][0] + (double)R[k][1] * Z[k][1] + (double)R[k][2] * Z[k][2];
                }
            chip_sum2<NW, H>(red, parity, tid, rn2, rzn2);
            parity ^= 1;
            const double rn = rn2[0], rzn = rzn2[0];
            if (rn <= rr0 || rn <= 0.25 * tol2 * bb) break;
            const float bf = (float)(rzn / rz);
            rz = rzn;
#pragma unroll
            for (int k = 0; k < SN; ++k)
                if (k == 0 || wd[k] > 0)
                    for (int p = 0; p < 3; ++p) P[k][p] = fmaf(bf, P[k][p], Z[k][p]);
        }
        // x += d
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int a = tid + T * k;
            if (a < nf)
                for (int p = 0; p < 3; ++p) x64[3 * a + p] += (double)D[k][p];
        }
        __syncthreads();
        if (outer == 7 && !done && status == ST_CONVERGED) status = ST_CG_MAXITER;
    }

    // assembly (x64 complete: barrier above, or no update since the RHS sum)
    double acc[9];
    assembly_partial<TAN>(A, c, r, kk, ll, x64, tid, T, acc);
    double tot[9];
#pragma unroll
    for (int p = 0; p < 9; p += 3) {
        double a1 = acc[p], a2 = acc[p + 1], a3 = acc[p + 2];
        block_sum3<NW>(red, parity, a1, a2, a3);
        parity ^= 1;
        tot[p] = a1;
        tot[p + 1] = a2;
        tot[p + 2] = a3;
    }
    if (tid == 0) assembly_write<TAN>(A, r, col, tot, status, it_total);
    __syncthreads();
}

template <bool TAN, int T, int SN>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(SN > 2 ? 2 : 4))) void cg_chip_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    __shared__ float4 zl[T * SN + 1];   // the last entry stays zero
    __shared__ ChipExtra<T * SN> X;
    __shared__ CgRed red;
    __shared__ int task;
    if (threadIdx.x == 0) zl[T * SN] = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int per = TAN ? 9 : 1;
    const int64_t n_tasks = A.n_order * per;
    for (;;) {
        if (threadIdx.x == 0) task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(task);
        __syncthreads();
        if (t >= n_tasks) break;
        cg_chip_task<TAN, T, SN>(A, __builtin_amdgcn_readfirstlane(A.order[t / per]), t % per, zl, X, red);
    }
}

// ------------------------------------------------------------------ spread tasks
// Tasks of RVEs above 4096 free nodes: k workgroups per task, on the partition
// and with the exchange of the spread relaxation (rve_internal.h,
// rve_exchange.h).  A member holds its nodes (at most 2048) as cg_chip_task
// does, four per thread of 512; the streamed kernel read 3.7 MB per iteration
// and column at 10 300 free nodes, beyond every L2 once several columns run.
//
// Two exchanges per iteration: p.K p, and r.r and r.z with z of the nodes other
// parts hold as halo, whose p (and correction) each part then updates itself,
// with the operations of the owner.  Each is one round trip through memory
// (about 2 us), which with the barriers around it is what bounds an iteration.
// Microseconds per iteration, all nine columns at once, streamed -> here: one RVE
// of 4900 free nodes 22 -> 6.5, of 10 300 42 -> 8.2, of 16 000 76 -> 8.7; 28 RVEs
// 46 -> 34, 110 -> 38 and 184 -> 59.  The tangents of 256 RVEs of 100 to 3000 seeds took
// 50 ms with the streamed kernel and take 27.
//
// The arithmetic and its rounding are those of cg_stream_task but for the order
// of the FP64 sums.  A task whose team gave up keeps its mark and runs on the
// streamed kernel launched behind.

// z = P r with the order of the products in cg_stream_task
__device__ __forceinline__ void apply_block_yxz(const float* P, const float* r, float* z)
{
#pragma clang fp contract(off)
    z[0] = fmaf(P[2], r[2], fmaf(P[0], r[0], P[1] * r[1]));
    z[1] = fmaf(P[4], r[2], fmaf(P[1], r[0], P[3] * r[1]));
    z[2] = fmaf(P[5], r[2], fmaf(P[2], r[0], P[4] * r[1]));
}

struct SpreadCgArgs {
    TangentArgs t;
    SpreadArgs sp;
};
constexpr int kCgT = kSpreadThreads, kCgSN = kSpreadSlots, kCgHN = kSpreadNodes / kSpreadThreads;

struct CgSpreadRed : TeamSlot {
    double v[2][3][kCgT / 64];
    double sum[2][3][kTeamMax];
};

template <bool TAN>
__device__ __forceinline__ bool cg_spread_task(KernArgsT<SpreadCgArgs>& AA, Team& tm, float4* zl, f32x3* dh, f32x3* hz, float4* XA, int2* XB,
                                               CgSpreadRed& red)
{
    constexpr int T = kCgT, SN = kCgSN, HN = kCgHN, NW = T / 64;
    constexpr int per = TAN ? 9 : 1;
    TanArgs& A = AA.t;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wave64 = 64 * wave;
    const int r = __builtin_amdgcn_readfirstlane(A.order[tm.task / per]), col = tm.task % per;
    const int k = tm.k, rank = tm.rank, max_x = AA.sp.max_x, half = (AA.sp.area_words - 16) / 2;
    u64* const xbuf = tm.area + 16;
    auto words_of = [&](unsigned t) __attribute__((always_inline)) { return xbuf + (t & 1) * half + 3 * (int64_t)max_x; };
    if (__builtin_amdgcn_readfirstlane(A.solve_status[r]) != 0) {   // the same in every member
        ++tm.tag;
        const bool all = team_done(AA.sp, red, tm, words_of(tm.tag));
        if (rank == 0 && all) {
            no_state<TAN>(A, r, col, tid);
            if (tid == 0) A.done[tm.task] = 1;
        }
        return all;
    }
    const Ctx c = make_ctx(A, r);
    const int kk = col / 3, ll = col % 3;
    const int64_t pi = uni64(AA.sp.part_first[r]) + rank;
    const int nown = __builtin_amdgcn_readfirstlane(AA.sp.parts[pi].nown), nhalo = __builtin_amdgcn_readfirstlane(AA.sp.parts[pi].nhalo);
    const int x4 = __builtin_amdgcn_readfirstlane(AA.sp.parts[pi].x4), nx = nown - x4;
    const int64_t own0 = uni64(AA.sp.parts[pi].own0), halo0 = uni64(AA.sp.parts[pi].halo0);
    const int64_t cf = uni64(A.chunk_first[r]);
    // FP64 x (by position slot, the last entry zero) and b of this part
    double* x64 = A.slot_ws64 + (int64_t)blockIdx.x * (3 * (kSpreadZero + 1) + 3 * kSpreadNodes);
    double* b64 = x64 + 3 * (kSpreadZero + 1);
    int parity = 0;

    // exchange slots of the own nodes (low half, 0xffff: none) and the halo's
    // (high half); publish: z of a node other parts hold
    static_assert(HN == SN, "packed slots");
    uint32_t xh[SN];
    auto publish = [&](int s, const float* z) __attribute__((always_inline)) {
        if ((xh[s] & 0xffffu) != 0xffffu) {
            u64* p = xbuf + (tm.tag & 1) * half + (xh[s] & 0xffffu);
            put_word(p, tm.tag, __float_as_uint(z[0]));
            put_word(p + max_x, tm.tag, __float_as_uint(z[1]));
            put_word(p + 2 * max_x, tm.tag, __float_as_uint(z[2]));
        }
    };
    // The exchange of tag tm.tag: the team's totals of N sums (the same in
    // every member) and, on request, z of the halo (each thread its own).  Two barriers; false when a
    // poll gave up.
    auto exchange = [&](auto& v, bool halo) __attribute__((always_inline)) -> bool {
        constexpr int N = sizeof(v) / sizeof(double);
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        const int lane = t & 63, limit = AA.sp.spin_limit;
        if (N == 2) {
            double x = halves_xor32(v[0], v[N - 1]);
            x = add_xor16(x);
            x += dpp_mov<kDppRor8>(x);
            x += dpp_mov<kDppRor4>(x);
            x += dpp_mov<kDppXor2>(x);
            x += dpp_mov<kDppXor1>(x);
            if ((lane & 31) == 0) red.v[parity][lane >> 5][wave] = x;
        } else {
#pragma unroll
            for (int q = 0; q < N; ++q) v[q] = wave_sum(v[q]);
            if (lane == 0)
                for (int q = 0; q < N; ++q) red.v[parity][q][wave] = v[q];
        }
        __syncthreads();
        u64* const words = words_of(tm.tag);
        int polls = 1;
        bool ok = true;
        if (wave == 0) {
            if (lane < N) {
                const double x = sum_in_order<NW>(red.v[parity][lane]);
                put_word(words + 2 * (N * rank + lane), tm.tag, (unsigned)__double2loint(x));
                put_word(words + 2 * (N * rank + lane) + 1, tm.tag, (unsigned)__double2hiint(x));
            }
            if (lane < N * k) {   // (k <= 16)
                const u64* p = words + 2 * lane;
                u64 lo = get_word(p), hi = get_word(p + 1);
                while (!(tagged(lo, tm.tag) && tagged(hi, tm.tag)) && polls++ < limit) {
                    lo = get_word(p);
                    hi = get_word(p + 1);
                }
                ok = tagged(lo, tm.tag) && tagged(hi, tm.tag);
                red.sum[parity][lane % N][lane / N] = __hiloint2double((int)(unsigned)hi, (int)(unsigned)lo);
            }
        }
        if (halo) {
#pragma unroll
            for (int u = 0; u < HN; ++u)
                if (xh[u] < 0xffff0000u) {
                    const u64* p = xbuf + (tm.tag & 1) * half + (xh[u] >> 16);
                    u64 x = get_word(p), y = get_word(p + max_x), z = get_word(p + 2 * max_x);
                    while (!(tagged(x, tm.tag) && tagged(y, tm.tag) && tagged(z, tm.tag)) && polls++ < limit) {
                        x = get_word(p);
                        y = get_word(p + max_x);
                        z = get_word(p + 2 * max_x);
                    }
                    ok = ok && tagged(x, tm.tag) && tagged(y, tm.tag) && tagged(z, tm.tag);
                    hz[t + T * u] = f32x3{__uint_as_float((unsigned)x), __uint_as_float((unsigned)y), __uint_as_float((unsigned)z)};
                }
        }
        if (!ok) red.bad = 1;
        __syncthreads();
        // row q of the wave adds the members' parts of sum q (the same tree in
        // every member)
        {
            const int q = lane >> 4, p = lane & 15;
            double x = q < N && p < k ? red.sum[parity][q < N ? q : 0][p] : 0.0;
            x += dpp_mov<kDppRor8>(x);
            x += dpp_mov<kDppRor4>(x);
            x += dpp_mov<kDppXor2>(x);
            x += dpp_mov<kDppXor1>(x);
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = readlane_d(x, 16 * i);
        }
        parity ^= 1;
        return __builtin_amdgcn_readfirstlane(red.bad) == 0;
    };

    // right-hand side (FP64) and x = 0
    double one[1], two[2];
    {
        double bb = 0.0;
        asm volatile("" : "+v"(bb));
        double F[9], G[9];
        for (int q = 0; q < 9; ++q) F[q] = A.F[9 * r + q];
        if (!TAN)
            for (int q = 0; q < 9; ++q) G[q] = A.gsigma[9 * r + q];
#pragma unroll 1
        for (int s = tid; s < nown; s += T) {
            double b[3];
            rhs_node<TAN>(A, c, AA.sp.own[own0 + s], kk, ll, F, G, b);
            for (int p = 0; p < 3; ++p) {
                b64[3 * s + p] = b[p];
                x64[3 * s + p] = 0.0;
            }
            bb += b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
        }
        for (int s = tid; s < 3 * nhalo; s += T) x64[3 * kSpreadNodes + s] = 0.0;
        if (tid < 3) x64[3 * kSpreadZero + tid] = 0.0;
        one[0] = bb;
    }
    ++tm.tag;
    if (!exchange(one, false)) return false;
    const double bb = one[0];

    // records, blocks and extra records on chip (read once per task)
    float zf = 0.f;
    asm volatile("" : "+v"(zf));
    float rx[SN][4], ry[SN][4], rz_[SN][4], rc[SN][4], rg[SN][4];
    uint32_t ro[SN][2];   // LDS byte offsets / 8 of the other ends, two per word
    float Pb[SN][6];
    int degw[SN];         // the wave's largest degree of the slot
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        const int i = tid + T * s;
        float4 p0 = make_float4(zf, zf, zf, zf), p1 = p0;
        uint32_t o4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            rx[s][u] = ry[s][u] = rz_[s][u] = rc[s][u] = rg[s][u] = zf;
            o4[u] = 2u * kSpreadZero;
        }
        xh[s] = 0xffffffffu;
        int deg = 0;
        if (i < nown) {
            const int a = AA.sp.own[own0 + i];
            xh[s] = 0xffff0000u | (AA.sp.xslot[own0 + i] & 0xffff);
            p0 = A.precond[2 * (c.a0 + a)];
            p1 = A.precond[2 * (c.a0 + a) + 1];
            const int64_t e0 = c.incoff[a], rec = A.chunk_rec[cf + (a >> 6)] + (a & 63);
            deg = (int)(c.incoff[a + 1] - e0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (u < deg) {
                    const float4 ra = A.recA[rec + 64 * u];
                    rx[s][u] = ra.x; ry[s][u] = ra.y; rz_[s][u] = ra.z;
                    rg[s][u] = __int_as_float(A.recB[rec + 64 * u].y);
                    rc[s][u] = ra.w - rg[s][u];
                    o4[u] = 2u * AA.sp.oslot[e0 + u];
                }
#pragma unroll 1
            for (int u = 4; u < deg; ++u) {
                float4 ra = A.recA[rec + 64 * u];
                const int g = A.recB[rec + 64 * u].y;
                ra.w -= __int_as_float(g);
                XA[(u - 4) * nx + (i - x4)] = ra;
                XB[(u - 4) * nx + (i - x4)] = make_int2((int)AA.sp.oslot[e0 + u] | deg << 16, g);
            }
        }
        ro[s][0] = o4[0] | o4[1] << 16;
        ro[s][1] = o4[2] | o4[3] << 16;
        Pb[s][0] = p0.x; Pb[s][1] = p0.y; Pb[s][2] = p0.z; Pb[s][3] = p0.w; Pb[s][4] = p1.x; Pb[s][5] = p1.y;
        degw[s] = __builtin_amdgcn_readfirstlane((int)__float_as_uint(wave_max_nonneg(__uint_as_float((unsigned)deg))));
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < HN; ++u) {
        const int i = tid + T * u;
        if (i < nhalo) xh[u] = (xh[u] & 0xffffu) | (uint32_t)AA.sp.halo_xslot[halo0 + i] << 16;
    }
    float P[SN][3], R[SN][3], Q[SN][3], D[SN][3];
    const char* zb = reinterpret_cast<const char*>(zl);

    int status = ST_CONVERGED;
    double cgt = A.cg_tol;
    asm volatile("" : "+v"(cgt));
    const double tol2 = uniformd(cgt * cgt);
    const int64_t maxit = A.cg_max > 0 ? A.cg_max : 6 * c.nf + 100;
    int64_t it_total = 0;
    bool done = !(bb > 0.0);
    for (int outer = 0; outer < 8 && !done; ++outer) {
        asm volatile("" : "+v"(tid));
        // FP64 residual of the FP64 solution (x64 of own and halo nodes are
        // this part's own, complete: barrier above); d = 0, p = z = P r
        two[0] = two[1] = 0.0;
        ++tm.tag;
#pragma unroll
        for (int s = 0; s < SN; ++s) {
            const int i = tid + T * s;
            double z0 = 0.0;
            asm volatile("" : "+v"(z0));
            double ra[3] = {z0, z0, z0};
            if (i < nown) {
                for (int p = 0; p < 3; ++p) ra[p] = b64[3 * i + p];
                if (outer > 0) {
                    const int a = AA.sp.own[own0 + i];
                    const double xa[3] = {x64[3 * i], x64[3 * i + 1], x64[3 * i + 2]};
#pragma unroll 1
                    for (int64_t e = c.incoff[a]; e < c.incoff[a + 1]; ++e) {
                        const double* xo = x64 + 3 * (int)AA.sp.oslot[e];
                        double w3[3];
                        apply_B64(c.par64 + 6 * (int64_t)(A.net.inc[e] & 0x7fffffffu), xa[0] - xo[0], xa[1] - xo[1], xa[2] - xo[2],
                                  w3[0], w3[1], w3[2]);
                        for (int p = 0; p < 3; ++p) ra[p] -= w3[p];
                    }
                }
            }
            for (int p = 0; p < 3; ++p) {
                R[s][p] = (float)ra[p];
                D[s][p] = Q[s][p] = 0.f;
            }
            two[0] += ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2];
            apply_block_yxz(Pb[s], R[s], P[s]);
            publish(s, P[s]);
            two[1] += (double)R[s][0] * P[s][0] + (double)R[s][1] * P[s][1] + (double)R[s][2] * P[s][2];
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!exchange(two, true)) return false;
        const double rr = two[0];
        double rz = two[1];
        if (rr <= tol2 * bb) {
            done = true;
            break;
        }
        if (it_total >= maxit) {
            status = ST_CG_MAXITER;
            break;
        }
        // inner preconditioned CG, as cg_chip_task
        double drop = 1e-6;
        asm volatile("" : "+s"(drop));
        const double rr0 = uniformd(drop * rr);
        f32x3* const zh = reinterpret_cast<f32x3*>(zl) + kSpreadNodes;
#pragma unroll
        for (int u = 0; u < HN; ++u)
            if (T * u + wave64 < nhalo) {
                zh[tid + T * u] = hz[tid + T * u];
                dh[tid + T * u] = f32x3{zf, zf, zf};
            }
        for (;;) {
            if (it_total >= maxit) break;
            ++it_total;
            asm volatile("" : "+v"(tid));
#pragma unroll
            for (int s = 0; s < SN; ++s) asm volatile("" : "+v"(ro[s][0]), "+v"(ro[s][1]), "+v"(xh[s]));
#pragma unroll
            for (int s = 0; s < SN; ++s) *(f32x3*)&zl[tid + T * s] = f32x3{P[s][0], P[s][1], P[s][2]};
            __syncthreads();
            double pq = 0.0;
#pragma unroll
            for (int s = 0; s < SN; ++s) {
                if (T * s + wave64 < nown) {
                    f32x3 po[4];
                    float q[3] = {0.f, 0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        po[u] = *(const f32x3*)(zb + 8u * ((u & 1) ? ro[s][u >> 1] >> 16 : ro[s][u >> 1] & 0xffffu));
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        add_record(rx[s][u], ry[s][u], rz_[s][u], rc[s][u], rg[s][u], P[s], po[u], q);
                    if (degw[s] > 4) {
                        const int i = tid + T * s - x4;
                        if (i >= 0 && i < nx) {
                            int2 b = XB[i];
                            const int extra = (b.x >> 16) - 4;
#pragma unroll 1
                            for (int j = 0; j < extra; ++j) {
                                const float4 ra = XA[j * nx + i];
                                if (j > 0) b = XB[j * nx + i];
                                add_record(ra.x, ra.y, ra.z, ra.w, __int_as_float(b.y), P[s], *(const f32x3*)&zl[b.x & 0xffff], q);
                            }
                        }
                    }
                    for (int p = 0; p < 3; ++p) Q[s][p] = q[p];
                    pq += (double)P[s][0] * q[0] + (double)P[s][1] * q[1] + (double)P[s][2] * q[2];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            ++tm.tag;
            one[0] = pq;
            if (!exchange(one, false)) return false;
            pq = one[0];
            if (!(pq > 0.0)) {
                status = ST_CG_INDEFINITE;
                done = true;
                break;
            }
            const float af = uniform((float)(rz / pq));
            two[0] = two[1] = 0.0;
            ++tm.tag;
            float Z[SN][3];
#pragma unroll
            for (int s = 0; s < SN; ++s) {
                for (int p = 0; p < 3; ++p) {
                    D[s][p] = fmaf(af, P[s][p], D[s][p]);
                    R[s][p] = fmaf(-af, Q[s][p], R[s][p]);
                }
                apply_block_yxz(Pb[s], R[s], Z[s]);
                publish(s, Z[s]);
                two[0] += (double)R[s][0] * R[s][0] + (double)R[s][1] * R[s][1] + (double)R[s][2] * R[s][2];
                two[1] += (double)R[s][0] * Z[s][0] + (double)R[s][1] * Z[s][1] + (double)R[s][2] * Z[s][2];
            }
#pragma unroll
            for (int u = 0; u < HN; ++u)
                if (T * u + wave64 < nhalo) {
                    const f32x3 p = zh[tid + T * u], d = dh[tid + T * u];
                    dh[tid + T * u] = f32x3{fmaf(af, p.x, d.x), fmaf(af, p.y, d.y), fmaf(af, p.z, d.z)};
                }
            if (!exchange(two, true)) return false;
            const double rn = two[0], rzn = two[1];
            if (rn <= rr0 || rn <= 0.25 * tol2 * bb) break;
            const float bf = uniform((float)(rzn / rz));
            rz = rzn;
#pragma unroll
            for (int s = 0; s < SN; ++s)
                for (int p = 0; p < 3; ++p) P[s][p] = fmaf(bf, P[s][p], Z[s][p]);
#pragma unroll
            for (int u = 0; u < HN; ++u)
                if (T * u + wave64 < nhalo) {
                    const f32x3 p = zh[tid + T * u], z = hz[tid + T * u];
                    zh[tid + T * u] = f32x3{fmaf(bf, p.x, z.x), fmaf(bf, p.y, z.y), fmaf(bf, p.z, z.z)};
                }
        }
        // x += d, of the own and of the halo nodes
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int s = 0; s < SN; ++s) {
            const int i = tid + T * s;
            if (i < nown)
                for (int p = 0; p < 3; ++p) x64[3 * i + p] += (double)D[s][p];
        }
#pragma unroll 1
        for (int i = tid; i < nhalo; i += T) {
            const f32x3 d = dh[i];
            double* x = x64 + 3 * (kSpreadNodes + i);
            x[0] += (double)d.x; x[1] += (double)d.y; x[2] += (double)d.z;
        }
        __syncthreads();
        if (outer == 7 && !done && status == ST_CONVERGED) status = ST_CG_MAXITER;
    }

    // assembly over the part's boundary nodes (x64 complete: barrier above, or
    // no update since the first exchange)
    double tot[9];
    {
        double acc[9];
        for (int p = 0; p < 9; ++p) acc[p] = 0.0;
        double F[9], G[9];
        for (int q = 0; q < 9; ++q) F[q] = A.F[9 * r + q];
        if (!TAN)
            for (int q = 0; q < 9; ++q) G[q] = A.gsigma[9 * r + q];
        const int64_t bp0 = uni64(AA.sp.parts[pi].bnd0);
        const int nbnd = __builtin_amdgcn_readfirstlane(AA.sp.parts[pi].nbnd);
#pragma unroll 1
        for (int q = tid; q < nbnd; q += T) {
            const int64_t bn = c.b0 + AA.sp.bnd[bp0 + q];
#pragma unroll 1
            for (int64_t e = A.net.binc_off[bn]; e < A.net.binc_off[bn + 1]; ++e) {
                const uint32_t w = A.net.binc[e];
                assembly_end<TAN>(A, c, F, G, kk, ll, (int64_t)(w & 0x7fffffffu), (w >> 31) ? 0 : 1,
                                  x64 + 3 * (int)AA.sp.bslot[e], acc);
            }
        }
#pragma unroll
        for (int p = 0; p < 9; p += 3) {
            double three[3] = {acc[p], acc[p + 1], acc[p + 2]};
            ++tm.tag;
            if (!exchange(three, false)) return false;
            for (int q = 0; q < 3; ++q) tot[p + q] = three[q];
        }
    }
    ++tm.tag;
    const bool all = team_done(AA.sp, red, tm, words_of(tm.tag));
    if (rank == 0 && all && threadIdx.x == 0) {
        assembly_write<TAN>(A, r, col, tot, status, it_total);
        A.done[tm.task] = 1;
    }
    return all;
}

template <bool TAN>
__global__ __launch_bounds__(kCgT) __attribute__((amdgpu_waves_per_eu(2))) void cg_spread_kernel(SpreadCgArgs)
{
    __shared__ float4 zl[kSpreadZero + 1];   // p: own, halo, zero
    __shared__ f32x3 dh[kSpreadNodes];       // correction of the halo
    __shared__ f32x3 hz[kSpreadNodes];       // z of the halo
    __shared__ float4 XA[kSpreadExtra];      // records beyond the fourth: (n, k_t/L0 - T/l)
    __shared__ int2 XB[kSpreadExtra];        // (slot of the other end | degree << 16, bits of T/l)
    __shared__ CgSpreadRed red;
    auto& AA = *kernel_args<SpreadCgArgs>();
    if (threadIdx.x == 0) {
        red.bad = 0;
        zl[kSpreadZero] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    Team tm;
    while (team_take(AA.sp, red, tm))
        if (!cg_spread_task<TAN>(*kernel_args<SpreadCgArgs>(), tm, zl, dh, hz, XA, XB, red)) break;
}

// ------------------------------------------------------------------ resident tasks
// One workgroup of T threads per task, for the RVEs whose records no longer fit
// the registers; thread tid owns free nodes tid + T k (k < SN), so wavefront w
// owns ELL chunks w + (T/64) k.  The residual, the product, the correction and
// the inverse blocks stay in registers, p (which the matrix-free product
// gathers) lives in LDS (PL, the only layout), and the records are read from L2,
// those of the next slot while the current one is worked on.
//
// Eight nodes in 512 threads, with the sums in the order of 1024 threads (as
// cg_chip_task).  Four nodes in 1024 threads left no registers for the
// correction, the blocks and the next records, and read the first two from
// global memory as well.  Microseconds per iteration and column, four in 1024 ->
// eight in 512: 8.3 -> 6.6 at 2532 free nodes alone, 10.4 -> 7.6 on a full chip;
// 11.0 -> 8.5 and 16 -> 10.2 at 4090.
//
// The inner solve is plain preconditioned CG with a fresh product q = K p
// every iteration: three workgroup barriers per iteration (p exchanged, p.q
// summed, (r,r) and (r,z) summed).  Recurrence forms with one reduction (the
// Chronopoulos-Gear update of q) lose the sign of p.Kp to FP32 cancellation
// on these ill-conditioned systems.
template <bool TAN, int T, int SN, bool PL>
__device__ void cg_res_task(TanArgs& A, int r, int col, float4* zl, CgRed& red)
{
    static_assert(PL, "p in LDS");
    constexpr int NW = T / 64, H = T == 512 ? 2 : 1;   // H partial sums per thread (chip_sum)
    // thread id made opaque per task: otherwise the compiler hoists every
    // per-thread address of every slot out of the persistent task loop and
    // keeps them live (spilled) across the whole kernel
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (__builtin_amdgcn_readfirstlane(A.solve_status[r]) != 0) {
        no_state<TAN>(A, r, col, tid);
        return;
    }
    const Ctx c = make_ctx(A, r);
    const int64_t nf = c.nf;
    const int kk = col / 3, ll = col % 3;
    const float4* Pc = A.precond + 2 * c.a0;
    const int64_t cf = uni64(A.chunk_first[r]);
    const int64_t S = A.slot_nodes;
    double* x64 = A.slot_ws64 + (int64_t)blockIdx.x * 8 * S;   // x, b (3 S each)
    double* b64 = x64 + 3 * S;

    // ELL chunk of each slot (uniform over the wavefront); width 0 past the
    // end.  Record offsets are 32-bit, relative to the RVE's first record.
    const int64_t rec0 = uni64(A.chunk_rec[cf]);
    const float4* recA = A.recA + rec0;
    const int2* recB = A.recB + rec0;
    int rb[SN];
    int wd[SN];
#pragma unroll
    for (int k = 0; k < SN; ++k) {
        const int64_t ch = wave + NW * k;
        rb[k] = 0;
        wd[k] = 0;
        if (64 * ch < nf) {
            const int64_t c0 = uni64(A.chunk_rec[cf + ch]);
            wd[k] = (int)((uni64(A.chunk_rec[cf + ch + 1]) - c0) >> 6);
            rb[k] = (int)(c0 - rec0);
        }
    }
    int parity = 0;

    // right-hand side (FP64)
    double b2[2] = {0.0, 0.0};
    {
        double F[9], G[9];
        for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
        if (!TAN)
            for (int k = 0; k < 9; ++k) G[k] = A.gsigma[9 * r + k];
#pragma unroll 1
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            if (a < nf) {
                double b[3];
                rhs_node<TAN>(A, c, a, kk, ll, F, G, b);
                for (int p = 0; p < 3; ++p) {
                    b64[3 * a + p] = b[p];
                    x64[3 * a + p] = 0.0;
                }
                const double bn = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
                if (k % H)
                    b2[1] += bn;
                else
                    b2[0] += bn;
            }
        }
        if (tid < 3) x64[3 * nf + tid] = 0.0;
    }
    const double bb = chip_sum<NW, H>(red, parity, tid, b2);
    parity ^= 1;

    float R[SN][3], Q[SN][3], D[SN][3], Pb[SN][6];
#pragma unroll
    for (int k = 0; k < SN; ++k) {
        const int64_t a = tid + T * k;
        float4 p0 = make_float4(0.f, 0.f, 0.f, 0.f), p1 = p0;
        if (a < nf) {
            p0 = Pc[2 * a];
            p1 = Pc[2 * a + 1];
        }
        Pb[k][0] = p0.x; Pb[k][1] = p0.y; Pb[k][2] = p0.z; Pb[k][3] = p0.w; Pb[k][4] = p1.x; Pb[k][5] = p1.y;
    }
    auto own_p = [&](int k) __attribute__((always_inline)) -> f32x3 { return *(const f32x3*)&zl[tid + T * k]; };
    int status = ST_CONVERGED;
    // per-task copy: a kernel-lifetime value would be kept live across tasks
    double cgt = A.cg_tol;
    asm volatile("" : "+v"(cgt));
    const double tol2 = uniformd(cgt * cgt);
    const int64_t maxit = A.cg_max > 0 ? A.cg_max : 6 * nf + 100;
    int64_t it_total = 0;
    bool done = !(bb > 0.0);
    for (int outer = 0; outer < 8 && !done; ++outer) {
        // thread id opaque per phase: no per-thread address is hoisted out of
        // the loops and kept live across them
        asm volatile("" : "+v"(tid));
        // FP64 residual of the FP64 solution (x64 complete: barrier above);
        // d = 0, p = z = P r
        double rr2[2] = {0.0, 0.0}, rz2[2] = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            double ra[3] = {0.0, 0.0, 0.0};
            if (a < nf) residual_node(A, c, a, x64, b64, outer == 0, ra);
            for (int p = 0; p < 3; ++p) {
                R[k][p] = (float)ra[p];
                Q[k][p] = D[k][p] = 0.f;
            }
            rr2[k % H] += ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2];
            float z[3];
            apply_block(Pb[k], R[k], z);
            rz2[k % H] += (double)R[k][0] * z[0] + (double)R[k][1] * z[1] + (double)R[k][2] * z[2];
            *(f32x3*)&zl[tid + T * k] = f32x3{z[0], z[1], z[2]};
            __builtin_amdgcn_sched_barrier(0);
        }
        chip_sum2<NW, H>(red, parity, tid, rr2, rz2);
        parity ^= 1;
        const double rr = rr2[0];
        double rz = rz2[0];
        if (rr <= tol2 * bb) {
            done = true;
            break;
        }
        if (it_total >= maxit) {
            status = ST_CG_MAXITER;
            break;
        }
        // inner preconditioned CG (FP32 vectors, p exchanged through LDS):
        // q = K p, alpha = rz / p.q, d += alpha p, r -= alpha q, z = P r,
        // beta = r.z / rz, p = z + beta p
        const double rr0 = rr;
        for (;;) {
            if (it_total >= maxit) break;
            ++it_total;
            asm volatile("" : "+v"(tid));
            __syncthreads();
            double pq2[2] = {0.0, 0.0};
            // the first four records of a slot (chunk widths are multiples of 4)
            float4 nA[2][4];
            int2 ob[2][4];
            const uint32_t ln = tid & 63;   // (an offset from a scalar base)
            auto rec_a = [&](int i) __attribute__((always_inline)) { return *(const float4*)((const char*)(recA + i) + 16 * ln); };
            auto rec_b = [&](int i) __attribute__((always_inline)) { return *(const int2*)((const char*)(recB + i) + 8 * ln); };
            auto load = [&](int k, int j) __attribute__((always_inline)) {
                if (wd[k] > 0)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        nA[j][u] = rec_a(rb[k] + 64 * u);
                        ob[j][u] = rec_b(rb[k] + 64 * u);
                    }
            };
            load(0, 0);
#pragma unroll
            for (int k = 0; k < SN; ++k) {
                if (k + 1 < SN) load(k + 1, (k + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
                if (wd[k] > 0) {
                    const int j = k & 1;
                    const f32x3 pk = own_p(k);
                    const float pv[3] = {pk.x, pk.y, pk.z};
                    float q[3] = {0.f, 0.f, 0.f};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float g = __int_as_float(ob[j][u].y);
                        add_record(nA[j][u].x, nA[j][u].y, nA[j][u].z, nA[j][u].w - g, g, pv, *(const f32x3*)&zl[ob[j][u].x], q);
                    }
#pragma unroll 1
                    for (int s0 = 4; s0 < wd[k]; ++s0) {
                        const float4 ra = rec_a(rb[k] + 64 * s0);
                        const int2 o = rec_b(rb[k] + 64 * s0);
                        const float g = __int_as_float(o.y);
                        add_record(ra.x, ra.y, ra.z, ra.w - g, g, pv, *(const f32x3*)&zl[o.x], q);
                    }
                    for (int p = 0; p < 3; ++p) Q[k][p] = q[p];
                    pq2[k % H] += (double)pk.x * q[0] + (double)pk.y * q[1] + (double)pk.z * q[2];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            const double pq = chip_sum<NW, H>(red, parity, tid, pq2);
            parity ^= 1;
            if (!(pq > 0.0)) {
                status = ST_CG_INDEFINITE;
                done = true;
                break;
            }
            const float af = (float)(rz / pq);
            double rn2[2] = {0.0, 0.0}, rzn2[2] = {0.0, 0.0};
            float (&Z)[SN][3] = Q;   // (q is done with)
#pragma unroll
            for (int k = 0; k < SN; ++k)
                if (k == 0 || wd[k] > 0) {
                    const f32x3 pk = own_p(k);
                    D[k][0] = fmaf(af, pk.x, D[k][0]);
                    D[k][1] = fmaf(af, pk.y, D[k][1]);
                    D[k][2] = fmaf(af, pk.z, D[k][2]);
                    for (int p = 0; p < 3; ++p) R[k][p] = fmaf(-af, Q[k][p], R[k][p]);
                    apply_block(Pb[k], R[k], Z[k]);
                    rn2[k % H] += (double)R[k][0] * R[k][0] + (double)R[k][1] * R[k][1] + (double)R[k][2] * R[k][2];
                    rzn2[k % H] += (double)R[k][0] * Z[k][0] + (double)R[k][1] * Z[k][1] + (double)R[k][2] * Z[k][2];
                    __builtin_amdgcn_sched_barrier(0);
                }
            chip_sum2<NW, H>(red, parity, tid, rn2, rzn2);
            parity ^= 1;
            const double rn = rn2[0], rzn = rzn2[0];
            if (rn <= 1e-6 * rr0 || rn <= 0.25 * tol2 * bb) break;
            const float bf = (float)(rzn / rz);
            rz = rzn;
#pragma unroll
            for (int k = 0; k < SN; ++k)
                if (k == 0 || wd[k] > 0) {
                    const f32x3 pk = own_p(k);
                    *(f32x3*)&zl[tid + T * k] = f32x3{fmaf(bf, pk.x, Z[k][0]), fmaf(bf, pk.y, Z[k][1]), fmaf(bf, pk.z, Z[k][2])};
                }
        }
        // x += d
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            if (a < nf) {
                for (int p = 0; p < 3; ++p) x64[3 * a + p] += (double)D[k][p];
            }
        }
        __syncthreads();
        if (outer == 7 && !done && status == ST_CONVERGED) status = ST_CG_MAXITER;
    }

    // assembly (x64 complete: barrier above, or no update since the RHS sum)
    double acc[9];
    assembly_partial<TAN>(A, c, r, kk, ll, x64, tid, T, acc);
    double tot[9];
#pragma unroll
    for (int p = 0; p < 9; p += 3) {
        double a1 = acc[p], a2 = acc[p + 1], a3 = acc[p + 2];
        block_sum3<NW>(red, parity, a1, a2, a3);
        parity ^= 1;
        tot[p] = a1;
        tot[p + 1] = a2;
        tot[p + 2] = a3;
    }
    if (tid == 0) assembly_write<TAN>(A, r, col, tot, status, it_total);
    __syncthreads();
}

template <bool TAN, int T, int SN, bool PL>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T == 512 ? 2 : 4))) void cg_res_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    extern __shared__ float4 zl[];   // [T * SN + 1]; the last entry stays zero
    __shared__ CgRed red;
    __shared__ int task;
    if (threadIdx.x == 0) zl[T * SN] = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int per = TAN ? 9 : 1;
    const int64_t n_tasks = A.n_order * per;
    for (;;) {
        if (threadIdx.x == 0) task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(task);
        __syncthreads();
        if (t >= n_tasks) break;
        cg_res_task<TAN, T, SN, PL>(A, __builtin_amdgcn_readfirstlane(A.order[t / per]), t % per, zl, red);
    }
}

// ------------------------------------------------------------------ blocked tangent tasks
// Tangent only: one workgroup solves the three right-hand sides F_k0, F_k1,
// F_k2 of one column group k together.  Every ELL record is read once per
// iteration for the three products, and every workgroup reduction carries
// the three columns' sums, so one record read and one barrier serve three
// solves.  Per column the arithmetic is that of cg_res_task, in the same
// order and with the same workgroup sums, so each column's result equals
// the per-column kernel's bitwise.  A column whose inner solve has met its
// criterion (or has ended) makes no further update while the others finish
// theirs; then the columns of the round take the refinement step x += d
// together.  p of each column lives in LDS, its correction d in the
// workgroup's global slot, z = P r is recomputed where needed.
constexpr int kBlk = kTanBlkRhs;

struct BlkRed {
    double s[2][2 * kBlk][16];   // per-wavefront partial sums, alternating buffers
};

// Workgroup sums of N values; each value is summed exactly as block_sum3
// sums it (wavefront sum, then the wavefronts in order).
template <int NW, int N>
__device__ __forceinline__ void block_sum_n(BlkRed& red, int parity, double (&v)[N])
{
    static_assert(N <= 2 * kBlk, "too many values");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double w = wave_sum(v[i]);
        if (lane == 0) red.s[parity][i][wave] = w;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double x = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) x += red.s[parity][i][q];
        v[i] = uniformd(x);
    }
}

template <int T, int SN, int BLK_RB>
__device__ void cg_blk_task(TanArgs& A, int r, int grp, float4* zl, BlkRed& red)
{
    constexpr int NW = T / 64;
    constexpr int ZS = T * SN + 1;   // LDS entries of one column's p
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (__builtin_amdgcn_readfirstlane(A.solve_status[r]) != 0) {
        // as no_state, with the opaque thread id (nothing kept live across tasks)
        if (tid == 0) atomicMax(&A.status[r], ST_NO_STATE);
        if (tid < 9) {
            // one double per store (a vector store would keep a NaN tuple live)
#pragma unroll 1
            for (int j = 0; j < kBlk; ++j) {
                double nanv = NAN;
                asm volatile("" : "+v"(nanv));
                A.out[(int64_t)r * 81 + 9 * tid + kBlk * grp + j] = nanv;
            }
        }
        return;
    }
    const Ctx c = make_ctx(A, r);
    const int64_t nf = c.nf;
    const int kk = grp;
    const float4* Pc = A.precond + 2 * c.a0;
    const int64_t cf = uni64(A.chunk_first[r]);
    const int64_t S = A.slot_nodes;
    // slot: x, b (FP64, 3 S each), then d and q = K p (FP32 float4, S each)
    // per column
    double* ws = A.slot_ws64 + (int64_t)blockIdx.x * 10 * kBlk * S;
    auto x64 = [&](int j) __attribute__((always_inline)) { return ws + 6 * S * j; };
    auto b64 = [&](int j) __attribute__((always_inline)) { return ws + 6 * S * j + 3 * S; };
    float4* d32 = reinterpret_cast<float4*>(ws + 6 * S * kBlk);
    float4* q32 = d32 + S * kBlk;
    const int64_t rec0 = uni64(A.chunk_rec[cf]);
    const float4* recA = A.recA + rec0;
    const int2* recB = A.recB + rec0;
    int rb[SN];
    int wd[SN];
#pragma unroll
    for (int k = 0; k < SN; ++k) {
        const int64_t ch = wave + NW * k;
        rb[k] = 0;
        wd[k] = 0;
        if (64 * ch < nf) {
            const int64_t c0 = uni64(A.chunk_rec[cf + ch]);
            wd[k] = (int)((uni64(A.chunk_rec[cf + ch + 1]) - c0) >> 6);
            rb[k] = (int)(c0 - rec0) + lane;
        }
    }
    int parity = 0;

    // right-hand sides (FP64)
    double bb[kBlk];
    {
        double F[9], G[9];
        for (int k = 0; k < 9; ++k) F[k] = A.F[9 * r + k];
#pragma unroll
        for (int j = 0; j < kBlk; ++j) bb[j] = 0.0;
#pragma unroll 1
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            if (a < nf) {
#pragma unroll 1
                for (int j = 0; j < kBlk; ++j) {
                    double b[3];
                    rhs_node<true>(A, c, a, kk, j, F, G, b);
                    for (int p = 0; p < 3; ++p) {
                        b64(j)[3 * a + p] = b[p];
                        x64(j)[3 * a + p] = 0.0;
                    }
                    bb[j] += b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
                }
            }
        }
        if (tid < 3)
            for (int j = 0; j < kBlk; ++j) x64(j)[3 * nf + tid] = 0.0;
    }
    block_sum_n<NW>(red, parity, bb);
    parity ^= 1;

    float R[kBlk][SN][3];
    auto own_p = [&](int j, int k) __attribute__((always_inline)) -> float4 { return zl[ZS * j + tid + T * k]; };
    // inverse block of slot k (reloaded where needed, as in cg_res_task)
    auto pblock = [&](int k, float4& p0, float4& p1) __attribute__((always_inline)) {
        const int64_t a = tid + T * k;
        p0 = make_float4(0.f, 0.f, 0.f, 0.f);
        p1 = p0;
        if (a < nf) {
            const float4* pp = Pc + 2 * a;
            asm volatile("" : "+v"(pp));
            p0 = pp[0];
            p1 = pp[1];
        }
    };
    auto papply = [&](const float4& p0, const float4& p1, const float* v) __attribute__((always_inline)) -> float4 {
        return make_float4(p0.x * v[0] + p0.y * v[1] + p0.z * v[2], p0.y * v[0] + p0.w * v[1] + p1.x * v[2],
                           p0.z * v[0] + p1.x * v[1] + p1.y * v[2], 0.f);
    };
    int status[kBlk];
    int it_total[kBlk];
    // bit j: column j's solve has ended (converged, cap, indefinite) / is in
    // this round's inner solve / took part in this round
    unsigned fin = 0u, act = 0u, in_round = 0u;
    // per-task copy: a kernel-lifetime value would be kept live across tasks
    double cgt = A.cg_tol;
    asm volatile("" : "+v"(cgt));
    const double tol2 = uniformd(cgt * cgt);
    const int64_t maxit = A.cg_max > 0 ? A.cg_max : 6 * nf + 100;
#pragma unroll
    for (int j = 0; j < kBlk; ++j) {
        status[j] = ST_CONVERGED;
        it_total[j] = 0;
        if (!(bb[j] > 0.0)) fin |= 1u << j;
    }
    for (int outer = 0; outer < 8; ++outer) {
        // thread id opaque per phase: no per-thread address of any column is
        // hoisted out of the loops and kept live
        asm volatile("" : "+v"(tid));
        if (fin == (1u << kBlk) - 1u) break;
        // FP64 residuals of the columns still running; d = 0, p = z = P r
        double sums[2 * kBlk];
#pragma unroll
        for (int i = 0; i < 2 * kBlk; ++i) sums[i] = 0.0;
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            float4 p0, p1;
            pblock(k, p0, p1);
#pragma unroll
            for (int j = 0; j < kBlk; ++j) {
                if (fin & (1u << j)) continue;
                double ra[3] = {0.0, 0.0, 0.0};
                if (a < nf) residual_node(A, c, a, x64(j), b64(j), outer == 0, ra);
                for (int p = 0; p < 3; ++p) R[j][k][p] = (float)ra[p];
                sums[j] += ra[0] * ra[0] + ra[1] * ra[1] + ra[2] * ra[2];
                const float4 z = papply(p0, p1, R[j][k]);
                sums[kBlk + j] += (double)R[j][k][0] * z.x + (double)R[j][k][1] * z.y + (double)R[j][k][2] * z.z;
                zl[ZS * j + tid + T * k] = z;
                if (a < nf) d32[S * j + a] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        block_sum_n<NW>(red, parity, sums);
        parity ^= 1;
        double rz[kBlk], rr0[kBlk];
        act = 0u;
#pragma unroll
        for (int j = 0; j < kBlk; ++j) {
            rz[j] = sums[kBlk + j];
            rr0[j] = sums[j];
            if (fin & (1u << j)) continue;
            if (sums[j] <= tol2 * bb[j]) {
                fin |= 1u << j;   // converged
                continue;
            }
            if (it_total[j] >= maxit) {
                status[j] = ST_CG_MAXITER;
                fin |= 1u << j;
                continue;
            }
            act |= 1u << j;
        }
        in_round = act;
        for (;;) {
#pragma unroll
            for (int j = 0; j < kBlk; ++j) {
                if ((act & (1u << j)) && it_total[j] >= maxit) act &= ~(1u << j);
                if (act & (1u << j)) ++it_total[j];
            }
            if (!act) break;
            asm volatile("" : "+v"(tid));
            __syncthreads();
            // q = K p for the active columns: each record read once
            double pq[kBlk];
#pragma unroll
            for (int i = 0; i < kBlk; ++i) pq[i] = 0.0;
#pragma unroll
            for (int k = 0; k < SN; ++k) {
                float sx[kBlk], sy[kBlk], sz[kBlk];
                float px[kBlk], py[kBlk], pz[kBlk];
#pragma unroll
                for (int j = 0; j < kBlk; ++j) {
                    sx[j] = sy[j] = sz[j] = 0.f;
                    const float4 q = (act & (1u << j)) ? own_p(j, k) : make_float4(0.f, 0.f, 0.f, 0.f);
                    px[j] = q.x;
                    py[j] = q.y;
                    pz[j] = q.z;
                }
                constexpr int RB = BLK_RB;
#pragma unroll 1
                for (int s0 = 0; s0 < wd[k]; s0 += RB) {
                    float4 nA[RB];
                    int2 ob[RB];
#pragma unroll
                    for (int u = 0; u < RB; ++u) {
                        nA[u] = recA[rb[k] + 64 * (s0 + u)];
                        ob[u] = recB[rb[k] + 64 * (s0 + u)];
                    }
#pragma unroll
                    for (int j = 0; j < kBlk; ++j) {
                        if (!(act & (1u << j))) continue;
#pragma unroll
                        for (int u = 0; u < RB; ++u) {
                            const float4 po = zl[ZS * j + ob[u].x];
                            const float g = __int_as_float(ob[u].y);
                            const float dx = px[j] - po.x, dy = py[j] - po.y, dz = pz[j] - po.z;
                            const float cn = (nA[u].w - g) * (nA[u].x * dx + nA[u].y * dy + nA[u].z * dz);
                            sx[j] += fmaf(g, dx, cn * nA[u].x);
                            sy[j] += fmaf(g, dy, cn * nA[u].y);
                            sz[j] += fmaf(g, dz, cn * nA[u].z);
                        }
                    }
                }
                const int64_t a = tid + T * k;
#pragma unroll
                for (int j = 0; j < kBlk; ++j) {
                    if (!(act & (1u << j))) continue;
                    if (a < nf) q32[S * j + a] = make_float4(sx[j], sy[j], sz[j], 0.f);
                    pq[j] += (double)px[j] * sx[j] + (double)py[j] * sy[j] + (double)pz[j] * sz[j];
                }
            }
            block_sum_n<NW>(red, parity, pq);
            parity ^= 1;
            float af[kBlk];
#pragma unroll
            for (int j = 0; j < kBlk; ++j) {
                af[j] = 0.f;
                if (!(act & (1u << j))) continue;
                if (!(pq[j] > 0.0)) {
                    status[j] = ST_CG_INDEFINITE;
                    fin |= 1u << j;
                    act &= ~(1u << j);
                    continue;
                }
                af[j] = (float)(rz[j] / pq[j]);
            }
            double rs[2 * kBlk];
#pragma unroll
            for (int i = 0; i < 2 * kBlk; ++i) rs[i] = 0.0;
#pragma unroll
            for (int k = 0; k < SN; ++k) {
                const int64_t a = tid + T * k;
                float4 p0, p1;
                pblock(k, p0, p1);
#pragma unroll
                for (int j = 0; j < kBlk; ++j) {
                    if (!(act & (1u << j))) continue;
                    const float4 pk = own_p(j, k);
                    if (a < nf) {
                        float4 d = d32[S * j + a];
                        d.x = fmaf(af[j], pk.x, d.x);
                        d.y = fmaf(af[j], pk.y, d.y);
                        d.z = fmaf(af[j], pk.z, d.z);
                        d32[S * j + a] = d;
                    }
                    const float4 qa = a < nf ? q32[S * j + a] : make_float4(0.f, 0.f, 0.f, 0.f);
                    R[j][k][0] = fmaf(-af[j], qa.x, R[j][k][0]);
                    R[j][k][1] = fmaf(-af[j], qa.y, R[j][k][1]);
                    R[j][k][2] = fmaf(-af[j], qa.z, R[j][k][2]);
                    const float4 z = papply(p0, p1, R[j][k]);
                    rs[j] += (double)R[j][k][0] * R[j][k][0] + (double)R[j][k][1] * R[j][k][1] +
                             (double)R[j][k][2] * R[j][k][2];
                    rs[kBlk + j] += (double)R[j][k][0] * z.x + (double)R[j][k][1] * z.y + (double)R[j][k][2] * z.z;
                }
            }
            block_sum_n<NW>(red, parity, rs);
            parity ^= 1;
            float bf[kBlk];
#pragma unroll
            for (int j = 0; j < kBlk; ++j) {
                bf[j] = 0.f;
                if (!(act & (1u << j))) continue;
                if (rs[j] <= 1e-6 * rr0[j] || rs[j] <= 0.25 * tol2 * bb[j]) {
                    act &= ~(1u << j);   // inner solve of this round done
                    continue;
                }
                bf[j] = (float)(rs[kBlk + j] / rz[j]);
                rz[j] = rs[kBlk + j];
            }
#pragma unroll
            for (int k = 0; k < SN; ++k) {
                float4 p0, p1;
                if (!act) break;
                pblock(k, p0, p1);
#pragma unroll
                for (int j = 0; j < kBlk; ++j) {
                    if (!(act & (1u << j))) continue;
                    const float4 z = papply(p0, p1, R[j][k]);
                    const float4 pk = own_p(j, k);
                    zl[ZS * j + tid + T * k] =
                        make_float4(fmaf(bf[j], pk.x, z.x), fmaf(bf[j], pk.y, z.y), fmaf(bf[j], pk.z, z.z), 0.f);
                }
            }
        }
        // x += d for the columns of this round
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int k = 0; k < SN; ++k) {
            const int64_t a = tid + T * k;
            if (a < nf) {
#pragma unroll
                for (int j = 0; j < kBlk; ++j) {
                    if (!(in_round & (1u << j))) continue;
                    const float4 d = d32[S * j + a];
                    x64(j)[3 * a] += (double)d.x;
                    x64(j)[3 * a + 1] += (double)d.y;
                    x64(j)[3 * a + 2] += (double)d.z;
                }
            }
        }
        __syncthreads();
        if (outer == 7)
#pragma unroll
            for (int j = 0; j < kBlk; ++j)
                if (!(fin & (1u << j)) && status[j] == ST_CONVERGED) status[j] = ST_CG_MAXITER;
    }

    // assembly of each column
#pragma unroll 1
    for (int j = 0; j < kBlk; ++j) {
        asm volatile("" : "+v"(tid));
        double acc[9];
        assembly_partial<true>(A, c, r, kk, j, x64(j), tid, T, acc);
        double tot[9];
#pragma unroll
        for (int p = 0; p < 9; p += 3) {
            double v3[3] = {acc[p], acc[p + 1], acc[p + 2]};
            block_sum_n<NW>(red, parity, v3);
            parity ^= 1;
            tot[p] = v3[0];
            tot[p + 1] = v3[1];
            tot[p + 2] = v3[2];
        }
        if (tid == 0) assembly_write<true>(A, r, kBlk * grp + j, tot, status[j], it_total[j]);
    }
    __syncthreads();
}

// Waves per SIMD WPE (registers 512 / WPE): the three columns' residuals
// stay in registers.
template <int T, int SN, int WPE>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(WPE))) void cg_blk_kernel(TangentArgs)
{
    TanArgs& A = *kernel_args<TangentArgs>();
    extern __shared__ float4 zl[];   // [kBlk][T * SN + 1]; entries past an RVE's nodes stay zero
    __shared__ BlkRed red;
    __shared__ int task;
    constexpr int ZS = T * SN + 1;
    if (threadIdx.x < kBlk) zl[ZS * threadIdx.x + T * SN] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int64_t n_tasks = A.n_order * kBlk;
    for (;;) {
        if (threadIdx.x == 0) task = atomicAdd(A.queue, 1);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(task);
        __syncthreads();
        if (t >= n_tasks) break;
        cg_blk_task<T, SN, WPE >= 4 ? 1 : 2>(A, __builtin_amdgcn_readfirstlane(A.order[t / kBlk]), t % kBlk, zl, red);
    }
}

__global__ void zero_status(int32_t* st, unsigned long long* it, int64_t n)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) {
        st[i] = 0;
        it[i] = 0;
    }
}

template <bool TAN, int T, int SN, bool PL>
const void* res_fn()
{
    return (const void*)cg_res_kernel<TAN, T, SN, PL>;
}

const void* res_kernel(int v, bool vjp)
{
    switch (v) {
    case 0: return vjp ? (const void*)cg_chip_kernel<false, 256, 2> : (const void*)cg_chip_kernel<true, 256, 2>;
    case 1: return vjp ? (const void*)cg_chip_kernel<false, 512, 2> : (const void*)cg_chip_kernel<true, 512, 2>;
    case 2: return vjp ? (const void*)cg_chip_kernel<false, 512, 4> : (const void*)cg_chip_kernel<true, 512, 4>;
    case 3: return vjp ? res_fn<false, 512, 8, true>() : res_fn<true, 512, 8, true>();
    default: return vjp ? res_fn<false, 1024, 8, true>() : res_fn<true, 1024, 8, true>();
    }
}

}  // namespace

const TangentVariant kTanRes[kNumTanRes] = {{256, 2}, {512, 2}, {512, 4}, {512, 8}, {1024, 8}};

hipError_t launch_tangent_prep(const TangentArgs& a, hipStream_t s)
{
    if (a.n_rve <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_status, dim3((unsigned)((a.n_rve + 255) / 256)), dim3(256), 0, s, a.status, a.iters, a.n_rve);
    if (a.build_static) hipLaunchKernelGGL(ell_build_kernel, dim3((unsigned)a.n_rve), dim3(kOpsThreads), 0, s, a);
    hipLaunchKernelGGL(fiber_ops_kernel, dim3((unsigned)a.n_rve), dim3(kOpsThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tangent_stream(const TangentArgs& a, int threads, int grid, hipStream_t s)
{
    if (a.n_order <= 0) return hipSuccess;
    if (threads == 64) {
        if (a.mode == 0)
            hipLaunchKernelGGL((cg_stream_kernel<true, 64>), dim3(grid), dim3(64), 0, s, a);
        else
            hipLaunchKernelGGL((cg_stream_kernel<false, 64>), dim3(grid), dim3(64), 0, s, a);
    } else if (threads == 1024) {
        if (a.mode == 0)
            hipLaunchKernelGGL((cg_stream_kernel<true, 1024>), dim3(grid), dim3(1024), 0, s, a);
        else
            hipLaunchKernelGGL((cg_stream_kernel<false, 1024>), dim3(grid), dim3(1024), 0, s, a);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_tangent_spread(const TangentArgs& a, const SpreadArgs& sp, hipStream_t s)
{
    if (a.n_order <= 0) return hipSuccess;
    const SpreadCgArgs args{a, sp};
    if (a.mode == 0)
        hipLaunchKernelGGL(cg_spread_kernel<true>, dim3((unsigned)sp.grid), dim3(kCgT), 0, s, args);
    else
        hipLaunchKernelGGL(cg_spread_kernel<false>, dim3((unsigned)sp.grid), dim3(kCgT), 0, s, args);
    return hipGetLastError();
}

size_t tangent_spread_slot_bytes() { return 8 * (3 * (size_t)(kSpreadZero + 1) + 3 * (size_t)kSpreadNodes); }

hipError_t tangent_spread_info(int* blocks_per_cu, size_t* private_bytes)
{
    for (const void* f : {(const void*)cg_spread_kernel<true>, (const void*)cg_spread_kernel<false>}) {
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, f, kCgT, 0);
        if (e != hipSuccess) return e;
        if (*blocks_per_cu < 1) return hipSuccess;
    }
    return max_private_bytes({(const void*)cg_spread_kernel<true>, (const void*)cg_spread_kernel<false>}, private_bytes);
}

// dynamic LDS (the on-chip builds hold theirs statically)
static size_t res_lds(int v)
{
    return v < 3 ? 0 : 16 * ((size_t)kTanRes[v].threads * kTanRes[v].sn + 1);
}

hipError_t tangent_res_blocks(int v, bool vjp, int* blocks_per_cu)
{
    if (v < 0 || v >= kNumTanRes) return hipErrorInvalidValue;
    const void* k = res_kernel(v, vjp);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)res_lds(v));
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, kTanRes[v].threads, res_lds(v));
}

hipError_t launch_tangent_res(int v, const TangentArgs& a, int grid, bool own_cu, hipStream_t s)
{
    if (v < 0 || v >= kNumTanRes) return hipErrorInvalidValue;
    if (a.n_order <= 0) return hipSuccess;
    const void* k = res_kernel(v, a.mode != 0);
    // more than half of a CU's LDS keeps a second workgroup away
    const size_t lds = own_cu && v < 3 ? 82 * 1024 - 15 * 1024 : res_lds(v);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    void* args[] = {const_cast<TangentArgs*>(&a)};
    return hipLaunchKernel(k, dim3(grid), dim3(kTanRes[v].threads), args, lds, s);
}

hipError_t tangent_res_scratch_bytes(int v, bool vjp, size_t* bytes)
{
    if (v < 0 || v >= kNumTanRes) return hipErrorInvalidValue;
    return max_private_bytes({res_kernel(v, vjp)}, bytes);
}

// Blocked tangent tasks (three right-hand sides per workgroup) with the
// node capacity of the per-column variants 0-2 (512, 1024, 2048 free nodes).
const TangentVariant kTanBlk[kNumTanBlk] = {{256, 2}, {512, 2}, {1024, 2}};

static const void* blk_kernel(int v)
{
    switch (v) {
    case 0: return (const void*)cg_blk_kernel<256, 2, 4>;
    case 1: return (const void*)cg_blk_kernel<512, 2, 4>;
    default: return (const void*)cg_blk_kernel<1024, 2, 4>;
    }
}

static size_t blk_lds(int v)
{
    return 16 * (size_t)kBlk * ((size_t)kTanBlk[v].threads * kTanBlk[v].sn + 1);
}

hipError_t tangent_blk_blocks(int v, int* blocks_per_cu)
{
    if (v < 0 || v >= kNumTanBlk) return hipErrorInvalidValue;
    const void* k = blk_kernel(v);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)blk_lds(v));
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, kTanBlk[v].threads, blk_lds(v));
}

hipError_t launch_tangent_blk(int v, const TangentArgs& a, int grid, hipStream_t s)
{
    if (v < 0 || v >= kNumTanBlk) return hipErrorInvalidValue;
    if (a.n_order <= 0) return hipSuccess;
    const void* k = blk_kernel(v);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)blk_lds(v));
    if (e != hipSuccess) return e;
    void* args[] = {const_cast<TangentArgs*>(&a)};
    return hipLaunchKernel(k, dim3(grid), dim3(kTanBlk[v].threads), args, blk_lds(v), s);
}

hipError_t tangent_blk_scratch_bytes(int v, size_t* bytes)
{
    if (v < 0 || v >= kNumTanBlk) return hipErrorInvalidValue;
    return max_private_bytes({blk_kernel(v)}, bytes);
}

hipError_t tangent_fixed_private(size_t* bytes)
{
    return max_private_bytes({(const void*)ell_build_kernel, (const void*)fiber_ops_kernel,
                              (const void*)cg_stream_kernel<true, 64>, (const void*)cg_stream_kernel<false, 64>,
                              (const void*)cg_stream_kernel<true, 1024>, (const void*)cg_stream_kernel<false, 1024>,
                              (const void*)zero_status},
                             bytes);
}

}  // namespace rve
