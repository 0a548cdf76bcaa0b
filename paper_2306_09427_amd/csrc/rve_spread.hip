// Spread relaxation for gfx950 (MI355X): k workgroups, one per CU, relax one
// RVE too large for one CU's registers.
//
// What bounds the single-CU incidence kernel on such an RVE is one CU: every
// iteration streams the network's records (1 MB at 10 300 free nodes) and
// evaluates each fiber at both ends, 15 to 51 us, while most CUs idle unless
// the batch holds hundreds of large RVEs.  Here each workgroup keeps the records of
// its nodes in registers, as the on-chip tangent does, and an iteration is
// the share of the arithmetic plus one exchange between the workgroups: one RVE
// of 10 300 free nodes takes 5.5 us per iteration on 12 CUs (27.5 on one), of
// 16 000 5.7 us on 16 (51.6); 512 of 4900 free nodes 0.077 us per iteration and
// RVE on 3 CUs each (0.080), 256 of 16 000 0.229 on 8 (0.714).  What bounds an
// iteration now is its chain: the force pass of the largest part (half of the
// time at 1700 nodes), then the exchange's round trip through memory (2.2 to 3.5
// us), which no work can hide, as the time step needs every part's maximum.
//
// Per iteration a workgroup publishes the acceleration of the nodes other
// parts hold as halo (three words each) and its time-step maximum (one word;
// on test iterations its three FP64 sums in six).  A reader advances its halo
// nodes itself, with the same operations as the owner, so nothing is exchanged
// between the time step and the next force pass.  A member that gives up at a
// poll leaves the RVE's status unfinished and stops, the others follow at
// their next exchange, and the incidence kernel launched behind takes every
// unfinished RVE.  Members that had passed the last exchange by then have
// stored their final positions; a warm start's are kept aside before the launch
// and put back (keep_state), so that kernel starts from what the caller left.
//
// One launch runs teams of every size (rve_exchange.h): as a launch per size,
// at most four at once, 256 RVEs of 100 to 3000 seeds took 135 ms, 71 ms so.
//
// 512 threads of up to 256 VGPRs with four nodes each: 1024 of 128 spill.
//
// Arithmetic, its rounding and the order of every node's sum are those of the
// incidence kernel (rve_kernels.hip): after the same number of iterations the
// states agree bit for bit.  The FP64 norms of a convergence test are summed in
// another order (parts, then members) and agree to rounding, so a test that
// falls on its threshold may end a run one test earlier or later.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rve_exchange.h"
#include "rve_fiber.h"
#include "rve_internal.h"
#include "rve_relax.h"
#include "rve_wave.h"

namespace rve {

namespace {

typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef KernArgsT<SpreadArgs> Args;

constexpr int T = kSpreadThreads, SN = kSpreadSlots, NW = T / 64;
constexpr int HN = kSpreadNodes / T;   // halo nodes per thread
constexpr int XN = kSpreadExtra;

struct SpreadRed : TeamSlot {
    double v[3][16];
    double sum[3][kTeamMax];
    float g[16];
    float gmax;
};

// (Dn, Qn, 1/L0) of one incidence under F, the fiber oriented so that the node
// is its end j; formed in FP64 (inc_record in rve_kernels.hip).
template <typename Net>
__device__ __forceinline__ void record_of(const double* F, const Net& net, int64_t f0, uint32_t w, float4& rc, float& iL)
{
    const int64_t k = f0 + (int64_t)(w & 0x7fffffffu);
    const double* d0 = net.d0 + 3 * k;
    const double L0 = net.L0[k], il = 1.0 / L0;
    const double Dx = F[0] * d0[0] + F[1] * d0[1] + F[2] * d0[2];
    const double Dy = F[3] * d0[0] + F[4] * d0[1] + F[5] * d0[2];
    const double Dz = F[6] * d0[0] + F[7] * d0[1] + F[8] * d0[2];
    const double sg = (w >> 31) ? -il : il;
    rc = make_float4((float)(Dx * sg), (float)(Dy * sg), (float)(Dz * sg),
                     (float)((((Dx * Dx + Dy * Dy + Dz * Dz) - L0 * L0) * il) * il));
    iL = (float)il;
}

// One RVE; returns false when a poll gave up.
__device__ __forceinline__ bool spread_solve(Args& A, int r, Team& tm, f32x3* H, f32x3* W, float4* XA, uint2* XB,
                                             SpreadRed& red)
{
    unsigned& tag = tm.tag;
    const int rank = tm.rank, k = tm.k;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave64 = uniform32(tid & ~63);
    auto& net = A.s.net;
    const int64_t f0 = uniform64(net.fib_off[r]), a0 = uniform64(net.free_off[r]), b0 = uniform64(net.bnd_off[r]);
    const int64_t pi = uniform64(A.part_first[r]) + rank;
    const int nown = uniform32(A.parts[pi].nown), nhalo = uniform32(A.parts[pi].nhalo);
    const int x4 = uniform32(A.parts[pi].x4);
    const int64_t own0 = uniform64(A.parts[pi].own0), halo0 = uniform64(A.parts[pi].halo0);
    const int max_x = A.max_x, half = (A.area_words - 16) / 2;
    u64* const xbuf = tm.area + 16;
    auto words_of = [&](unsigned t) __attribute__((always_inline)) { return xbuf + (t & 1) * half + 3 * (int64_t)max_x; };

    double F[9];
    bool finite = true;
    for (int q = 0; q < 9; ++q) {
        F[q] = A.s.F[9 * r + q];
        finite = finite && isfinite(F[q]);
    }
    const double J = det3(F);
    if (!finite || !(J > 0.0)) {   // the same in every member
        if (tid == 0 && rank == 0) {
            A.s.status[r] = ST_BAD_F;
            A.s.iters[r] = 0;
            A.s.Rres[r] = NAN; A.s.Dres[r] = NAN; A.s.Bres[r] = NAN;
            for (int q = 0; q < 9; ++q) A.s.sigma[9 * r + q] = NAN;
        }
        ++tag;
        return team_done(A, red, tm, words_of(tag));
    }
    const bool linear = A.s.law == kLawLinear;
    const float EA = uniform((float)A.s.EA), Bc = uniform((float)A.s.B), EAoB = uniform((float)(A.s.EA / A.s.B));
    const float c = uniform((float)A.s.c[r]);

    // ---- owned nodes: records, state and exchange slots in registers; the
    // records beyond four of the nodes x4 .. nown in LDS, row j of them for
    // incidence 4 + j
    const int nx = nown - x4;
    float dx_[SN][4], dy_[SN][4], dz_[SN][4], qn_[SN][4], il_[SN][4];
    uint32_t os[SN][2];   // byte offsets / 8 of the other ends' positions, two per word
    float vx[SN], vy[SN], vz[SN], hx[SN], hy[SN], hz[SN], im[SN];
    int xs[SN], degw[SN];
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        const int a = s * T + tid;
        float z0 = 0.f;
        asm volatile("" : "+v"(z0));
        uint32_t o4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dx_[s][q] = dy_[s][q] = dz_[s][q] = qn_[s][q] = il_[s][q] = z0;
            o4[q] = 2 * kSpreadZero;
        }
        vx[s] = vy[s] = vz[s] = hx[s] = hy[s] = hz[s] = im[s] = z0;
        xs[s] = -1;
        int deg = 0;
        if (a < nown) {
            const int id = A.own[own0 + a];
            xs[s] = A.xslot[own0 + a];
            im[s] = (float)(1.0 / (net.mass[a0 + id] * A.s.rhoA));
            if (A.s.init == kInitWarm) {
                const double* h = A.s.h_state + 3 * (a0 + id);
                hx[s] = (float)h[0]; hy[s] = (float)h[1]; hz[s] = (float)h[2];
            }
            const int64_t e0 = net.inc_off[a0 + id];
            deg = (int)(net.inc_off[a0 + id + 1] - e0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < deg) {
                    float4 rc;
                    record_of(F, net, f0, net.inc[e0 + q], rc, il_[s][q]);
                    dx_[s][q] = rc.x; dy_[s][q] = rc.y; dz_[s][q] = rc.z; qn_[s][q] = rc.w;
                    o4[q] = 2u * A.oslot[e0 + q];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll 1
            for (int q = 4; q < deg; ++q) {
                float4 rc;
                float il;
                record_of(F, net, f0, net.inc[e0 + q], rc, il);
                XA[(q - 4) * nx + (a - x4)] = rc;
                XB[(q - 4) * nx + (a - x4)] = make_uint2(__float_as_uint(il), (uint32_t)A.oslot[e0 + q] | (uint32_t)deg << 16);
            }
        }
        os[s][0] = o4[0] | o4[1] << 16;
        os[s][1] = o4[2] | o4[3] << 16;
        H[a] = f32x3{hx[s], hy[s], hz[s]};
        degw[s] = uniform32((int)__float_as_uint(wave_max_nonneg(__uint_as_float((unsigned)deg))));
        __builtin_amdgcn_sched_barrier(0);
    }
    // ---- halo nodes: velocity and position in LDS
    float bx[HN], by[HN], bz[HN];
    int hs[HN];
#pragma unroll
    for (int u = 0; u < HN; ++u) {
        const int i = u * T + tid;
        float x = 0.f, y = 0.f, z = 0.f;
        hs[u] = -1;
        bx[u] = by[u] = bz[u] = 0.f;
        W[i] = f32x3{x, y, z};
        if (i < nhalo) {
            hs[u] = A.halo_xslot[halo0 + i];
            if (A.s.init == kInitWarm) {
                const double* h = A.s.h_state + 3 * (a0 + A.halo[halo0 + i]);
                x = (float)h[0]; y = (float)h[1]; z = (float)h[2];
            }
        }
        H[kSpreadNodes + i] = f32x3{x, y, z};
    }
    if (tid == 0) {
        float z0 = 0.f;
        asm volatile("" : "+v"(z0));
        H[kSpreadZero] = f32x3{z0, z0, z0};
    }
    // boundary records of this part's boundary nodes
    {
        const int64_t bp0 = uniform64(A.parts[pi].bnd0);
        const int nbnd = uniform32(A.parts[pi].nbnd);
#pragma unroll 1
        for (int q = tid; q < nbnd; q += T) {
            const int64_t bn = b0 + A.bnd[bp0 + q];
#pragma unroll 1
            for (int64_t e = net.binc_off[bn]; e < net.binc_off[bn + 1]; ++e) {
                float4 rc;
                float il;
                record_of(F, net, f0, net.binc[e], rc, il);
                A.brec[e] = rc;
            }
        }
    }
    __syncthreads();

    // internal force and Gershgorin sum of the node in slot s
    auto force = [&](int s, int t, float& fx, float& fy, float& fz, float& G) __attribute__((always_inline)) {
        fx = fy = fz = G = 0.f;
        const char* Hb = reinterpret_cast<const char*>(H);
        auto add = [&](float Dx, float Dy, float Dz, float Qn, float iL, f32x3 o) __attribute__((always_inline)) {
            const FiberState f = fiber_state(linear, EA, Bc, EAoB, Dx, Dy, Dz, Qn, iL, hx[s] - o.x, hy[s] - o.y, hz[s] - o.z);
            fx = fmaf(f.ex, f.g, fx); fy = fmaf(f.ey, f.g, fy); fz = fmaf(f.ez, f.g, fz);
            G = fmaf(iL, f.b, G);
        };
        f32x3 o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            o[q] = *(const f32x3*)(Hb + 8u * ((q & 1) ? os[s][q >> 1] >> 16 : os[s][q >> 1] & 0xffffu));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            add(dx_[s][q], dy_[s][q], dz_[s][q], qn_[s][q], il_[s][q], o[q]);
        }
        if (degw[s] > 4) {   // wave-uniform
            const int i = s * T + t - x4;
            if (i >= 0 && i < nx) {
                uint2 b = XB[i];
                const int deg = (int)(b.y >> 16);
#pragma unroll 1
                for (int q = 0; q < deg - 4; ++q) {
                    const float4 rc = XA[q * nx + i];
                    if (q > 0) b = XB[q * nx + i];
                    add(rc.x, rc.y, rc.z, rc.w, __uint_as_float(b.x), H[b.y & 0xffffu]);
                }
            }
        }
        G += G;
    };
    // boundary reaction norm^2 partial of this thread (test iterations)
    auto bnorm2 = [&](int t) __attribute__((always_inline)) -> double {
        auto* K = kernel_args<SpreadArgs>();
        const int64_t bp0 = uniform64(K->parts[pi].bnd0);
        const int nbnd = uniform32(K->parts[pi].nbnd);
        double acc = 0.0;
#pragma unroll 1
        for (int q = t; q < nbnd; q += T) {
            const int64_t bn = b0 + K->bnd[bp0 + q];
            const int64_t e1 = K->s.net.binc_off[bn + 1];
            double x = 0.0, y = 0.0, z = 0.0;
#pragma unroll 1
            for (int64_t e = K->s.net.binc_off[bn]; e < e1; ++e) {
                const float4 rc = K->brec[e];
                const f32x3 o = H[K->bslot[e]];
                const FiberState f = fiber_state(linear, EA, Bc, EAoB, rc.x, rc.y, rc.z, rc.w,
                                                 __uint_as_float(K->brec_st[e].x), 0.f - o.x, 0.f - o.y, 0.f - o.z);
                x += (double)(f.g * f.ex); y += (double)(f.g * f.ey); z += (double)(f.g * f.ez);
            }
            acc += x * x + y * y + z * z;
        }
        return acc;
    };
    // Publish a node's acceleration.
    auto publish = [&](int s, float x, float y, float z) __attribute__((always_inline)) {
        if (xs[s] >= 0) {
            u64* p = xbuf + (tag & 1) * half + xs[s];
            put_word(p, tag, __float_as_uint(x));
            put_word(p + max_x, tag, __float_as_uint(y));
            put_word(p + 2 * max_x, tag, __float_as_uint(z));
        }
    };
    // The exchange of tag `tag`: the team's time-step maximum, on test
    // iterations the three sums (every member adds the parts in the same order),
    // and the accelerations of the halo.  Two barriers; false when a poll gave up.
    auto exchange = [&](int t, float g, double r2, double d2, double b2, bool full, float& gmax, double& R2, double& D2,
                        double& B2) __attribute__((always_inline)) -> bool {
        const int lane = t & 63, wave = t >> 6;
        g = wave_max_lane63(g);
        if (lane == 63) red.g[wave] = g;
        if (full) {
            r2 = wave_sum(r2);
            d2 = wave_sum(d2);
            b2 = wave_sum(b2);
            if (lane == 0) {
                red.v[0][wave] = r2;
                red.v[1][wave] = d2;
                red.v[2][wave] = b2;
            }
        }
        __syncthreads();
        u64* const words = words_of(tag);   // [k] maxima, [k][3][2] sums
        int polls = 0;
        const int limit = kernel_args<SpreadArgs>()->spin_limit;
        bool ok = true;
        if (wave64 == 0) {
            unsigned m = __float_as_uint(red.g[lane & 15]);
            m = dpp_max_step<kDppXor1, 0xf>(m);
            m = dpp_max_step<kDppXor2, 0xf>(m);
            m = dpp_max_step<0x141, 0xf>(m);
            m = dpp_max_step<0x140, 0xf>(m);
            if (lane == 0) put_word(words + rank, tag, m);
            if (full) {
                const int p = lane >> 4, w = lane & 15;
                double s = p < 3 && w < NW ? red.v[p < 3 ? p : 0][w] : 0.0, e = 0.0;
                combine_pairs<kDppRor8>(s, e);
                combine_pairs<kDppRor4>(s, e);
                combine_pairs<kDppXor2>(s, e);
                combine_pairs<kDppXor1>(s, e);
                const double tot = s + e;
                if (w == 0 && p < 3) {
                    put_word(words + k + 6 * rank + 2 * p, tag, (unsigned)__double2loint(tot));
                    put_word(words + k + 6 * rank + 2 * p + 1, tag, (unsigned)__double2hiint(tot));
                }
            }
            // every lane of a row polls the same word where k < 16
            unsigned gm = 0;
            {
                const u64* p = words + (lane & 15) % k;
                u64 v = get_word(p);
                while (!tagged(v, tag) && ++polls < limit) v = get_word(p);
                ok = ok && tagged(v, tag);
                gm = (unsigned)v;
            }
            if (full) {
#pragma unroll 1
                for (int i = lane; i < 3 * k; i += 64) {
                    const u64* p = words + k + 2 * i;
                    u64 lo = get_word(p), hi = get_word(p + 1);
                    while (!(tagged(lo, tag) && tagged(hi, tag)) && ++polls < limit) {
                        lo = get_word(p);
                        hi = get_word(p + 1);
                    }
                    ok = ok && tagged(lo, tag) && tagged(hi, tag);
                    red.sum[i % 3][i / 3] = __hiloint2double((int)(unsigned)hi, (int)(unsigned)lo);
                }
            }
            gm = dpp_max_step<kDppXor1, 0xf>(gm);
            gm = dpp_max_step<kDppXor2, 0xf>(gm);
            gm = dpp_max_step<0x141, 0xf>(gm);
            gm = dpp_max_step<0x140, 0xf>(gm);
            if (lane == 0) red.gmax = __uint_as_float(gm);
        }
#pragma unroll
        for (int u = 0; u < HN; ++u)
            if (hs[u] >= 0) {
                const u64* p = xbuf + (tag & 1) * half + hs[u];
                u64 x = get_word(p), y = get_word(p + max_x), z = get_word(p + 2 * max_x);
                while (!(tagged(x, tag) && tagged(y, tag) && tagged(z, tag)) && ++polls < limit) {
                    x = get_word(p);
                    y = get_word(p + max_x);
                    z = get_word(p + 2 * max_x);
                }
                ok = ok && tagged(x, tag) && tagged(y, tag) && tagged(z, tag);
                bx[u] = __uint_as_float((unsigned)x); by[u] = __uint_as_float((unsigned)y); bz[u] = __uint_as_float((unsigned)z);
            }
        if (!ok) red.bad = 1;
        __syncthreads();
        gmax = uniform(red.gmax);
        if (full) {
            double x = 0.0, y = 0.0, z = 0.0;
            for (int p = 0; p < k; ++p) {
                x += red.sum[0][p];
                y += red.sum[1][p];
                z += red.sum[2][p];
            }
            R2 = uniform(x);
            D2 = uniform(y);
            B2 = uniform(z);
        }
        return uniform32(red.bad) == 0;
    };

    // The first pass evaluates the start: a time step of zero moves nothing, the
    // mass is scaled on request, and its norms decide as a test's do.
    float ax[SN], ay[SN], az[SN];
#pragma unroll
    for (int s = 0; s < SN; ++s) ax[s] = ay[s] = az[s] = 0.f;
    float rdt = 0.f, hdt = 0.f, hprev = 0.f;
    double R2 = 0.0, D2 = 0.0, B2 = 0.0, Rref = 0.0;
    int stall = 0, status = ST_CONVERGED;
    const int ce = A.s.check_every > 0 ? A.s.check_every : 1;
    int64_t n = 0;
    int cd = 1, evn = 0;   // passes to the next event (the start, a test or n_max), iterations of this stretch
    bool ev_test = true, first = true;
    for (;;) {
        int t = tid;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int s = 0; s < SN; ++s) asm volatile("" : "+v"(os[s][0]), "+v"(os[s][1]));
        // half-step velocity and position of the owned and the halo nodes
#pragma unroll
        for (int s = 0; s < SN; ++s)
            if (s * T + wave64 < nown) {
                vx[s] = fmaf(ax[s], hdt, vx[s]); vy[s] = fmaf(ay[s], hdt, vy[s]); vz[s] = fmaf(az[s], hdt, vz[s]);
                hx[s] = fmaf(vx[s], rdt, hx[s]); hy[s] = fmaf(vy[s], rdt, hy[s]); hz[s] = fmaf(vz[s], rdt, hz[s]);
                H[s * T + t] = f32x3{hx[s], hy[s], hz[s]};
            }
#pragma unroll
        for (int u = 0; u < HN; ++u)
            if (u * T + wave64 < nhalo) {
                // second half step of the last iteration, then this one's first
                const f32x3 h = H[kSpreadNodes + u * T + t], w = W[u * T + t];
                const float wx = fmaf(bx[u], hdt, fmaf(bx[u], hprev, w.x)), wy = fmaf(by[u], hdt, fmaf(by[u], hprev, w.y)),
                            wz = fmaf(bz[u], hdt, fmaf(bz[u], hprev, w.z));
                W[u * T + t] = f32x3{wx, wy, wz};
                H[kSpreadNodes + u * T + t] = f32x3{fmaf(wx, rdt, h.x), fmaf(wy, rdt, h.y), fmaf(wz, rdt, h.z)};
            }
        hprev = hdt;
        __syncthreads();
        --cd;
        ++tag;
        const bool check = cd == 0 && ev_test;
        float gpart = 0.f;
        double r2p = 0.0, d2p = 0.0, b2p = 0.0;
#pragma unroll
        for (int s = 0; s < SN; ++s) {
            if (s * T + wave64 < nown) {
                float fx, fy, fz, G;
                force(s, t, fx, fy, fz, G);
                if (first && kernel_args<SpreadArgs>()->s.mass_mode == kMassScaled && s * T + t < nown)
                    im[s] = G > 0.f ? 4.f / G : 1.f;
                // damped acceleration with the half-step velocity, then second half step
                ax[s] = fmaf(im[s], -fx, -(c * vx[s]));
                ay[s] = fmaf(im[s], -fy, -(c * vy[s]));
                az[s] = fmaf(im[s], -fz, -(c * vz[s]));
                publish(s, ax[s], ay[s], az[s]);
                vx[s] = fmaf(ax[s], hdt, vx[s]); vy[s] = fmaf(ay[s], hdt, vy[s]); vz[s] = fmaf(az[s], hdt, vz[s]);
                gpart = fmaxf(gpart, G * im[s]);
                if (check) {
                    r2p += (double)fx * fx + (double)fy * fy + (double)fz * fz;
                    const float cm = c * __builtin_amdgcn_rcpf(im[s]);
                    const double px = (double)(cm * vx[s]), py = (double)(cm * vy[s]), pz = (double)(cm * vz[s]);
                    d2p += s * T + t < nown ? px * px + py * py + pz * pz : 0.0;   // (slots past the last node have im = 0)
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (check) b2p = bnorm2(t);
        float gmax;
        double r2n = R2, d2n = D2, b2n = B2;
        if (!exchange(t, gpart, r2p, d2p, b2p, check, gmax, r2n, d2n, b2n)) return false;
        auto* K = kernel_args<SpreadArgs>();
        if (check) {
            R2 = r2n;
            D2 = first ? 0.0 : d2n;   // (v = 0)
            B2 = b2n;
            if (!isfinite(R2) || !isfinite(D2)) {
                status = ST_NONFINITE;
                break;
            }
            if (first) Rref = uniform(sqrt(R2));
            if (test_in_reach(K->s, R2, B2)) {
                const double Rn = sqrt(R2), Dn = sqrt(D2), Bn = sqrt(B2);
                const double tol = fmax(K->s.tol_abs, K->s.tol_rel * Bn);
                if (Rn <= tol && Dn <= tol) break;
                if (!first && stagnated(K->s, Rn, Dn, Bn, Rref, stall)) {
                    status = ST_STAGNATED;
                    break;
                }
                Rref = uniform(Rref);
            }
        }
        if (!first && (!(gmax > 0.f) || !isfinite(gmax))) {
            status = ST_NONFINITE;
            break;
        }
        if (cd == 0) {
            n += evn;
            const int64_t left = K->s.n_max - n;
            if (left <= 0) {
                status = ST_MAXITER;
                evn = 0;
                break;
            }
            evn = cd = uniform32((int)(left < ce ? left : ce));
            ev_test = cd == ce;
            first = false;
        }
        rdt = uniform(uniform((float)(2.0 * K->s.alpha)) * __builtin_amdgcn_rsqf(gmax));
        hdt = 0.5f * rdt;
    }
    if (evn > 0) n += evn - cd;   // the stretch the loop was left in

    // ---- fluctuation state, then the first member reports the RVE
    auto* K = kernel_args<SpreadArgs>();
    int te = tid;
    asm volatile("" : "+v"(te));
#pragma unroll
    for (int s = 0; s < SN; ++s) {
        const int a = s * T + te;
        if (a < nown) {
            double* h = K->s.h_state + 3 * (K->s.net.free_off[r] + K->own[own0 + a]);
            h[0] = (double)hx[s]; h[1] = (double)hy[s]; h[2] = (double)hz[s];
        }
    }
    ++tag;
    const bool all = team_done(*K, red, tm, words_of(tag));
    if (te == 0 && rank == 0 && all) {
        K->s.status[r] = status;
        K->s.iters[r] = n;
        K->s.Rres[r] = sqrt(R2);
        K->s.Dres[r] = sqrt(D2);
        K->s.Bres[r] = sqrt(B2);
    }
    return all;
}

__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(2))) void dr_spread_kernel(SpreadArgs)
{
    __shared__ f32x3 H[kSpreadZero + 1];   // positions: owned, halo, zero
    __shared__ f32x3 W[kSpreadNodes];      // velocities of the halo
    __shared__ float4 XA[XN];
    __shared__ uint2 XB[XN];
    __shared__ SpreadRed red;
    auto& A = *kernel_args<SpreadArgs>();
    if (threadIdx.x == 0) red.bad = 0;
    if (threadIdx.x < 16) red.g[threadIdx.x] = 0.f;   // (a row of the maximum's tree; NW of them are written)
    Team tm;
    while (team_take(A, red, tm))
        if (!spread_solve(*kernel_args<SpreadArgs>(), uniform32(kernel_args<SpreadArgs>()->task_rve[tm.task]), tm, H, W, XA, XB, red))
            break;
}

// Tasks of a launch, list0 then list1, and the first slot of each (k slots per
// task).  One workgroup.
__global__ __launch_bounds__(1024) void team_slots(const int32_t* list0, int n0, const int32_t* list1, int n1,
                                                   const int32_t* k_of, int32_t* task_rve, int32_t* task_first)
{
    __shared__ int part[16], base;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = n0 + n1;
    if (t == 0) base = 0;
    for (int q0 = 0; q0 <= n; q0 += 1024) {
        const int q = q0 + t;
        const int r = q < n0 ? list0[q] : q < n ? list1[q - n0] : -1, k = r >= 0 ? k_of[r] : 0;
        int x = k;
        for (int d = 1; d < 64; d *= 2) {
            const int y = __shfl_up(x, d);
            x += lane >= d ? y : 0;
        }
        if (lane == 63) part[wave] = x;
        __syncthreads();
        int b = base;
        for (int w = 0; w < wave; ++w) b += part[w];
        if (q <= n) task_first[q] = b + x - k;
        if (r >= 0) task_rve[q] = r;
        __syncthreads();
        if (t == 1023) base = b + x;
        __syncthreads();
    }
}

__global__ void set_status(const int32_t* list, int n, int32_t* status, int32_t value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) status[list[i]] = value;
}

// The free nodes' fluctuation of the listed RVEs into `kept` (in the order of
// their parts' nodes) and their status to kStUnfinished; or (restore) back where
// the status still is.
__global__ __launch_bounds__(256) void keep_state(const int32_t* list, const SpreadPart* parts, const int64_t* part_first,
                                                  const int64_t* free_off, double* h, double* kept, int32_t* status,
                                                  bool restore)
{
    const int r = list[blockIdx.x];
    if (restore && status[r] != kStUnfinished) return;
    if (!restore && blockIdx.y == 0 && threadIdx.x == 0) status[r] = kStUnfinished;
    const int64_t a0 = 3 * free_off[r], n = 3 * free_off[r + 1] - a0, k0 = 3 * parts[part_first[r]].own0;
    for (int64_t q = blockIdx.y * 256 + threadIdx.x; q < n; q += 256 * gridDim.y) {
        if (restore)
            h[a0 + q] = kept[k0 + q];
        else
            kept[k0 + q] = h[a0 + q];
    }
}

}  // namespace

hipError_t launch_keep_state(const SpreadArgs& a, double* kept, bool restore, hipStream_t s)
{
    if (a.n_tasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(keep_state, dim3((unsigned)a.n_tasks, 8), dim3(256), 0, s, a.task_rve, a.parts, a.part_first,
                       a.s.net.free_off, a.s.h_state, kept, a.s.status, restore);
    return hipGetLastError();
}

hipError_t launch_spread(const SpreadArgs& a, hipStream_t s)
{
    if (a.n_tasks <= 0) return hipSuccess;
    hipLaunchKernelGGL(dr_spread_kernel, dim3((unsigned)a.grid), dim3(T), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_team_slots(const int32_t* list0, int n0, const int32_t* list1, int n1, const int32_t* k_of,
                             int32_t* task_rve, int32_t* task_first, hipStream_t s)
{
    hipLaunchKernelGGL(team_slots, dim3(1), dim3(1024), 0, s, list0, n0, list1, n1, k_of, task_rve, task_first);
    return hipGetLastError();
}

hipError_t launch_set_status(const int32_t* list, int n, int32_t* status, int32_t value, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(set_status, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, list, n, status, value);
    return hipGetLastError();
}

hipError_t spread_info(int* blocks_per_cu, size_t* private_bytes)
{
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, (const void*)dr_spread_kernel, T, 0);
    if (e != hipSuccess) return e;
    return max_private_bytes({(const void*)dr_spread_kernel, (const void*)team_slots, (const void*)set_status,
                              (const void*)keep_state}, private_bytes);
}

}  // namespace rve
