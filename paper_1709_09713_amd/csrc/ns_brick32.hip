// ns_brick32.hip -- the fused FP32-storage stage kernel for small grids.
//
// A block owns a brick of points and stages it whole, with its halo of two, in
// one round of loads, as ns_brick.hip does for FP64, and three groups of waves
// (A mass and energy, B momentum, C viscous terms) evaluate one point per
// thread.  The expressions are those of the one-thread march (ns_fused.hip,
// evaluation order 0) and every sum adds its terms in the march's order, so
// that both give the same result bit for bit: A and B stop before the first
// term of C's, and go on when C has handed its values over.
//
// Bound by latency like the FP64 kernel: 4.6 us a stage at 16^3, 1.7 us of it
// an empty launch; at 48^3, 3.4 bricks a compute unit, by LDS and vector issue
// (9.6 us).  us per RK3 step, march (its best tile) -> bricks: 16^3 21.9 -> 13.5,
// 32^3 22.9 -> 15.5, 40^3 27.5 -> 19.0, 48^3 29.7 -> 27.9.  Rows of one field
// instead of two: 32^3 16.5, 40^3 21.4, 48^3 30.8 (bank conflicts); one thread per
// point for all equations: 16.0, 17.4, 22.1, 28.9 at 16^3 to 48^3, before that.
#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

namespace {

constexpr int BRX = 8, BRY = 4;

__device__ __forceinline__ float recip_f32(float x)
{
    float r = __builtin_amdgcn_rcpf(x);
    const float e = __builtin_fmaf(-x, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}

template <int MODE> struct Types { using in = float; using out = float; };
template <> struct Types<1> { using in = double; using out = float; };
template <> struct Types<3> { using in = float; using out = double; };

}  // namespace

template <int BRZ, int MODE, bool DIAG>
__global__ void __launch_bounds__(3 * BRX * BRY * BRZ) brick32_stage_kernel(Consts c, StageArgs s)
{
#pragma clang fp contract(on)
    static_assert(!DIAG || MODE == 1, "diagnostics of the step's input state are taken in stage 1");
    using TIN = typename Types<MODE>::in;
    using TOUT = typename Types<MODE>::out;
    constexpr int HX = BRX + 4, HY = BRY + 4, HZ = BRZ + 4, HP = HX * HY, CELLS = HP * HZ;
    constexpr int NT = BRX * BRY * BRZ, NLOAD = (CELLS + 3 * NT - 1) / (3 * NT);
    constexpr int GP = BRX * BRY, GC = GP * HZ;      // own columns with their z halo
    constexpr int NW = 3 * NT / 64;
    static_assert(NT % 64 == 0, "each group must be whole waves");
    static_assert(GC <= 3 * NT, "one gradient point per thread");
    enum { L_RHO, L_M0, L_M1, L_M2, L_E, L_U, L_V, L_W, L_P, L_T, NF };
    enum { G_A, G_B, G_C, NG };                      // D_x u + D_y v, D_x w, D_y w
    // Two fields share a row of the array, side by side: with rows of 2 HX cells
    // the rows that a wave reads at once start in different banks.
    constexpr int RS = 2 * HX, PS = HY * RS;
    static_assert(NF % 2 == 0, "fields in pairs");
    __shared__ float lds[NF / 2][HZ * PS];
    __shared__ float grad[NG][GC];
    // handed over by C: in-plane and z parts of the viscous terms (momentum,
    // then energy) and the in-plane heat conduction
    enum { H_VX, H_VY, H_VZ, H_EN, H_ZX, H_ZY, H_ZZ, H_ZEN, H_HEAT, NH };
    __shared__ float vbuf[NH][NT];
    __shared__ double red[DIAG ? NW : 1][4];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / (NT / 64);
    const int pt = tid - grp * NT;
    const int tx = pt % BRX, ty = (pt / BRX) % BRY, tz = pt / GP;
    int skip = 0;
    if constexpr (MODE == 2) {
        skip = finalize_layer(c, s);
        if (skip < 0) return;
    }
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz, skip);
    const int x0 = tbx * BRX, y0 = tby * BRY, z0 = tbz * BRZ;
    const bool active = x0 + tx < c.nx && y0 + ty < c.ny && z0 + tz < c.nz;
    const int own = (tz + 2) * PS + (ty + 2) * RS + tx + 2;
    const int64_t N = c.N;
    const int64_t pidx = active ? ((int64_t)(z0 + tz) * c.ny + y0 + ty) * c.nx + x0 + tx : 0;
    const TIN *qin = (const TIN *)s.qin;
    const double *accsrc = (MODE >= 2) ? s.acc_in : (const double *)s.qin;
    const float c1x = (float)c.c1[0], c1y = (float)c.c1[1], c1z = (float)c.c1[2];
    const float c2x = (float)c.c2[0], c2y = (float)c.c2[1], c2z = (float)c.c2[2];
    const float inv_re = (float)c.inv_re, kappa = (float)c.kappa;
    const float gm1 = (float)c.gm1, gM2 = (float)c.gM2;
    const float half = 0.5f, third = 1.0f / 3.0f, four3 = 4.0f / 3.0f, two3 = 2.0f / 3.0f;
    const float kz = kappa * c2z;

#define AT(f, at) lds[(f) >> 1][((f) & 1) * HX + (at)]

    // ---- stage the brick with its halo, wrapped to valid memory everywhere: a
    // brick starts inside the grid at a multiple of its extent, so that with
    // five points or more one period each way is enough
    TIN q[NLOAD][5];
#pragma unroll
    for (int r = 0; r < NLOAD; ++r) {
        const int cell = min(tid + r * 3 * NT, CELLS - 1);
        const int xx = wrap1(x0 + cell % HX - 2, c.nx), yy = wrap1(y0 + (cell / HX) % HY - 2, c.ny);
        const int zz = wrap1(z0 + cell / HP - 2, c.nz);
        const TIN *src = qin + ((int64_t)zz * c.ny + yy) * c.nx + xx;
#pragma unroll
        for (int f = 0; f < 5; ++f) q[r][f] = src[f * N];
    }
    // accumulator of the own point: group A the mass and energy, B the momenta
    double acc[3] = {0.0, 0.0, 0.0};
    if (grp == 0) {
        acc[0] = accsrc[pidx];
        acc[1] = accsrc[4 * N + pidx];
    } else if (grp == 1) {
#pragma unroll
        for (int f = 0; f < 3; ++f) acc[f] = accsrc[(1 + f) * N + pidx];
    }
#pragma unroll
    for (int r = 0; r < NLOAD; ++r) {
        const int cell = tid + r * 3 * NT;
        if (CELLS % (3 * NT) != 0 && cell >= CELLS) continue;
        const int at = (cell / HX) * RS + cell % HX;
        float rho, m0, m1, m2, E;
        if constexpr (MODE == 1) {
            rho = (float)(q[r][0] - c.rho_ref);
            m0 = (float)q[r][1];
            m1 = (float)q[r][2];
            m2 = (float)q[r][3];
            E = (float)(q[r][4] - c.rhoE_ref);
        } else {
            rho = q[r][0];
            m0 = q[r][1];
            m1 = q[r][2];
            m2 = q[r][3];
            E = q[r][4];
        }
        const float rhof = 1.0f + rho;
        const float inv = recip_f32(rhof);
        const float u = m0 * inv, v = m1 * inv, w = m2 * inv;
        const float p = gm1 * (E - half * (m0 * u + m1 * v + m2 * w));
        AT(L_RHO, at) = rho;
        AT(L_M0, at) = m0;
        AT(L_M1, at) = m1;
        AT(L_M2, at) = m2;
        AT(L_E, at) = E;
        AT(L_U, at) = u;
        AT(L_V, at) = v;
        AT(L_W, at) = w;
        AT(L_P, at) = p;
        AT(L_T, at) = (gM2 * p - rho) * inv;
    }
    lds_barrier();

#define LV(f, dy, dx) AT(f, at + (dy) * RS + (dx))
#define LZ(f, dz) AT(f, own + (dz) * PS)
#define DX1(f) d1u(LV(f, 0, -2), LV(f, 0, -1), LV(f, 0, 1), LV(f, 0, 2))
#define DY1(f) d1u(LV(f, -2, 0), LV(f, -1, 0), LV(f, 1, 0), LV(f, 2, 0))
#define DX1P(f, g)                                                       \
    d1u(LV(f, 0, -2) * LV(g, 0, -2), LV(f, 0, -1) * LV(g, 0, -1),        \
        LV(f, 0, 1) * LV(g, 0, 1), LV(f, 0, 2) * LV(g, 0, 2))
#define DY1P(f, g)                                                       \
    d1u(LV(f, -2, 0) * LV(g, -2, 0), LV(f, -1, 0) * LV(g, -1, 0),        \
        LV(f, 1, 0) * LV(g, 1, 0), LV(f, 2, 0) * LV(g, 2, 0))
// (rhoE/2 + p) u_j at a tap: energy flux of the x or y direction
#define HF(dy, dx, g) ((half * LV(L_E, dy, dx) + LV(L_P, dy, dx)) * LV(g, dy, dx))
#define DX1H() d1u(HF(0, -2, L_U), HF(0, -1, L_U), HF(0, 1, L_U), HF(0, 2, L_U))
#define DY1H() d1u(HF(-2, 0, L_V), HF(-1, 0, L_V), HF(1, 0, L_V), HF(2, 0, L_V))
#define DX2(f) d2u(LV(f, 0, -2), LV(f, 0, -1), LV(f, 0, 0), LV(f, 0, 1), LV(f, 0, 2))
#define DY2(f) d2u(LV(f, -2, 0), LV(f, -1, 0), LV(f, 0, 0), LV(f, 1, 0), LV(f, 2, 0))
// D_x applied to D_y f and D_y applied to D_x f (16 taps), unscaled
#define DXDY(f)                                                          \
    d1u(d1u(LV(f, -2, -2), LV(f, -1, -2), LV(f, 1, -2), LV(f, 2, -2)),   \
        d1u(LV(f, -2, -1), LV(f, -1, -1), LV(f, 1, -1), LV(f, 2, -1)),   \
        d1u(LV(f, -2, 1), LV(f, -1, 1), LV(f, 1, 1), LV(f, 2, 1)),       \
        d1u(LV(f, -2, 2), LV(f, -1, 2), LV(f, 1, 2), LV(f, 2, 2)))
#define DYDX(f)                                                          \
    d1u(d1u(LV(f, -2, -2), LV(f, -2, -1), LV(f, -2, 1), LV(f, -2, 2)),   \
        d1u(LV(f, -1, -2), LV(f, -1, -1), LV(f, -1, 1), LV(f, -1, 2)),   \
        d1u(LV(f, 1, -2), LV(f, 1, -1), LV(f, 1, 1), LV(f, 1, 2)),       \
        d1u(LV(f, 2, -2), LV(f, 2, -1), LV(f, 2, 1), LV(f, 2, 2)))

    // ---- in-plane gradients of the own columns with their z halo
    if (tid < GC) {
        const int at = (tid / GP) * PS + ((tid % GP) / BRX + 2) * RS + tid % BRX + 2;
        const float gxx = c1x * DX1(L_U), gyy = c1y * DY1(L_V);
        grad[G_A][tid] = gxx + gyy;
        grad[G_B][tid] = c1x * DX1(L_W);
        grad[G_C][tid] = c1y * DY1(L_W);
    }
    lds_barrier();

#define DZ1(f) d1u(LZ(f, -2), LZ(f, -1), LZ(f, 1), LZ(f, 2))
#define DZ2(f, f0) d2u(LZ(f, -2), LZ(f, -1), f0, LZ(f, 1), LZ(f, 2))
#define GZ(f) d1u(grad[f][gat - 2 * GP], grad[f][gat - GP], grad[f][gat + GP], grad[f][gat + 2 * GP])
// rho u_i at the z taps
#define DZMD(k)                                                                                    \
    d1u((1.0f + LZ(L_RHO, -2)) * LZ(k, -2), (1.0f + LZ(L_RHO, -1)) * LZ(k, -1),                    \
        (1.0f + LZ(L_RHO, 1)) * LZ(k, 1), (1.0f + LZ(L_RHO, 2)) * LZ(k, 2))
// A sum takes the constant-coefficient flux terms of the planes around the
// point in the march's order: z - 2 and z - 1 before the in-plane terms, z + 1
// and z + 2 after them.
#define FLUX_BELOW(r, g) r += g[0]; r -= 8.0f * g[1]
#define FLUX_ABOVE(r, g) r += 8.0f * g[2]; r -= g[3]
    const int at = own, gat = (tz + 2) * GP + ty * BRX + tx;
    constexpr int ZT[4] = {-2, -1, 1, 2};
    // diagnostics of the point: group A mass and energy, B the momenta and
    // kinetic energy, C enstrophy
    double dsum[4] = {0.0, 0.0, 0.0, 0.0};
    const float a = grad[G_A][gat];
    const float rho = LZ(L_RHO, 0), u = LZ(L_U, 0), v = LZ(L_V, 0), w = LZ(L_W, 0);
    const float rhof = 1.0f + rho;
    const float wc = w * c1z;
    const float Gzz = c1z * DZ1(L_W);
    double Rd[3] = {0.0, 0.0, 0.0};
    if (grp == 0) {
        // ------------------------------------------------------------ group A
        const float E = LZ(L_E, 0);
        float r0 = 0.0f, r4 = 0.0f, g0[4], g4[4], gT[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            g0[t] = -half * c1z * LZ(L_M2, ZT[t]);
            g4[t] = -c1z * ((half * LZ(L_E, ZT[t]) + LZ(L_P, ZT[t])) * LZ(L_W, ZT[t]));
            gT[t] = kz * LZ(L_T, ZT[t]);
        }
        const float gT0 = kz * LZ(L_T, 0);
        const float uc = u * c1x, vc = v * c1y;
        FLUX_BELOW(r0, g0);
        r0 -= half * (c1x * DX1(L_M0) + c1y * DY1(L_M1) + rhof * a
                      + uc * DX1(L_RHO) + vc * DY1(L_RHO));
        FLUX_ABOVE(r0, g0);
        r4 += g4[0];
        r4 -= gT[0];
        r4 -= 8.0f * g4[1];
        r4 += 16.0f * gT[1];
        r4 -= 30.0f * gT0;
        const float flux = c1x * DX1H() + c1y * DY1H();
        const float skew = E * a + uc * DX1(L_E) + vc * DY1(L_E);
        const float zmass = rhof * Gzz + wc * DZ1(L_RHO), zskew = E * Gzz + wc * DZ1(L_E);
        lds_barrier();
        r4 += -flux - half * skew + inv_re * vbuf[H_EN][pt] + kappa * vbuf[H_HEAT][pt];
        r4 += 8.0f * g4[2];
        r4 += 16.0f * gT[2];
        r4 -= g4[3];
        r4 -= gT[3];
        r0 = r0 - half * zmass;
        r4 = r4 - half * zskew + inv_re * vbuf[H_ZEN][pt];
        Rd[0] = (double)r0;
        Rd[1] = (double)r4;
        Rd[1] -= c.H_ref * ((double)a + (double)Gzz);
    } else if (grp == 1) {
        // ------------------------------------------------------------ group B
        const float m[3] = {LZ(L_M0, 0), LZ(L_M1, 0), LZ(L_M2, 0)};
        float r1 = 0.0f, r2 = 0.0f, r3 = 0.0f, g1[4], g2[4], g3[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float wt = LZ(L_W, ZT[t]);
            g1[t] = -half * c1z * (LZ(L_M0, ZT[t]) * wt);
            g2[t] = -half * c1z * (LZ(L_M1, ZT[t]) * wt);
            g3[t] = -c1z * (half * (LZ(L_M2, ZT[t]) * wt) + LZ(L_P, ZT[t]));
        }
        const float uc = u * c1x, vc = v * c1y;
        FLUX_BELOW(r1, g1);
        FLUX_BELOW(r2, g2);
        FLUX_BELOW(r3, g3);
        r1 -= half * (c1x * DX1P(L_M0, L_U) + c1y * DY1P(L_M0, L_V) + m[0] * a
                      + uc * DX1(L_M0) + vc * DY1(L_M0))
              + c1x * DX1(L_P);
        r2 -= half * (c1x * DX1P(L_M1, L_U) + c1y * DY1P(L_M1, L_V) + m[1] * a
                      + uc * DX1(L_M1) + vc * DY1(L_M1))
              + c1y * DY1(L_P);
        r3 -= half * (c1x * DX1P(L_M2, L_U) + c1y * DY1P(L_M2, L_V) + m[2] * a
                      + uc * DX1(L_M2) + vc * DY1(L_M2));
        const float z1 = rhof * u * Gzz + wc * DZMD(L_U);
        const float z2 = rhof * v * Gzz + wc * DZMD(L_V);
        const float z3 = rhof * w * Gzz + wc * DZMD(L_W);
        lds_barrier();
        r1 += inv_re * vbuf[H_VX][pt];
        r2 += inv_re * vbuf[H_VY][pt];
        r3 += inv_re * vbuf[H_VZ][pt];
        FLUX_ABOVE(r1, g1);
        FLUX_ABOVE(r2, g2);
        FLUX_ABOVE(r3, g3);
        r1 = r1 - half * z1;
        r2 = r2 - half * z2;
        r3 = r3 - half * z3;
        r1 += inv_re * vbuf[H_ZX][pt];
        r2 += inv_re * vbuf[H_ZY][pt];
        r3 += inv_re * vbuf[H_ZZ][pt];
        Rd[0] = (double)r1;
        Rd[1] = (double)r2;
        Rd[2] = (double)r3;
    } else {
        // ------------------------------------------------------------ group C
        const float Gxx = c1x * DX1(L_U), Gxy = c1y * DY1(L_U);
        const float Gyx = c1x * DX1(L_V), Gyy = c1y * DY1(L_V);
        const float Gzx = grad[G_B][gat], Gzy = grad[G_C][gat];
        {
            const float Vx = four3 * (c2x * DX2(L_U)) + c2y * DY2(L_U)
                             + third * (c1x * c1y * DXDY(L_V));
            const float Vy = c2x * DX2(L_V) + four3 * (c2y * DY2(L_V))
                             + third * (c1x * c1y * DYDX(L_U));
            const float Vz = c2x * DX2(L_W) + c2y * DY2(L_W);
            // tau_ij du_i/dx_j restricted to terms without a z derivative
            const float phi = 2.0f * (Gxx * Gxx + Gyy * Gyy) + Gxy * Gxy + Gyx * Gyx
                              + 2.0f * Gxy * Gyx + Gzx * Gzx + Gzy * Gzy;
            vbuf[H_VX][pt] = Vx;
            vbuf[H_VY][pt] = Vy;
            vbuf[H_VZ][pt] = Vz;
            vbuf[H_EN][pt] = u * Vx + v * Vy + w * Vz + phi;
            vbuf[H_HEAT][pt] = c2x * DX2(L_T) + c2y * DY2(L_T);
        }
        // The velocities again, opaque to the compiler: a product of them
        // shared with the in-plane terms would be rounded on its own instead
        // of fused into its sum, unlike in the march.
        float uz = u, vz = v, wz = w;
        asm volatile("" : "+v"(uz), "+v"(vz), "+v"(wz));
        const float Gxz = c1z * DZ1(L_U), Gyz = c1z * DZ1(L_V);
        const float Da = c1z * GZ(G_A), Db = c1z * GZ(G_B), Dc = c1z * GZ(G_C);
        const float Vx = c2z * DZ2(L_U, uz) + third * Db;
        const float Vy = c2z * DZ2(L_V, vz) + third * Dc;
        const float Vz = four3 * (c2z * DZ2(L_W, wz)) + third * Da;
        const float div = a + Gzz;
        const float phi = Gxz * Gxz + Gyz * Gyz + 2.0f * Gzz * Gzz
                          + 2.0f * (Gxz * Gzx + Gyz * Gzy) - two3 * div * div;
        vbuf[H_ZX][pt] = Vx;
        vbuf[H_ZY][pt] = Vy;
        vbuf[H_ZZ][pt] = Vz;
        vbuf[H_ZEN][pt] = uz * Vx + vz * Vy + wz * Vz + phi;
        if constexpr (DIAG) {
            const double ox = (double)(Gzy - Gyz), oy = (double)(Gxz - Gzx), oz = (double)(Gyx - Gxy);
            dsum[0] = 0.5 * (double)rhof * (ox * ox + oy * oy + oz * oz);
        }
        lds_barrier();
    }
#undef DZ1
#undef DZ2
#undef GZ
#undef DZMD
#undef FLUX_BELOW
#undef FLUX_ABOVE
#undef AT
#undef LV
#undef LZ
#undef DX1
#undef DY1
#undef DX1P
#undef DY1P
#undef HF
#undef DX1H
#undef DY1H
#undef DX2
#undef DY2
#undef DXDY
#undef DYDX

    // ---- RK update, output
    if (grp < 2 && active) {
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            if (grp == 0 && f == 2) continue;
            const int field = grp == 0 ? 4 * f : 1 + f;
            const double ref = grp == 1 ? 0.0 : f == 0 ? c.rho_ref : c.rhoE_ref;
            const int64_t i = field * N + pidx;
            const double qn = acc[f] + s.a_dt * Rd[f];
            if constexpr (MODE == 3)
                ((TOUT *)s.qout)[i] = qn;
            else
                ((TOUT *)s.qout)[i] = (float)(qn - ref);
            if constexpr (MODE < 3) s.acc_out[i] = acc[f] + s.b_dt * Rd[f];
        }
        if constexpr (DIAG) {
#pragma unroll
            for (int f = 0; f < 3; ++f) dsum[f] = acc[f];
            if (grp == 1) dsum[3] = 0.5 * (acc[0] * (double)u + acc[1] * (double)v + acc[2] * (double)w);
        }
    }

    if constexpr (DIAG) {
        // block sum of the diagnostics in a fixed order
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const double vsum = wave_sum(active ? dsum[d] : 0.0);
            if ((tid & 63) == 63) red[wave][d] = vsum;
        }
        lds_barrier();
        if (tid < kDiag) {
            // a record's slots by group: A 0 and 4, B 1, 2, 3 and 5, C 6 and 7 (zero)
            const int g = (tid & 3) == 0 ? 0 : tid < 6 ? 1 : 2;
            const int d = g == 0 ? tid >> 2 : g == 1 ? tid - 1 - (tid >> 2) : tid - 6;
            const int64_t blin = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
            double t = 0.0;
#pragma unroll
            for (int wv = 0; wv < NW / 3; ++wv) t += red[g * (NW / 3) + wv][d];
            s.diag_partial[blin * kDiag + tid] = t;
        }
    }
}

template <int BRZ>
static hipError_t launch_brick32_z(const Consts &c, const StageArgs &s, hipStream_t st)
{
    const dim3 block(3 * BRX * BRY * BRZ);
    const dim3 grid((c.nx + BRX - 1) / BRX, (c.ny + BRY - 1) / BRY,
                    (c.nz + BRZ - 1) / BRZ + (s.fin_out != nullptr));
    switch (s.mode) {
    case 1:
        if (s.diag_partial != nullptr)
            hipLaunchKernelGGL((brick32_stage_kernel<BRZ, 1, true>), grid, block, 0, st, c, s);
        else
            hipLaunchKernelGGL((brick32_stage_kernel<BRZ, 1, false>), grid, block, 0, st, c, s);
        break;
    case 2: hipLaunchKernelGGL((brick32_stage_kernel<BRZ, 2, false>), grid, block, 0, st, c, s); break;
    case 3: hipLaunchKernelGGL((brick32_stage_kernel<BRZ, 3, false>), grid, block, 0, st, c, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_brick32_stage(const Consts &c, const StageArgs &s, int bz, hipStream_t st)
{
    return bz == 2 ? launch_brick32_z<2>(c, s, st) : launch_brick32_z<4>(c, s, st);
}

}  // namespace ns
