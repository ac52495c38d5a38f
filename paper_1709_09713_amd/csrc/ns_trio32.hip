// ns_trio32.hip -- FP32-storage stage kernel with each column split over three
// groups of waves (tiles 8-10 of FP32 storage).
//
// A block marches a BX x BY column tile along z as the one-thread kernel
// (ns_fused.hip) does, with the same staged fields and the same expressions,
// and every sum adds its terms in that kernel's order, so that both give the
// same result bit for bit.  The equations of a column are split over three
// threads in different waves: A loads and stages the planes and holds mass and
// energy, B momentum, C the viscous terms, dissipation and heat conduction.
// C hands its values over through LDS: those of plane zp formed in the plane,
// and the z parts of plane zp - 2.  A and B take them in the next step, before
// the terms that the one-thread kernel adds after them, and finish plane zp - 3.
//
// Bound by vector issue and LDS reads: a plane of 32x8 points takes 1.2 us with
// one block (three waves per SIMD) on a compute unit, against 2.0 us in the
// one-thread kernel, whose single wave per SIMD waits for each of its
// dependent reads, and whose second block hides that only where there are
// blocks enough.  So it is the faster one on grids that give each compute unit
// a block or two (us per RK3 step, one thread -> three groups: 56^3 40.1 -> 37.4,
// 64^3 42.7 -> 40.2, 101x77x53 66.5 -> 63.0), and 4-8% slower on large ones, which
// memory bounds.  Two blocks a compute unit would need 80 registers: 93-300
// values spill.
#include <type_traits>

#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

namespace {

template <int V>
using TIC = std::integral_constant<int, V>;

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

template <int BX, int BY, int MODE, bool DIAG, bool PAIR>
__global__ void __launch_bounds__(3 * BX * BY) trio32_stage_kernel(Consts c, StageArgs s)
{
    // Multiply-adds are fused only within one expression, as in the one-thread
    // kernel.
#pragma clang fp contract(on)
    static_assert(!DIAG || MODE == 1, "diagnostics of the step's input state are taken in stage 1");
    using TIN = typename Types<MODE>::in;
    using TOUT = typename Types<MODE>::out;
    constexpr int HX = BX + 4, HY = BY + 4, HP = HX * HY, NT = BX * BY;
    static_assert(BX % 2 == 0 && HP % 2 == 0, "pairs need an even tile width and even LDS offsets");
    static_assert(NT % 64 == 0, "each group must be whole waves");
    constexpr int PW = PAIR ? 2 : 1;                      // points per load slot
    constexpr int NLOAD = (HP + PW * NT - 1) / (PW * NT);
    constexpr int NW = 3 * NT / 64;
    typedef TIN pair_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    enum { L_RHO, L_M0, L_M1, L_M2, L_E, L_U, L_V, L_W, L_P, L_T, NF };
    // handed over by C: of plane zp the in-plane viscous vector, its work with
    // the in-plane dissipation, and the in-plane heat conduction; of plane
    // zp - 2 the z parts of the first two
    enum { H_VX, H_VY, H_VZ, H_EN, H_HEAT, H_ZX, H_ZY, H_ZZ, H_ZEN, NH };
    __shared__ __attribute__((aligned(16))) float lds[2][NF][HP];
    __shared__ float vbuf[2][NH][NT];
    __shared__ double red[DIAG ? NW : 1][4];

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = wave / (NT / 64);
    const int pt = (int)threadIdx.x - grp * NT;
    const int tx = pt % BX, ty = pt / BX;
    int skip = 0;
    if constexpr (MODE == 2) {
        skip = finalize_layer(c, s);
        if (skip < 0) return;
    }
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz, skip);
    const int x0 = tbx * BX, y0 = tby * BY;
    const int z0 = tbz * s.zchunk;
    const int z1 = min(z0 + s.zchunk, c.nz);
    const int gx = x0 + tx, gy = y0 + ty;
    const bool active = (gx < c.nx) && (gy < c.ny);
    const int own = (ty + 2) * HX + tx + 2;
    const int64_t N = c.N;
    const int64_t col = active ? (int64_t)gy * c.nx + gx : 0;
    const TIN *qin = (const TIN *)s.qin;
    // stages 2 and 3 read the accumulator, stage 1 the state
    const double *accsrc = (MODE >= 2) ? s.acc_in : (const double *)s.qin;

    const float c1x = (float)c.c1[0], c1y = (float)c.c1[1], c1z = (float)c.c1[2];
    const float c2x = (float)c.c2[0], c2y = (float)c.c2[1], c2z = (float)c.c2[2];
    const float inv_re = (float)c.inv_re, kappa = (float)c.kappa;
    const float gm1 = (float)c.gm1, gM2 = (float)c.gM2;
    const float half = 0.5f, third = 1.0f / 3.0f, four3 = 4.0f / 3.0f, two3 = 2.0f / 3.0f;
    const float kz = kappa * c2z;

    // diagnostics of the column: group A mass and energy, B the momenta and
    // kinetic energy, C enstrophy
    double dsum[4] = {0.0, 0.0, 0.0, 0.0};

    // The march covers planes z0-2 .. z1+2 (A and B finish a plane three steps
    // after it was staged); planes beyond the halo are loaded (wrapped, valid
    // memory) but never output.
    const int zlast = z1 + 2;

// the value is computed here and not where a later plane's step uses it
#define KEEP(x) asm volatile("" : "+v"(x))
#define LV(f, dy, dx) lds[b][f][own + (dy) * HX + (dx)]
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
// D_y applied to D_x f (16 taps), unscaled
#define DYDX(f)                                                          \
    d1u(d1u(LV(f, -2, -2), LV(f, -2, -1), LV(f, -2, 1), LV(f, -2, 2)),   \
        d1u(LV(f, -1, -2), LV(f, -1, -1), LV(f, -1, 1), LV(f, -1, 2)),   \
        d1u(LV(f, 1, -2), LV(f, 1, -1), LV(f, 1, 1), LV(f, 1, 2)),       \
        d1u(LV(f, 2, -2), LV(f, 2, -1), LV(f, 2, 1), LV(f, 2, 2)))
#define DZ1(f) d1u(qz[SM4][f], qz[SM3][f], qz[SM1][f], qz[S0][f])
#define DZ2(f) d2u(qz[SM4][f], qz[SM3][f], qz[SM2][f], qz[SM1][f], qz[S0][f])
// the constant-coefficient flux g of plane zp, added to the planes around it
#define SCATTER(f, g)             \
    ra[SM2][f] -= g;              \
    ra[SM1][f] += 8.0f * (g);     \
    ra[SP1][f] -= 8.0f * (g);     \
    ra[SP2][f] = 0.0f + (g)
// ring slots: plane zp + k lives in slot (PH + k) mod 5
#define PHASES                                                                  \
    constexpr int PH = decltype(phc)::value;                                    \
    constexpr int S0 = PH, SM1 = (PH + 4) % 5, SM2 = (PH + 3) % 5;              \
    constexpr int SM3 = (PH + 2) % 5, SM4 = (PH + 1) % 5;                       \
    constexpr int SP1 = (PH + 1) % 5, SP2 = (PH + 2) % 5;                       \
    (void)S0, (void)SM1, (void)SM2, (void)SM3, (void)SM4, (void)SP1, (void)SP2
// the five phases of the ring, left at the last plane of the march
#define MARCH(step)                                       \
    for (int zp = z0 - 2;;) {                             \
        step(TIC<0>{}, zp);                               \
        if (++zp > zlast) break;                          \
        step(TIC<1>{}, zp);                               \
        if (++zp > zlast) break;                          \
        step(TIC<2>{}, zp);                               \
        if (++zp > zlast) break;                          \
        step(TIC<3>{}, zp);                               \
        if (++zp > zlast) break;                          \
        step(TIC<4>{}, zp);                               \
        if (++zp > zlast) break;                          \
    }

    auto acc_point = [&](int zf) {   // accumulator point of plane zf (a valid one outside the chunk)
        return (int64_t)((zf >= z0 && zf < z1) ? zf : z0) * c.nxy + col;
    };
    auto put = [&](int field, int64_t pidx, double acc, double R, double ref) {
        const int64_t i = field * N + pidx;
        const double q = acc + s.a_dt * R;
        if constexpr (MODE == 3)
            __builtin_nontemporal_store(q, (double *)s.qout + i);
        else
            __builtin_nontemporal_store((float)(q - ref), (float *)s.qout + i);
        if constexpr (MODE < 3) __builtin_nontemporal_store(acc + s.b_dt * R, s.acc_out + i);
    };

    if (grp == 0) {
        // ------------------------------------------------------------ group A
        enum { Z_RHO, Z_E, Z_W, NZ };
        enum { R_MASS, R_EN, NR };
        float qz[5][NZ], qa[5], ra[5][NR];
        float pend = 0.0f;                      // in-plane energy terms of plane zp - 1, without C's
        float f0 = 0.0f, f4 = 0.0f, fa = 0.0f, fg = 0.0f;   // plane zp - 3: residuals before C's part, div u
        double acc[2] = {0.0, 0.0}, accn[2] = {0.0, 0.0};   // of this and the next step's point
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            qa[q] = 0.0f;
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = 0.0f;
#pragma unroll
            for (int f = 0; f < NR; ++f) ra[q][f] = 0.0f;
        }
        // plane offsets and LDS cells of the points this thread loads;
        // lcell < 0 marks an unused slot
        int loff[NLOAD], lcell[NLOAD];
#pragma unroll
        for (int r = 0; r < NLOAD; ++r) {
            const int idx = PW * (pt + r * NT);
            lcell[r] = idx < HP ? idx : -1;
            loff[r] = 0;
            if (idx < HP) {
                int xx = (x0 + idx % HX - 2) % c.nx;
                if (xx < 0) xx += c.nx;
                int yy = (y0 + idx / HX - 2) % c.ny;
                if (yy < 0) yy += c.ny;
                loff[r] = yy * c.nx + xx;
            }
        }
        TIN pf[NLOAD][5][PW];   // plane zp + 1, staged in step zp
        TIN pg[NLOAD][5][PW];   // plane zp + 2, loaded in step zp
        auto load_plane = [&](int zp, TIN (&dst)[NLOAD][5][PW]) {
            // -2 <= zp <= nz + 4 and nz >= 5: one period
            const int64_t base = (int64_t)wrap1(zp, c.nz) * c.nxy;
#pragma unroll
            for (int r = 0; r < NLOAD; ++r)
#pragma unroll
                for (int f = 0; f < 5; ++f) {
                    if constexpr (PAIR) {
                        const pair_t v = *(const pair_t *)(qin + base + loff[r] + f * N);
                        dst[r][f][0] = v.x;
                        dst[r][f][1] = v.y;
                    } else {
                        dst[r][f][0] = qin[base + loff[r] + f * N];
                    }
                }
        };
        auto stage_plane = [&](int b) {
#pragma unroll
            for (int r = 0; r < NLOAD; ++r) {
                if (lcell[r] < 0) continue;
                float val[NF][PW];
#pragma unroll
                for (int j = 0; j < PW; ++j) {
                    float rho, m0, m1, m2, E;
                    if constexpr (MODE == 1) {
                        rho = (float)(pf[r][0][j] - c.rho_ref);
                        m0 = (float)pf[r][1][j];
                        m1 = (float)pf[r][2][j];
                        m2 = (float)pf[r][3][j];
                        E = (float)(pf[r][4][j] - c.rhoE_ref);
                    } else {
                        rho = pf[r][0][j];
                        m0 = pf[r][1][j];
                        m1 = pf[r][2][j];
                        m2 = pf[r][3][j];
                        E = pf[r][4][j];
                    }
                    const float rhof = 1.0f + rho;
                    const float inv = recip_f32(rhof);
                    const float u = m0 * inv, v = m1 * inv, w = m2 * inv;
                    const float p = gm1 * (E - half * (m0 * u + m1 * v + m2 * w));
                    val[L_RHO][j] = rho;
                    val[L_M0][j] = m0;
                    val[L_M1][j] = m1;
                    val[L_M2][j] = m2;
                    val[L_E][j] = E;
                    val[L_U][j] = u;
                    val[L_V][j] = v;
                    val[L_W][j] = w;
                    val[L_P][j] = p;
                    val[L_T][j] = (gM2 * p - rho) * inv;
                }
                const int i = lcell[r];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    if constexpr (PAIR) {
                        f2_t v2;
                        v2.x = val[f][0];
                        v2.y = val[f][1];
                        ((f2_t *)&lds[b][f][0])[i >> 1] = v2;
                    } else {
                        lds[b][f][i] = val[f][0];
                    }
                }
            }
        };
        auto next_plane = [&]() {
#pragma unroll
            for (int r = 0; r < NLOAD; ++r)
#pragma unroll
                for (int f = 0; f < 5; ++f)
#pragma unroll
                    for (int j = 0; j < PW; ++j) pf[r][f][j] = pg[r][f][j];
        };

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 3;
            const bool do_fin = (zf >= z0 && zf < z1);
            // Plane zp + 2 and the accumulator of the next step's point are
            // loaded now, before this step's stores: vector memory counters
            // retire loads and stores in issue order, so a load issued after
            // a store could only be waited for together with that store.
            load_plane(zp + 2, pg);
            {
                const int64_t pn = acc_point(zf + 1);
                acc[0] = accn[0];
                acc[1] = accn[1];
                accn[0] = __builtin_nontemporal_load(accsrc + pn);
                accn[1] = __builtin_nontemporal_load(accsrc + 4 * N + pn);
            }
            // in-plane energy terms of plane zp - 1 with C's (outside the
            // chunk an undefined value, in a residual that is never output)
            ra[SM1][R_EN] += pend + inv_re * vbuf[b ^ 1][H_EN][pt] + kappa * vbuf[b ^ 1][H_HEAT][pt];
            const float rho = LV(L_RHO, 0, 0), E = LV(L_E, 0, 0), w = LV(L_W, 0, 0);
            {
                const float g0 = -half * c1z * LV(L_M2, 0, 0);               // -1/2 d(rho w)/dz
                const float g4 = -c1z * ((half * E + LV(L_P, 0, 0)) * w);    // -1/2 d(rhoE w)/dz - d(p w)/dz
                const float gT = kz * LV(L_T, 0, 0);                         // kappa d2T/dz2
                SCATTER(R_MASS, g0);
                SCATTER(R_EN, g4);
                ra[SM2][R_EN] -= gT;
                ra[SM1][R_EN] += 16.0f * gT;
                ra[S0][R_EN] -= 30.0f * gT;
                ra[SP1][R_EN] += 16.0f * gT;
                ra[SP2][R_EN] -= gT;
            }
            qz[S0][Z_RHO] = rho;
            qz[S0][Z_E] = E;
            qz[S0][Z_W] = w;
            if (zp >= z0 && zp < z1) {
                const float u = LV(L_U, 0, 0), v = LV(L_V, 0, 0);
                const float Gxx = c1x * DX1(L_U), Gyy = c1y * DY1(L_V);
                const float a = Gxx + Gyy;
                const float rhof = 1.0f + rho;
                const float uc = u * c1x, vc = v * c1y;
                ra[S0][R_MASS] -= half * (c1x * DX1(L_M0) + c1y * DY1(L_M1) + rhof * a
                                          + uc * DX1(L_RHO) + vc * DY1(L_RHO));
                // skew convection and pressure work
                pend = -(c1x * DX1H() + c1y * DY1H())
                       - half * (E * a + uc * DX1(L_E) + vc * DY1(L_E));
                qa[S0] = a;
                KEEP(pend);
                KEEP(qa[S0]);
            }
#pragma unroll
            for (int f = 0; f < NR; ++f) {
                KEEP(ra[SM2][f]);
                KEEP(ra[SM1][f]);
                KEEP(ra[S0][f]);
                KEEP(ra[SP1][f]);
                KEEP(ra[SP2][f]);
            }

            // stage plane zp + 1 into the other buffer (last read in the
            // previous step, before its barrier)
            stage_plane(b ^ 1);

            // finish plane zp - 3: C's part, RK update, output
            if (do_fin) {
                const float R4 = f4 + inv_re * vbuf[b ^ 1][H_ZEN][pt];
                double Rd = (double)R4;
                Rd -= c.H_ref * ((double)fa + (double)fg);
                if (active) {
                    const int64_t pidx = (int64_t)zf * c.nxy + col;
                    if constexpr (DIAG) {
                        dsum[0] += acc[0];
                        dsum[1] += acc[1];
                    }
                    put(0, pidx, acc[0], (double)f0, c.rho_ref);
                    put(4, pidx, acc[1], Rd, c.rhoE_ref);
                }
            }
            // plane zp - 2: gathered z terms
            {
                const float rf = 1.0f + qz[SM2][Z_RHO], Ef = qz[SM2][Z_E];
                const float wc = qz[SM2][Z_W] * c1z;
                const float Gzz = c1z * DZ1(Z_W);
                f0 = ra[SM2][R_MASS] - half * (rf * Gzz + wc * DZ1(Z_RHO));
                f4 = ra[SM2][R_EN] - half * (Ef * Gzz + wc * DZ1(Z_E));
                fa = qa[SM2];
                fg = Gzz;
                KEEP(f0);
                KEEP(f4);
                KEEP(fg);
            }
            next_plane();
            lds_barrier();
        };

        load_plane(z0 - 2, pf);
        stage_plane(0);
        load_plane(z0 - 1, pf);
        lds_barrier();
        MARCH(step)
    } else if (grp == 1) {
        // ------------------------------------------------------------ group B
        enum { Z_MU, Z_MV, Z_MW, Z_W, NZ };     // rho u, rho v, rho w from the staged rho and u_i; w
        float qz[5][NZ], ra[5][3];
        float fr[3] = {0.0f, 0.0f, 0.0f};       // plane zp - 3: residuals before C's part
        float qu[DIAG ? 4 : 1][3];              // u, v, w of planes zp .. zp - 3
        double acc[3] = {0.0, 0.0, 0.0}, accn[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 5; ++q) {
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = 0.0f;
#pragma unroll
            for (int f = 0; f < 3; ++f) ra[q][f] = 0.0f;
        }
#pragma unroll
        for (int q = 0; q < (DIAG ? 4 : 1); ++q) qu[q][0] = qu[q][1] = qu[q][2] = 0.0f;

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 3;
            const bool do_fin = (zf >= z0 && zf < z1);
            {
                const int64_t pn = acc_point(zf + 1);
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    acc[f] = accn[f];
                    accn[f] = __builtin_nontemporal_load(accsrc + (1 + f) * N + pn);
                }
            }
            // the in-plane viscous terms of plane zp - 1 (see group A)
#pragma unroll
            for (int f = 0; f < 3; ++f) ra[SM1][f] += inv_re * vbuf[b ^ 1][H_VX + f][pt];
            const float m0 = LV(L_M0, 0, 0), m1 = LV(L_M1, 0, 0), m2 = LV(L_M2, 0, 0);
            const float u = LV(L_U, 0, 0), v = LV(L_V, 0, 0), w = LV(L_W, 0, 0);
            {
                const float g1 = -half * c1z * (m0 * w);                     // -1/2 d(rho u w)/dz
                const float g2 = -half * c1z * (m1 * w);                     // -1/2 d(rho v w)/dz
                const float g3 = -c1z * (half * (m2 * w) + LV(L_P, 0, 0));   // -1/2 d(rho w w)/dz - dp/dz
                SCATTER(0, g1);
                SCATTER(1, g2);
                SCATTER(2, g3);
                const float rhof = 1.0f + LV(L_RHO, 0, 0);
                qz[S0][Z_MU] = rhof * u;
                qz[S0][Z_MV] = rhof * v;
                qz[S0][Z_MW] = rhof * w;
                qz[S0][Z_W] = w;
            }
            if (zp >= z0 && zp < z1) {
                const float Gxx = c1x * DX1(L_U), Gyy = c1y * DY1(L_V);
                const float a = Gxx + Gyy;
                const float uc = u * c1x, vc = v * c1y;
                ra[S0][0] -= half * (c1x * DX1P(L_M0, L_U) + c1y * DY1P(L_M0, L_V) + m0 * a
                                     + uc * DX1(L_M0) + vc * DY1(L_M0))
                             + c1x * DX1(L_P);
                ra[S0][1] -= half * (c1x * DX1P(L_M1, L_U) + c1y * DY1P(L_M1, L_V) + m1 * a
                                     + uc * DX1(L_M1) + vc * DY1(L_M1))
                             + c1y * DY1(L_P);
                ra[S0][2] -= half * (c1x * DX1P(L_M2, L_U) + c1y * DY1P(L_M2, L_V) + m2 * a
                                     + uc * DX1(L_M2) + vc * DY1(L_M2));
            }
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                KEEP(qz[S0][f]);
                KEEP(ra[SM2][f]);
                KEEP(ra[SM1][f]);
                KEEP(ra[S0][f]);
                KEEP(ra[SP1][f]);
                KEEP(ra[SP2][f]);
            }
            // finish plane zp - 3: C's part, RK update, output
            if (do_fin) {
                float R[3];
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    R[f] = fr[f];
                    R[f] += inv_re * vbuf[b ^ 1][H_ZX + f][pt];
                }
                if (active) {
                    const int64_t pidx = (int64_t)zf * c.nxy + col;
                    if constexpr (DIAG) {
#pragma unroll
                        for (int f = 0; f < 3; ++f) dsum[f] += acc[f];
                        dsum[3] += 0.5 * (acc[0] * (double)qu[2][0] + acc[1] * (double)qu[2][1]
                                          + acc[2] * (double)qu[2][2]);
                    }
#pragma unroll
                    for (int f = 0; f < 3; ++f) put(1 + f, pidx, acc[f], (double)R[f], 0.0);
                }
            }
            // plane zp - 2: gathered z terms
            {
                const float wc = qz[SM2][Z_W] * c1z;
                const float Gzz = c1z * DZ1(Z_W);
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    fr[f] = ra[SM2][f] - half * (qz[SM2][f] * Gzz + wc * DZ1(f));
                    KEEP(fr[f]);
                }
            }
            if constexpr (DIAG) {
#pragma unroll
                for (int f = 0; f < 3; ++f) {
                    qu[2][f] = qu[1][f];
                    qu[1][f] = qu[0][f];
                }
                qu[0][0] = u;
                qu[0][1] = v;
                qu[0][2] = w;
            }
            lds_barrier();
        };

        lds_barrier();   // group A's prologue
        MARCH(step)
    } else {
        // ------------------------------------------------------------ group C
        enum { Z_U, Z_V, Z_W, NZ };
        float qz[5][NZ];                // ring: u, v, w of the own column
        float qa[5], qb[5], qc[5];      // ring: D_x u + D_y v, D_x w, D_y w
        float qo[DIAG ? 5 : 1][2];      // rho and omega_z of planes zp .. zp - 2
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            qa[q] = qb[q] = qc[q] = 0.0f;
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = 0.0f;
        }
#pragma unroll
        for (int q = 0; q < (DIAG ? 5 : 1); ++q) qo[q][0] = qo[q][1] = 0.0f;
        const int hx = (tx < 2) ? -2 : (tx >= BX - 2 ? 2 : 0);
#define LVH(f, dy) lds[b][f][own + (dy) * HX + hx]

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 2;
            const bool do_fin = (zf >= z0 && zf < z1);
            const float u = LV(L_U, 0, 0), v = LV(L_V, 0, 0), w = LV(L_W, 0, 0);
            const float dyv = DY1(L_V);
            const float Gxx = c1x * DX1(L_U), Gyy = c1y * dyv;
            const float Gzx = c1x * DX1(L_W), Gzy = c1y * DY1(L_W);
            const float a = Gxx + Gyy;
            qz[S0][Z_U] = u;
            qz[S0][Z_V] = v;
            qz[S0][Z_W] = w;
            qa[S0] = a;
            qb[S0] = Gzx;
            qc[S0] = Gzy;
            if (zp >= z0 && zp < z1) {
                const float Gxy = c1y * DY1(L_U), Gyx = c1x * DX1(L_V);
                // D_x applied to D_y v: the x-stencil across the row's lanes,
                // whose two ends take the y-derivative at their halo column
                const float hv = d1u(LVH(L_V, -2), LVH(L_V, -1), LVH(L_V, 1), LVH(L_V, 2));
                const float dxdyv = d1u_x_lanes<BX>(dyv, hv, tx);
                const float Vx = four3 * (c2x * DX2(L_U)) + c2y * DY2(L_U)
                                 + third * (c1x * c1y * dxdyv);
                const float Vy = c2x * DX2(L_V) + four3 * (c2y * DY2(L_V))
                                 + third * (c1x * c1y * DYDX(L_U));
                const float Vz = c2x * DX2(L_W) + c2y * DY2(L_W);
                // tau_ij du_i/dx_j restricted to terms without a z derivative
                const float phi = 2.0f * (Gxx * Gxx + Gyy * Gyy) + Gxy * Gxy + Gyx * Gyx
                                  + 2.0f * Gxy * Gyx + Gzx * Gzx + Gzy * Gzy;
                vbuf[b][H_VX][pt] = Vx;
                vbuf[b][H_VY][pt] = Vy;
                vbuf[b][H_VZ][pt] = Vz;
                vbuf[b][H_EN][pt] = u * Vx + v * Vy + w * Vz + phi;
                vbuf[b][H_HEAT][pt] = c2x * DX2(L_T) + c2y * DY2(L_T);
                if constexpr (DIAG) {
                    qo[S0][0] = LV(L_RHO, 0, 0);
                    qo[S0][1] = Gyx - Gxy;
                }
            }
            KEEP(qz[S0][Z_U]);
            KEEP(qz[S0][Z_V]);
            KEEP(qz[S0][Z_W]);
            KEEP(qa[S0]);
            KEEP(qb[S0]);
            KEEP(qc[S0]);
            // plane zp - 2: z parts
            if (do_fin) {
                const float uf = qz[SM2][Z_U], vf = qz[SM2][Z_V], wf = qz[SM2][Z_W];
                const float af = qa[SM2], bb = qb[SM2], cc = qc[SM2];
                const float Gxz = c1z * DZ1(Z_U), Gyz = c1z * DZ1(Z_V), Gzz = c1z * DZ1(Z_W);
                const float Da = c1z * d1u(qa[SM4], qa[SM3], qa[SM1], qa[S0]);
                const float Db = c1z * d1u(qb[SM4], qb[SM3], qb[SM1], qb[S0]);
                const float Dc = c1z * d1u(qc[SM4], qc[SM3], qc[SM1], qc[S0]);
                const float Vx = c2z * DZ2(Z_U) + third * Db;
                const float Vy = c2z * DZ2(Z_V) + third * Dc;
                const float Vz = four3 * (c2z * DZ2(Z_W)) + third * Da;
                const float div = af + Gzz;
                const float phi = Gxz * Gxz + Gyz * Gyz + 2.0f * Gzz * Gzz
                                  + 2.0f * (Gxz * bb + Gyz * cc) - two3 * div * div;
                vbuf[b][H_ZX][pt] = Vx;
                vbuf[b][H_ZY][pt] = Vy;
                vbuf[b][H_ZZ][pt] = Vz;
                vbuf[b][H_ZEN][pt] = uf * Vx + vf * Vy + wf * Vz + phi;
                if constexpr (DIAG) {
                    if (active) {
                        const double ox = (double)(cc - Gyz), oy = (double)(Gxz - bb), oz = (double)qo[SM2][1];
                        dsum[0] += 0.5 * (double)(1.0f + qo[SM2][0]) * (ox * ox + oy * oy + oz * oz);
                    }
                }
            }
            lds_barrier();
        };

        lds_barrier();   // group A's prologue
        MARCH(step)
#undef LVH
    }
#undef KEEP
#undef LV
#undef DX1
#undef DY1
#undef DX1P
#undef DY1P
#undef HF
#undef DX1H
#undef DY1H
#undef DX2
#undef DY2
#undef DYDX
#undef DZ1
#undef DZ2
#undef SCATTER
#undef PHASES
#undef MARCH

    if constexpr (DIAG) {
        // block sum of the diagnostics in a fixed order
        const int tid = threadIdx.x;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const double vsum = wave_sum(dsum[d]);
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

namespace {

template <int BX, int BY, bool PAIR>
hipError_t launch_trio32_p(const Consts &c, const StageArgs &s, hipStream_t st)
{
    const dim3 block(3 * BX * BY, 1, 1);
    const dim3 grid((c.nx + BX - 1) / BX, (c.ny + BY - 1) / BY,
                    (c.nz + s.zchunk - 1) / s.zchunk + (s.fin_out != nullptr));
    switch (s.mode) {
    case 1:
        if (s.diag_partial != nullptr)
            hipLaunchKernelGGL((trio32_stage_kernel<BX, BY, 1, true, PAIR>), grid, block, 0, st, c, s);
        else
            hipLaunchKernelGGL((trio32_stage_kernel<BX, BY, 1, false, PAIR>), grid, block, 0, st, c, s);
        break;
    case 2: hipLaunchKernelGGL((trio32_stage_kernel<BX, BY, 2, false, PAIR>), grid, block, 0, st, c, s); break;
    case 3: hipLaunchKernelGGL((trio32_stage_kernel<BX, BY, 3, false, PAIR>), grid, block, 0, st, c, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The halo plane is loaded in x-neighbour pairs when nx is even: pairs start
// at even x, so they never straddle the periodic wrap.
template <int BX, int BY>
hipError_t launch_trio32(const Consts &c, const StageArgs &s, hipStream_t st)
{
    return c.nx % 2 == 0 ? launch_trio32_p<BX, BY, true>(c, s, st) : launch_trio32_p<BX, BY, false>(c, s, st);
}

template <int BX, int BY>
int resident_trio32()
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per, reinterpret_cast<const void *>(&trio32_stage_kernel<BX, BY, 2, false, true>), 3 * BX * BY, 0) != hipSuccess)
        return 0;
    return cus * (per > 0 ? per : 1);
}

}  // namespace

int trio32_resident_blocks(int tile)
{
    switch (tile) {
    case TILE_16x8_3G: return resident_trio32<16, 8>();
    case TILE_32x8_3G: return resident_trio32<32, 8>();
    case TILE_16x4_3G: return resident_trio32<16, 4>();
    default: return 0;
    }
}

hipError_t launch_trio32_stage(const Consts &c, const StageArgs &s, int tile, hipStream_t st)
{
    switch (tile) {
    case TILE_16x8_3G: return launch_trio32<16, 8>(c, s, st);
    case TILE_32x8_3G: return launch_trio32<32, 8>(c, s, st);
    case TILE_16x4_3G: return launch_trio32<16, 4>(c, s, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ns
