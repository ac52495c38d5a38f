// ns_trio.hip -- the fused on-the-fly FP64 stage kernel with the work of each
// grid point split between three groups of waves (tiles 8-10; tile 9, 32x8,
// is the FP64 default).
//
// Same algorithm class as the one-thread-per-column kernel of ns_fused.hip
// (minimal storage: every derivative of the governing-equations section is
// evaluated on the fly from an LDS-staged (x, y) tile marching along z, the
// low-storage RK3 update of the generic-algorithm figure in the same pass),
// but a block holds three threads per column of its tile:
//  * group A (threads [0, NT)) loads and stages each plane and evaluates the
//    energy equation with heat conduction, and the pressure gradient;
//  * group B evaluates the mass and momentum equations;
//  * group C evaluates div u, the viscous vector V_i = lap u_i + (1/3) d_i
//    div u and the viscous work and dissipation.
// The groups hand values over through vbuf, double buffered like the planes:
// what one writes in the step of plane zp another reads in the next step,
// after the plane barrier.  C finishes plane zp - 2 in that step, A and B
// finish plane zp - 3.
//
// Arithmetic.  The skew-symmetric convective terms are taken in differences to
// the point's own value: with the first-derivative weights c_k (odd in k, so
// they sum to zero)
//   1/2 [D(f u) + f D u + u D f] = f_0 D u + sum_k c_k (f_k - f_0) (u_0 + u_k) / 2,
// one subtraction and one multiply-add per tap where the three stencils of the
// left side take about twice that, and f_0 div u once per point.  Along z the
// term of a pair of planes is formed once and added to both, so a residual is
// complete two planes on and no ring of five planes is needed (the viscous
// vector and the velocity gradient still gather from one).  Pressure enters by
// its differences too, formed from those of energy and kinetic energy:
//   D(p u) = p_0 D u + sum_k c_k (p_k - p_0) u_k.
// Differences lose nothing to a large mean, whatever it is.  No reference state
// is taken out: a caller's density and energy need not be near any, and those
// below it would lose their low bits.  Temperature is staged as the specific
// internal energy e, one rounding less.  Relative rms error of the residual
// (mass, worst momentum, energy) against 80-bit arithmetic, 64x40x28, the
// two-group kernel that formed the stencils of the full fields -> deviations
// from a reference state -> here: random state at M = 0.1 1.8e-16 2.2e-13
// 2.4e-16 -> 1.9e-16 1.7e-15 2.0e-16 -> 1.6e-16 2.0e-16 1.7e-16; the same with
// density and energy times 1e-4 1.8e-16 6.7e-16 3.9e-14 -> 3.8e-12 6.6e-12
// 3.0e-10 -> 1.6e-16 4.5e-16 3.4e-14; inviscid, p = 1 at M = 1e-3 1.8e-16 6.0e-15
// 2.1e-16 -> 1.9e-16 2.1e-9 1.2e-10 -> 1.6e-16 1.6e-16 1.7e-16; mean flow 4.8e-15
// 1.2e-14 5.7e-15 -> 4.6e-15 1.7e-14 1.1e-14 -> 3.3e-15 2.7e-15 3.3e-15.  Against
// the deviations a step costs 0 (256^3) to 2% (64^3, 101x77x53) more: one addition
// per pressure tap, and div u times the point's own values.  (Heat conduction is
// group A's, which needs it: in B and handed over, 512^3 took 13.24 ms instead of
// 13.03, 101x77x53 79.9 us instead of 77.5.)
//
// What bounds it: at 512^3 a stage moves 18-24 GB (4.2 ms at the rate of a
// plain kernel of the same access pattern for stage 2, 3.2 ms for stages 1
// and 3) and needs about 3.2 ms of LDS and vector issue when its planes come
// from L2 (measured before the differences); a stage takes 4.2-4.6 ms because one barrier per plane keeps the
// groups in step, so the three do not overlap fully.  Two groups (momentum |
// the rest) at two waves per SIMD had 30 dependent LDS waits per plane in the
// longer group; three groups of about equal length fit 168 registers, three
// waves per SIMD, and hide them better.  Measured (ms per step without
// diagnostics, two groups -> three): 512^3 13.99 -> 12.92, 256^3 1.739 ->
// 1.571, 192^3 0.843 -> 0.735, 101x77x53 0.0884 -> 0.0753, 64^3 0.0552 ->
// 0.0483 (on small grids also because the march ends at its last plane instead
// of at a multiple of five).
#include <type_traits>

#include "ns_common.hpp"
#include "ns_fp64.hpp"
#include "ns_kernels.hpp"

namespace ns {

namespace {

typedef double d2_t __attribute__((ext_vector_type(2)));

template <int V>
using TIC = std::integral_constant<int, V>;

}  // namespace

// MODE: 0 = residual only (R to s.rout), 1..3 = RK stage.
// GRAD: the intermediate-storage class: group C takes the nine velocity
// gradients from the arrays that rs_gradient_kernel wrote (s.grad) instead of
// evaluating them, and the mixed viscous derivatives are first derivatives of
// the stored diagonal ones.
template <int BX, int BY, int MODE, bool DIAG, bool PAIR, bool GRAD>
__global__ void __launch_bounds__(3 * BX * BY) __attribute__((amdgpu_waves_per_eu(BX * BY >= 128 ? 3 : 2)))
trio_stage_kernel(Consts c, Coef64 k, StageArgs s)
{
    // Multiply-adds are fused only within one expression, never across
    // statements: the march's five phases are compiled separately, and
    // fusion across statements can differ between them, which would make a
    // point's rounding depend on where its plane falls in a z-chunk.
#pragma clang fp contract(on)
    static_assert(!DIAG || (MODE == 1 && !GRAD), "diagnostics of the step's input state are taken in stage 1");
    constexpr int HX = BX + 4, HY = BY + 4, HP = HX * HY, NT = BX * BY;
    static_assert(BX % 2 == 0 && HP % 2 == 0, "pairs need an even tile width and even LDS offsets");
    constexpr int PW = PAIR ? 2 : 1;                      // points per load slot
    constexpr int NLOAD = (HP + PW * NT - 1) / (PW * NT);
    constexpr int NW = 3 * NT / 64;
    static_assert(NT % 64 == 0, "each group must be whole waves");
    // staged fields: rho, rho u_i, E, u, v, w, kinetic energy, e = T / (gamma (gamma - 1) M^2)
    enum { L_R, L_M0, L_M1, L_M2, L_E, L_U, L_V, L_W, L_K, L_T, NF };
    // handed over: V, dissipative energy terms and div u of plane zp - 2 (C),
    // pressure gradient, in-plane of plane zp and along z of plane zp - 2 (A);
    // with diagnostics omega_z of plane zp and omega_x, omega_y of plane zp - 2
    // (C)
    enum { H_VX, H_VY, H_VZ, H_EN, H_DIV, H_PX, H_PY, H_PZ, H_OZ, H_OX, H_OY };
    __shared__ __attribute__((aligned(16))) double lds[2][NF][HP];
    __shared__ double vbuf[2][DIAG ? 11 : 8][NT];
    __shared__ double red[NW][kDiag];
    __shared__ double sbuf[GRAD ? 2 : 1][GRAD ? HY : 1][BX];   // GRAD: D_x u + D_z w with two halo rows each side

    // The group is a property of the wave; reading it through a scalar
    // register makes the branches below scalar branches, so each wave runs
    // exactly one group's march (and its barriers).
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int grp = wave / (NT / 64);
    const int pt = (int)threadIdx.x - grp * NT;
    const int tx = pt % BX, ty = pt / BX;
    int skip = 0;
    if constexpr (MODE == 2 && !GRAD) {
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

    const double c1x = c.c1[0], c1y = c.c1[1], c1z = c.c1[2];
    const double c2x = c.c2[0], c2y = c.c2[1], c2z = c.c2[2];
    const double inv_re = c.inv_re;

    // per-column diagnostic sums of stage 1, added in program order
    // (deterministic): group A energy, kinetic energy and enstrophy, group B
    // mass and momenta
    double dr[4] = {0.0, 0.0, 0.0, 0.0};

    // The march covers planes z0-2 .. z1+2 (A and B finish a plane three
    // steps after it was staged); planes beyond the halo are loaded (wrapped,
    // valid memory) but never output.
    const int zlast = z1 + 2;
    const double *qin = (const double *)s.qin;
    // stages 2 and 3 read the accumulator, stage 1 the state
    const double *accsrc = (MODE >= 2) ? s.acc_in : qin;

#define LV(f, dy, dx) lds[b][f][own + (dy) * HX + (dx)]
#define TAPS_X(t, f) const double t[4] = {LV(f, 0, -2), LV(f, 0, -1), LV(f, 0, 1), LV(f, 0, 2)}
#define TAPS_Y(t, f) const double t[4] = {LV(f, -2, 0), LV(f, -1, 0), LV(f, 1, 0), LV(f, 2, 0)}
#define D1T(t) d1(t[0], t[1], t[2], t[3])
#define D2T(t, t0) d2(t[0], t[1], t0, t[2], t[3])
// Makes a value be computed here.  Left alone, the compiler moves arithmetic
// whose result is used in a later plane's step into that step and keeps its
// operands, many more, in registers: up to 445 spilled registers in group C,
// none with this.
#define KEEP(x) asm volatile("" : "+v"(x))
// Scheduling fence of the narrow tiles' group C: without it their reads run
// ahead until registers spill (16x8: 2.00 -> 1.76 ms per step at 256^3); the
// 32-wide tile does not spill and is 1% faster without.
#define SB() do { if constexpr (BX < 32) __builtin_amdgcn_sched_barrier(0); } while (0)
// |c_k| (u_0 + u_k) / 2 with the first-derivative weights c_k
#define HALF_SUMS(s, u0, t, w4, wh)                                                               \
    const double s[4] = {(wh) * ((u0) + t[0]), (w4) * ((u0) + t[1]), (w4) * ((u0) + t[2]), (wh) * ((u0) + t[3])}
#define DZ1(f) d1(qz[SM4][f], qz[SM3][f], qz[SM1][f], qz[S0][f])
#define DZ2(f) d2(qz[SM4][f], qz[SM3][f], qz[SM2][f], qz[SM1][f], qz[S0][f])
#define PHASES                                                                  \
    constexpr int PH = decltype(phc)::value;                                    \
    constexpr int S0 = PH, SM1 = (PH + 4) % 5, SM2 = (PH + 3) % 5;              \
    constexpr int SM3 = (PH + 2) % 5, SM4 = (PH + 1) % 5;                       \
    (void)S0, (void)SM1, (void)SM2, (void)SM3, (void)SM4
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

    if (grp == 0) {
        // ------------------------------------------------------------ group A
        // Group A alone loads: pairs of points with one 16-byte load each
        // (even nx).  Sharing the loads between A and B, one point per
        // thread, balances the arithmetic better but was 10% slower.
        enum { Z_E, Z_K, Z_W, Z_T, Z_R, NZ };
        enum { R_EN, R_PZ, NR };
        double qz[5][NZ];      // E, kinetic energy (with diagnostics rho) of planes zp .. zp - 3, w and T of zp .. zp - 2
        double ra[5][NR];      // pending energy residual and pressure gradient along z
        double acc = 0.0, accn = 0.0;   // of this and the next step's point
#pragma unroll
        for (int q = 0; q < 5; ++q) {
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = 0.0;
#pragma unroll
            for (int f = 0; f < NR; ++f) ra[q][f] = 0.0;
        }

        // Plane offsets and LDS cells of the points this thread loads;
        // lcell < 0 marks an unused slot.
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
        double pf[NLOAD][5][PW];   // plane zp + 1, staged in step zp
        double pg[NLOAD][5][PW];   // plane zp + 2, loaded in step zp
        auto load_plane = [&](int zp, double (&dst)[NLOAD][5][PW]) {
            int zw = zp % c.nz;
            if (zw < 0) zw += c.nz;
            const int64_t base = (int64_t)zw * c.nxy;
#pragma unroll
            for (int r = 0; r < NLOAD; ++r)
#pragma unroll
                for (int f = 0; f < 5; ++f) {
                    if constexpr (PAIR) {
                        const d2_t v = *(const d2_t *)(qin + base + loff[r] + f * N);
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
                double val[NF][PW];
#pragma unroll
                for (int j = 0; j < PW; ++j) {
                    const double rho = pf[r][0][j], m0 = pf[r][1][j], m1 = pf[r][2][j], m2 = pf[r][3][j];
                    const double E = pf[r][4][j];
                    const double inv = recip_f64(rho);
                    const double u = quotient_f64(m0, rho, inv);
                    const double v = quotient_f64(m1, rho, inv);
                    const double w = quotient_f64(m2, rho, inv);
                    const double ke = 0.5 * (m0 * u + m1 * v + m2 * w);
                    val[L_R][j] = rho;
                    val[L_M0][j] = m0;
                    val[L_M1][j] = m1;
                    val[L_M2][j] = m2;
                    val[L_E][j] = E;
                    val[L_U][j] = u;
                    val[L_V][j] = v;
                    val[L_W][j] = w;
                    val[L_K][j] = ke;
                    val[L_T][j] = (E - ke) * inv;
                }
                const int i = lcell[r];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    if constexpr (PAIR) {
                        d2_t v2;
                        v2.x = val[f][0];
                        v2.y = val[f][1];
                        ((d2_t *)&lds[b][f][0])[i >> 1] = v2;
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
            const bool do_plane = (zp >= z0 && zp < z1);
            // Plane zp + 2 and the accumulator of the next step's point are
            // loaded now, before this step's stores: vector memory counters
            // retire loads and stores in issue order, so a load issued after
            // a store could only be waited for together with that store.
            // Idle lanes read a valid address they ignore.
            load_plane(zp + 2, pg);
            if constexpr (MODE >= 1) {
                const int64_t pn = acc_point(zf + 1);
                acc = accn;
                accn = __builtin_nontemporal_load(accsrc + 4 * N + pn);
            }
            const double E = LV(L_E, 0, 0), ke = LV(L_K, 0, 0), w = LV(L_W, 0, 0), T = LV(L_T, 0, 0);
            double re = 0.0;
            if (do_plane) {
                const double u = LV(L_U, 0, 0), v = LV(L_V, 0, 0);
                {
                    TAPS_X(ut, L_U);
                    TAPS_X(et, L_E);
                    TAPS_X(kt, L_K);
                    TAPS_X(tt, L_T);
                    HALF_SUMS(su, u, ut, k.x4, k.xh);
                    double dE[4], dp[4];
                    diffs(E, et, dE);
                    pressure_diffs(dE, ke, kt, dp);
                    re = conv(re, dE, su);
                    re = __builtin_fma(-k.gx, d1_prod(dp, ut), re);
                    re = __builtin_fma(k.kx, D2T(tt, T), re);
                    vbuf[b][H_PX][pt] = k.gx * D1T(dp);
                }
                {
                    TAPS_Y(vt, L_V);
                    TAPS_Y(et, L_E);
                    TAPS_Y(kt, L_K);
                    TAPS_Y(tt, L_T);
                    HALF_SUMS(sv, v, vt, k.y4, k.yh);
                    double dE[4], dp[4];
                    diffs(E, et, dE);
                    pressure_diffs(dE, ke, kt, dp);
                    re = conv(re, dE, sv);
                    re = __builtin_fma(-k.gy, d1_prod(dp, vt), re);
                    re = __builtin_fma(k.ky, D2T(tt, T), re);
                    vbuf[b][H_PY][pt] = k.gy * D1T(dp);
                }
                if constexpr (DIAG) {
                    if (active) dr[1] += ke;
                }
            }
            // terms between plane zp and planes zp - 1, zp - 2
            {
                const double w1 = qz[SM1][Z_W], w2 = qz[SM2][Z_W];
                const double s1 = k.z4 * (w + w1), s2 = k.zh * (w + w2);
                const double dE1 = E - qz[SM1][Z_E], dE2 = E - qz[SM2][Z_E];
                const double p1 = k.gz8 * (dE1 - (ke - qz[SM1][Z_K])), p2 = k.gz * (dE2 - (ke - qz[SM2][Z_K]));
                const double e1 = dE1 * s1, e2 = dE2 * s2;
                const double h1 = k.kz16 * (T - qz[SM1][Z_T]), h2 = k.kz * (T - qz[SM2][Z_T]);
                const double a1 = __builtin_fma(p1, w1, e1) + h1, a2 = __builtin_fma(p2, w2, e2) + h2;
                const double b1 = __builtin_fma(p1, w, e1) - h1, b2 = __builtin_fma(p2, w, e2) - h2;
                ra[S0][R_EN] = re - (a1 - a2);
                ra[SM1][R_EN] -= b1;
                ra[SM2][R_EN] += b2;
                ra[S0][R_PZ] = p1 - p2;
                ra[SM1][R_PZ] += p1;
                ra[SM2][R_PZ] -= p2;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    KEEP(ra[S0][q]);
                    KEEP(ra[SM1][q]);
                    KEEP(ra[SM2][q]);
                }
                vbuf[b][H_PZ][pt] = ra[SM2][R_PZ];
                qz[S0][Z_E] = E;
                if constexpr (DIAG) qz[S0][Z_R] = LV(L_R, 0, 0);
                qz[S0][Z_K] = ke;
                qz[S0][Z_W] = w;
                qz[S0][Z_T] = T;
            }

            // stage plane zp + 1 into the other buffer (last read in the
            // previous step, before its barrier)
            stage_plane(b ^ 1);

            // finish plane zp - 3: group C's part, RK update, output
            if (do_fin) {
                const int64_t pidx = (int64_t)zf * c.nxy + col;
                const double E3 = qz[SM3][Z_E];
                const double H = __builtin_fma(c.gm1, E3 - qz[SM3][Z_K], E3);   // E + p
                const double R = __builtin_fma(-H, vbuf[b ^ 1][H_DIV][pt],
                                               ra[SM3][R_EN] + vbuf[b ^ 1][H_EN][pt]);
                if (active) {
                    if constexpr (MODE == 0) {
                        s.rout[4 * N + pidx] = R;
                    } else {
                        if constexpr (DIAG) {
                            dr[0] += acc;
                            const double ox = vbuf[b ^ 1][H_OX][pt], oy = vbuf[b ^ 1][H_OY][pt];
                            dr[2] += (0.5 * qz[SM3][Z_R]) * (ox * ox + oy * oy);
                        }
                        __builtin_nontemporal_store(acc + s.a_dt * R, (double *)s.qout + 4 * N + pidx);
                        if constexpr (MODE < 3)
                            __builtin_nontemporal_store(acc + s.b_dt * R, s.acc_out + 4 * N + pidx);
                    }
                }
            }
            if constexpr (DIAG) {
                // omega_z is complete in its plane
                if (active && zp - 1 >= z0 && zp - 1 < z1) {
                    const double oz = vbuf[b ^ 1][H_OZ][pt];
                    dr[2] += (0.5 * qz[SM1][Z_R]) * (oz * oz);
                }
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
        // the fields carried with the flow: density and momenta (the first four)
        enum { Z_W = 4, NZ };
        double qz[5][NZ];      // rho and rho u_i of planes zp .. zp - 3, w of zp .. zp - 2
        double ra[5][4];       // pending mass and momentum residuals
        double acc[4] = {0.0, 0.0, 0.0, 0.0}, accn[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 5; ++q) {
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = 0.0;
#pragma unroll
            for (int f = 0; f < 4; ++f) ra[q][f] = 0.0;
        }

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 3;
            const bool do_fin = (zf >= z0 && zf < z1);
            const bool do_plane = (zp >= z0 && zp < z1);
            if constexpr (MODE >= 1) {
                const int64_t pn = acc_point(zf + 1);
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    acc[f] = accn[f];
                    accn[f] = __builtin_nontemporal_load(accsrc + f * N + pn);
                }
            }
            // Residuals of plane zp - 3: pressure gradient along z from A, div u
            // and the viscous vector from C.  Before the taps of this plane are
            // read, so that its terms do not occupy registers beside them; the
            // update is left to the step's end, where the accumulator has had
            // two steps to arrive.
            double R[4] = {0.0, 0.0, 0.0, 0.0};
            if (do_fin) {
                const double div = vbuf[b ^ 1][H_DIV][pt];
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    R[f] = __builtin_fma(-qz[SM3][f], div, ra[SM3][f]);
                    if (f == 3) R[f] -= vbuf[b ^ 1][H_PZ][pt];
                    if (f > 0) R[f] = __builtin_fma(inv_re, vbuf[b ^ 1][H_VX + f - 1][pt], R[f]);
                    KEEP(R[f]);
                }
            }
            const double m[4] = {LV(L_R, 0, 0), LV(L_M0, 0, 0), LV(L_M1, 0, 0), LV(L_M2, 0, 0)};
            const double w = LV(L_W, 0, 0);
            double rr[4] = {0.0, 0.0, 0.0, 0.0};
            if (do_plane) {
                const double u = LV(L_U, 0, 0), v = LV(L_V, 0, 0);
                {
                    TAPS_X(ut, L_U);
                    TAPS_X(rt, L_R);
                    TAPS_X(m0t, L_M0);
                    TAPS_X(m1t, L_M1);
                    TAPS_X(m2t, L_M2);
                    HALF_SUMS(su, u, ut, k.x4, k.xh);
                    rr[0] = conv(0.0, m[0], rt, su);
                    rr[1] = conv(0.0, m[1], m0t, su);
                    rr[2] = conv(0.0, m[2], m1t, su);
                    rr[3] = conv(0.0, m[3], m2t, su);
                }
                {
                    TAPS_Y(vt, L_V);
                    TAPS_Y(rt, L_R);
                    TAPS_Y(m0t, L_M0);
                    TAPS_Y(m1t, L_M1);
                    TAPS_Y(m2t, L_M2);
                    HALF_SUMS(sv, v, vt, k.y4, k.yh);
                    rr[0] = conv(rr[0], m[0], rt, sv);
                    rr[1] = conv(rr[1], m[1], m0t, sv);
                    rr[2] = conv(rr[2], m[2], m1t, sv);
                    rr[3] = conv(rr[3], m[3], m2t, sv);
                }
            }
            // the in-plane pressure gradient of plane zp - 1, from A's last
            // step (outside the chunk an undefined value, in a residual that
            // is never output)
            ra[SM1][1] -= vbuf[b ^ 1][H_PX][pt];
            ra[SM1][2] -= vbuf[b ^ 1][H_PY][pt];
            // terms between plane zp and planes zp - 1, zp - 2
            {
                const double s1 = k.z4 * (w + qz[SM1][Z_W]), s2 = k.zh * (w + qz[SM2][Z_W]);
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    const double f1 = (m[f] - qz[SM1][f]) * s1, f2 = (m[f] - qz[SM2][f]) * s2;
                    ra[S0][f] = rr[f] - (f1 - f2);
                    ra[SM1][f] -= f1;
                    ra[SM2][f] += f2;
                    KEEP(ra[S0][f]);
                    KEEP(ra[SM1][f]);
                    KEEP(ra[SM2][f]);
                    qz[S0][f] = m[f];
                }
                qz[S0][Z_W] = w;
            }
            // RK update and output of plane zp - 3
            if (do_fin && active) {
                const int64_t pidx = (int64_t)zf * c.nxy + col;
                if constexpr (MODE == 0) {
#pragma unroll
                    for (int f = 0; f < 4; ++f) s.rout[f * N + pidx] = R[f];
                } else {
                    if constexpr (DIAG) {
#pragma unroll
                        for (int f = 0; f < 4; ++f) dr[f] += acc[f];
                    }
                    double *qo = (double *)s.qout;
#pragma unroll
                    for (int f = 0; f < 4; ++f) {
                        __builtin_nontemporal_store(acc[f] + s.a_dt * R[f], qo + f * N + pidx);
                        if constexpr (MODE < 3)
                            __builtin_nontemporal_store(acc[f] + s.b_dt * R[f], s.acc_out + f * N + pidx);
                    }
                }
            }
            lds_barrier();
        };

        lds_barrier();   // group A's prologue
        MARCH(step)
    } else if constexpr (GRAD) {
        // ---------------------------------------- group C, stored gradients
        // Reads 72 B per point more than the fused form (232 B in all in
        // stage 2), which then bounds the stage: 0.90 ms at 256^3 in stage 2,
        // 4.3 TB/s.  A step with the gradient sweep: 6.14 -> 3.48 ms against
        // one thread per point with thirteen divisions and every tap through
        // the caches.
        enum { Z_U, Z_V, Z_W, NZ };
        enum { XX, XY, XZ, YX, YY, YZ, ZX, ZY, ZZ, NG };   // du_i / dx_j
        double qz[5][NZ];      // ring: u, v, w of the own column
        double qs[5];          // ring: D_x u + D_y v
        double rv[5][3];       // in-plane viscous vector of planes zp .. zp - 2
        double rp[5], rd[5];   // dissipation and div u, same planes and zp + 1
        double rx[5];          // mixed x-derivative of plane zp + 1
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            qs[q] = rp[q] = rd[q] = rx[q] = 0.0;
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = rv[q][f] = 0.0;
        }
        // Every lane reads gradients, at its column wrapped into the grid:
        // a lane beyond the grid's edge holds its neighbours' x-taps.
        // Column of the row's end lanes' halo (others: their own), and the
        // halo-row point that threads below 4 BX put into sbuf.
        const int wx = gx % c.nx, wy = gy % c.ny;
        const int hx = (tx < 2) ? -2 : (tx >= BX - 2 ? 2 : 0);
        int hxx = (gx + hx) % c.nx;
        if (hxx < 0) hxx += c.nx;
        const int row = pt / BX, hy = row < 2 ? row : BY + row;
        int hyy = (y0 + hy - 2) % c.ny;
        if (hyy < 0) hyy += c.ny;
        const bool halo_row = pt < 4 * BX;
        const int gown = wy * c.nx + wx, ghx = wy * c.nx + hxx, ghy = halo_row ? hyy * c.nx + wx : gown;
        double gn[NG], hn[2], yn[2];   // plane zp + 1: own column; D_y v, D_z w of the x-halo
                                       // column; D_x u, D_z w of the halo-row point
        auto load_grad = [&](int zp) {
            int zw = zp % c.nz;
            if (zw < 0) zw += c.nz;
            const double *G = s.grad + (int64_t)zw * c.nxy;
#pragma unroll
            for (int q = 0; q < NG; ++q) gn[q] = G[q * N + gown];
            hn[0] = G[YY * N + ghx];
            hn[1] = G[ZZ * N + ghx];
            yn[0] = G[XX * N + ghy];
            yn[1] = G[ZZ * N + ghy];
        };
        // Everything the gradients of one plane give at their own point, into
        // ring slot S, and the field of the y-stencil into sbuf: four values
        // wait for the plane's step instead of eleven.
        auto take_grad = [&](auto sc, int b) {
            constexpr int S = decltype(sc)::value;
            const double g_xx = gn[XX], g_yy = gn[YY], g_zz = gn[ZZ];
            sbuf[b][ty + 2][tx] = g_xx + g_zz;
            if (halo_row) sbuf[b][hy][tx] = yn[0] + yn[1];
            double div = g_xx + g_yy + g_zz, sxy = g_xx + g_yy;
            double phi = 2.0 * (g_xx * g_xx + g_yy * g_yy + g_zz * g_zz) + gn[XY] * gn[XY] + gn[YX] * gn[YX]
                         + gn[XZ] * gn[XZ] + gn[ZX] * gn[ZX] + gn[YZ] * gn[YZ] + gn[ZY] * gn[ZY]
                         + 2.0 * (gn[XY] * gn[YX] + gn[XZ] * gn[ZX] + gn[YZ] * gn[ZY]) - (2.0 / 3.0) * div * div;
            // the x-stencil of D_y v + D_z w across the row's lanes
            double mix = k.mx * d1u_x_lanes<BX>(g_yy + g_zz, hn[0] + hn[1], tx);
            KEEP(div);
            KEEP(sxy);
            KEEP(phi);
            KEEP(mix);
            rd[S] = div;
            qs[S] = sxy;
            rp[S] = phi;
            rx[S] = mix;
        };

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 2;
            const bool do_fin = (zf >= z0 && zf < z1);
            load_grad(zp + 1);
            double r0, r1, r2;
            {
                const double u = LV(L_U, 0, 0);
                TAPS_X(ux, L_U);
                TAPS_Y(uy, L_U);
                const double sy[4] = {sbuf[b][ty][tx], sbuf[b][ty + 1][tx], sbuf[b][ty + 3][tx], sbuf[b][ty + 4][tx]};
                r0 = k.vx * D2T(ux, u) + c2y * D2T(uy, u) + rx[S0];
                r1 = k.my * D1T(sy);
                qz[S0][Z_U] = u;
            }
            {
                const double v = LV(L_V, 0, 0);
                TAPS_X(vx, L_V);
                TAPS_Y(vy, L_V);
                r1 += c2x * D2T(vx, v) + k.vy * D2T(vy, v);
                qz[S0][Z_V] = v;
            }
            {
                const double w = LV(L_W, 0, 0);
                TAPS_X(wx4, L_W);
                TAPS_Y(wy4, L_W);
                r2 = c2x * D2T(wx4, w) + c2y * D2T(wy4, w);
                qz[S0][Z_W] = w;
            }
            KEEP(r0);
            KEEP(r1);
            KEEP(r2);
            rv[S0][0] = r0;
            rv[S0][1] = r1;
            rv[S0][2] = r2;
            // plane zf = zp - 2: gathered z terms, hand-over to A and B
            if (do_fin) {
                const double u = qz[SM2][Z_U], v = qz[SM2][Z_V], w = qz[SM2][Z_W];
                const double Vx = rv[SM2][0] + c2z * DZ2(Z_U);
                const double Vy = rv[SM2][1] + c2z * DZ2(Z_V);
                const double Vz = rv[SM2][2] + (k.vz * DZ2(Z_W) + k.mz * d1(qs[SM4], qs[SM3], qs[SM1], qs[S0]));
                vbuf[b][H_VX][pt] = Vx;
                vbuf[b][H_VY][pt] = Vy;
                vbuf[b][H_VZ][pt] = Vz;
                vbuf[b][H_EN][pt] = inv_re * (u * Vx + v * Vy + w * Vz + rp[SM2]);
                vbuf[b][H_DIV][pt] = rd[SM2];
            }
            take_grad(TIC<SM4>{}, b ^ 1);   // plane zp + 1's slot
            lds_barrier();
        };

        load_grad(z0 - 2);
        take_grad(TIC<0>{}, 0);
        lds_barrier();   // group A's prologue
        MARCH(step)
    } else {
        // ------------------------------------------------------------ group C
        enum { Z_U, Z_V, Z_W, NZ };
        double qz[5][NZ];               // ring: u, v, w of the own column
        double qa[5], qb[5], qc[5];     // ring: D_x u + D_y v, D_x w, D_y w
        double rv[5][3];                // in-plane viscous vector of planes zp .. zp - 2
        double rp[5];                   // in-plane part of the dissipation, same planes
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            qa[q] = qb[q] = qc[q] = rp[q] = 0.0;
#pragma unroll
            for (int f = 0; f < NZ; ++f) qz[q][f] = rv[q][f] = 0.0;
        }

        auto step = [&](auto phc, int zp) {
            PHASES;
            const int b = (zp - z0) & 1;
            const int zf = zp - 2;
            const bool do_fin = (zf >= z0 && zf < z1);
            // The reads of a field are kept ahead of the arithmetic of the
            // field before it, and its arithmetic behind them: a few waits
            // for LDS, and no more taps in registers than two fields need.
            const int hx = (tx < 2) ? -2 : (tx >= BX - 2 ? 2 : 0);
#define LVH(f, dy) lds[b][f][own + (dy) * HX + hx]
            double phi, r0, r1, r2;
            {
                const double u = LV(L_U, 0, 0);
                TAPS_Y(uy, L_U);
                TAPS_X(ux, L_U);
                const double hu4[4] = {LVH(L_U, -2), LVH(L_U, -1), LVH(L_U, 1), LVH(L_U, 2)};
                SB();
                const double v = LV(L_V, 0, 0);
                TAPS_Y(vy, L_V);
                TAPS_X(vx, L_V);
                const double hv4[4] = {LVH(L_V, -2), LVH(L_V, -1), LVH(L_V, 1), LVH(L_V, 2)};
                SB();
                // mixed derivatives d_x d_y u and d_x d_y v: the x-stencil
                // applied across the row's lanes to the y-derivatives they
                // already hold; a row's two end lanes on each side take the
                // y-derivative at their halo column (x - 2 at the start of
                // the row, x + 2 at its end).  The other lanes read their own
                // column, which keeps the wave's addresses on distinct banks.
                const double dyu = D1T(uy);
                const double Gxx = c1x * D1T(ux), Gxy = c1y * dyu;
                r0 = k.vx * D2T(ux, u) + c2y * D2T(uy, u);
                r1 = k.mxy * d1u_x_lanes<BX>(dyu, D1T(hu4), tx);
                qz[S0][Z_U] = u;
                SB();
                const double w = LV(L_W, 0, 0);
                TAPS_Y(wy, L_W);
                TAPS_X(wx, L_W);
                SB();
                const double dyv = D1T(vy);
                const double Gyx = c1x * D1T(vx), Gyy = c1y * dyv;
                r1 += c2x * D2T(vx, v) + k.vy * D2T(vy, v);
                r0 += k.mxy * d1u_x_lanes<BX>(dyv, D1T(hv4), tx);
                qz[S0][Z_V] = v;
                qa[S0] = Gxx + Gyy;
                // tau_ij du_i/dx_j restricted to terms without a z derivative
                phi = 2.0 * (Gxx * Gxx + Gyy * Gyy) + Gxy * Gxy + Gyx * Gyx + 2.0 * Gxy * Gyx;
                if constexpr (DIAG) vbuf[b][H_OZ][pt] = Gyx - Gxy;
                SB();
                const double Gzx = c1x * D1T(wx), Gzy = c1y * D1T(wy);
                r2 = c2x * D2T(wx, w) + c2y * D2T(wy, w);
                phi += Gzx * Gzx + Gzy * Gzy;
                qz[S0][Z_W] = w;
                qb[S0] = Gzx;
                qc[S0] = Gzy;
            }
#undef LVH
            KEEP(r0);
            KEEP(r1);
            KEEP(r2);
            KEEP(phi);
            KEEP(qa[S0]);
            KEEP(qb[S0]);
            KEEP(qc[S0]);
            rv[S0][0] = r0;
            rv[S0][1] = r1;
            rv[S0][2] = r2;
            rp[S0] = phi;
            // plane zf = zp - 2: gathered z terms, hand-over to A and B
            if (do_fin) {
                const double u = qz[SM2][Z_U], v = qz[SM2][Z_V], w = qz[SM2][Z_W];
                const double a = qa[SM2], bb = qb[SM2], cc = qc[SM2];
                const double Gxz = c1z * DZ1(Z_U), Gyz = c1z * DZ1(Z_V), Gzz = c1z * DZ1(Z_W);
                const double Vx = rv[SM2][0] + (c2z * DZ2(Z_U) + k.mz * d1(qb[SM4], qb[SM3], qb[SM1], qb[S0]));
                const double Vy = rv[SM2][1] + (c2z * DZ2(Z_V) + k.mz * d1(qc[SM4], qc[SM3], qc[SM1], qc[S0]));
                const double Vz = rv[SM2][2] + (k.vz * DZ2(Z_W) + k.mz * d1(qa[SM4], qa[SM3], qa[SM1], qa[S0]));
                const double div = a + Gzz;
                const double phi = Gxz * Gxz + Gyz * Gyz + 2.0 * Gzz * Gzz
                                   + 2.0 * (Gxz * bb + Gyz * cc) - (2.0 / 3.0) * div * div;
                vbuf[b][H_VX][pt] = Vx;
                vbuf[b][H_VY][pt] = Vy;
                vbuf[b][H_VZ][pt] = Vz;
                vbuf[b][H_EN][pt] = inv_re * (u * Vx + v * Vy + w * Vz + (rp[SM2] + phi));
                vbuf[b][H_DIV][pt] = div;
                if constexpr (DIAG) {
                    vbuf[b][H_OX][pt] = cc - Gyz;
                    vbuf[b][H_OY][pt] = Gxz - bb;
                }
            }
            lds_barrier();
        };

        lds_barrier();   // group A's prologue
        MARCH(step)
    }
#undef MARCH
#undef PHASES
#undef DZ1
#undef DZ2
#undef HALF_SUMS
#undef SB
#undef KEEP
#undef D1T
#undef D2T
#undef TAPS_X
#undef TAPS_Y
#undef LV

    if constexpr (DIAG) {
        // block reduction of the diagnostic partial sums, fixed order: each
        // thread takes the column sums of its own group's slots (the other
        // groups' slots count zero for it), then waves, then the block
        const int tid = threadIdx.x;
        __syncthreads();
        double dsum[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if (grp == 0) {
            dsum[4] = dr[0];
            dsum[5] = dr[1];
            dsum[6] = dr[2];
        } else if (grp == 1) {
#pragma unroll
            for (int f = 0; f < 4; ++f) dsum[f] = dr[f];
        }
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            const double vsum = wave_sum(dsum[k]);
            if ((tid & 63) == 63) red[tid >> 6][k] = vsum;
        }
        __syncthreads();
        if (tid < 8) {
            const int64_t blin = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
            double t = 0.0;
            for (int wv = 0; wv < NW && tid < 7; ++wv) t += red[wv][tid];
            s.diag_partial[blin * kDiag + tid] = t;
        }
    }
}

namespace {

template <int BX, int BY, bool PAIR, bool GRAD>
hipError_t launch_trio_p(const Consts &c, const StageArgs &s, hipStream_t st)
{
    const dim3 block(3 * BX * BY, 1, 1);
    const dim3 grid((c.nx + BX - 1) / BX, (c.ny + BY - 1) / BY,
                    (c.nz + s.zchunk - 1) / s.zchunk + (s.fin_out != nullptr));
    const Coef64 k = make_coef64(c);
    switch (s.mode) {
    case 0: hipLaunchKernelGGL((trio_stage_kernel<BX, BY, 0, false, PAIR, GRAD>), grid, block, 0, st, c, k, s); break;
    case 1:
        if constexpr (!GRAD) {
            if (s.diag_partial != nullptr) {
                hipLaunchKernelGGL((trio_stage_kernel<BX, BY, 1, true, PAIR, GRAD>), grid, block, 0, st, c, k, s);
                break;
            }
        }
        hipLaunchKernelGGL((trio_stage_kernel<BX, BY, 1, false, PAIR, GRAD>), grid, block, 0, st, c, k, s);
        break;
    case 2: hipLaunchKernelGGL((trio_stage_kernel<BX, BY, 2, false, PAIR, GRAD>), grid, block, 0, st, c, k, s); break;
    case 3: hipLaunchKernelGGL((trio_stage_kernel<BX, BY, 3, false, PAIR, GRAD>), grid, block, 0, st, c, k, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// The halo plane is loaded in x-neighbour pairs when nx is even: pairs start
// at even x, so they never straddle the periodic wrap.
template <int BX, int BY, bool GRAD = false>
hipError_t launch_trio(const Consts &c, const StageArgs &s, hipStream_t st)
{
    return c.nx % 2 == 0 ? launch_trio_p<BX, BY, true, GRAD>(c, s, st) : launch_trio_p<BX, BY, false, GRAD>(c, s, st);
}

template <int BX, int BY>
int resident_trio()
{
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per, reinterpret_cast<const void *>(&trio_stage_kernel<BX, BY, 2, false, true, false>), 3 * BX * BY, 0) != hipSuccess)
        return 0;
    return cus * (per > 0 ? per : 1);
}

}  // namespace

int trio_resident_blocks(int tile)
{
    switch (tile) {
    case TILE_16x8_3G: return resident_trio<16, 8>();
    case TILE_32x8_3G: return resident_trio<32, 8>();
    case TILE_16x4_3G: return resident_trio<16, 4>();
    default: return 0;
    }
}

hipError_t launch_trio_grad(const Consts &c, const StageArgs &s, hipStream_t st)
{
    return launch_trio<32, 8, true>(c, s, st);
}

hipError_t launch_trio_stage(const Consts &c, const StageArgs &s, int tile, hipStream_t st)
{
    switch (tile) {
    case TILE_16x8_3G: return launch_trio<16, 8>(c, s, st);
    case TILE_32x8_3G: return launch_trio<32, 8>(c, s, st);
    case TILE_16x4_3G: return launch_trio<16, 4>(c, s, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ns
