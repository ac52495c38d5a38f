// ns_brick.hip -- the fused FP64 stage kernel for small grids.
//
// The marching kernels step through at least five planes one after another,
// each with a barrier and, on a small grid that cannot hide it, a wait for
// memory: about 7 us a stage at 16^3 whose data would take 0.1 us.  Here a
// block owns a brick of 8 x 4 x BRZ points and stages it whole, with its halo
// of two, in one round of loads; then three groups of waves evaluate the
// equations of one point per thread (A mass, energy and the pressure gradient,
// B momentum, C viscous terms) with the expressions of ns_trio.hip in the same
// order, so that the result is the same bit for bit.
// Three barriers in all: after the staging, after the in-plane gradients that
// are differentiated along z, and before A and B take over C's values.
//
// Bound by latency: of 4.7 us a stage at 16^3 (14.2 us an RK3 step, the
// march's best shape 20.9), 1.7 us are an empty launch of a chain; the round
// of loads and its share of the conversions (1.8 us), the gradients (0.3 us)
// and one thread's arithmetic (about 140 double operations, 1.5 us) are the
// rest.  Rows of two fields side by side keep a wave's reads on distinct banks
// (rows of one field: 16^3 14.6 -> 14.2 us a step, 32^3 18.4 -> 17.1).  Two
// planes put one wave on each of three SIMDs (16^3 16.3 -> 14.6 us a step
// against four planes) but load nine points per point of the brick against six,
// so they are taken only while each brick has a compute unit.
// One kernel for all stages and the residual: with the stage known at compile
// time, each stage fetched its code anew (0.1 us).
#include "ns_common.hpp"
#include "ns_fp64.hpp"
#include "ns_kernels.hpp"

namespace ns {

namespace {

constexpr int BRX = 8, BRY = 4;

}  // namespace

template <int BRZ, bool DIAG>
__global__ void __launch_bounds__(3 * BRX * BRY * BRZ) brick_stage_kernel(Consts c, Coef64 k, StageArgs s)
{
#pragma clang fp contract(on)
    constexpr int HX = BRX + 4, HY = BRY + 4, HZ = BRZ + 4, HP = HX * HY, CELLS = HP * HZ;
    constexpr int NT = BRX * BRY * BRZ, NLOAD = (CELLS + 3 * NT - 1) / (3 * NT);
    constexpr int GP = BRX * BRY, GC = GP * HZ;      // own columns with their z halo
    constexpr int NW = 3 * NT / 64;
    static_assert(NT % 64 == 0, "each group must be whole waves");
    static_assert(GC <= 3 * NT, "one gradient point per thread");
    // staged fields: rho, rho u_i, E, u, v, w, kinetic energy, e = T / (gamma (gamma - 1) M^2)
    enum { L_R, L_M0, L_M1, L_M2, L_E, L_U, L_V, L_W, L_K, L_T, NF };
    enum { G_A, G_B, G_C, NG };                      // D_x u + D_y v, D_x w, D_y w
    enum { H_VX, H_VY, H_VZ, H_EN, H_DIV, H_PX, H_PY, H_PZ, NH };
    // Two fields share a row of the array, side by side: with rows of 2 HX cells
    // the rows that a wave reads at once start in different banks.
    constexpr int RS = 2 * HX, PS = HY * RS;
    static_assert(NF % 2 == 0, "fields in pairs");
    __shared__ double lds[NF / 2][HZ * PS];
    __shared__ double grad[NG][GC];
    __shared__ double vbuf[NH][NT];
    __shared__ double red[DIAG ? NW : 1][4];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / (NT / 64);
    const int pt = tid - grp * NT;
    const int tx = pt % BRX, ty = (pt / BRX) % BRY, tz = pt / GP;
    const int skip = DIAG ? 0 : finalize_layer(c, s);
    if (skip < 0) return;
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz, skip);
    const int x0 = tbx * BRX, y0 = tby * BRY, z0 = tbz * BRZ;
    const bool active = x0 + tx < c.nx && y0 + ty < c.ny && z0 + tz < c.nz;
    const int own = (tz + 2) * PS + (ty + 2) * RS + tx + 2;
    const int64_t N = c.N;
    const int64_t pidx = active ? ((int64_t)(z0 + tz) * c.ny + y0 + ty) * c.nx + x0 + tx : 0;
    const double *qin = (const double *)s.qin;
    const double *accsrc = (s.mode >= 2) ? s.acc_in : qin;
    const double c1x = c.c1[0], c1y = c.c1[1], c1z = c.c1[2];
    const double c2x = c.c2[0], c2y = c.c2[1], c2z = c.c2[2];

#define AT(f, at) lds[(f) >> 1][((f) & 1) * HX + (at)]

    // ---- stage the brick with its halo, wrapped to valid memory everywhere: a
    // brick starts inside the grid at a multiple of its extent, so that with
    // five points or more one period each way is enough
    double q[NLOAD][5];
#pragma unroll
    for (int r = 0; r < NLOAD; ++r) {
        const int cell = min(tid + r * 3 * NT, CELLS - 1);
        const int xx = wrap1(x0 + cell % HX - 2, c.nx), yy = wrap1(y0 + (cell / HX) % HY - 2, c.ny);
        const int zz = wrap1(z0 + cell / HP - 2, c.nz);
        const double *src = qin + ((int64_t)zz * c.ny + yy) * c.nx + xx;
#pragma unroll
        for (int f = 0; f < 5; ++f) q[r][f] = src[f * N];
    }
    // accumulator of the own point: group A the mass and energy, B the momenta
    double acc[3] = {0.0, 0.0, 0.0};
    if (s.mode >= 1) {
        if (grp == 0) {
            acc[0] = accsrc[pidx];
            acc[1] = accsrc[4 * N + pidx];
        } else if (grp == 1) {
#pragma unroll
            for (int f = 0; f < 3; ++f) acc[f] = accsrc[(1 + f) * N + pidx];
        }
    }
#pragma unroll
    for (int r = 0; r < NLOAD; ++r) {
        const int cell = tid + r * 3 * NT;
        if (CELLS % (3 * NT) != 0 && cell >= CELLS) continue;
        const int at = (cell / HX) * RS + cell % HX;
        const double rho = q[r][0], m0 = q[r][1], m1 = q[r][2], m2 = q[r][3];
        const double E = q[r][4];
        const double inv = recip_f64(rho);
        const double u = quotient_f64(m0, rho, inv), v = quotient_f64(m1, rho, inv), w = quotient_f64(m2, rho, inv);
        const double ke = 0.5 * (m0 * u + m1 * v + m2 * w);
        AT(L_R, at) = rho;
        AT(L_M0, at) = m0;
        AT(L_M1, at) = m1;
        AT(L_M2, at) = m2;
        AT(L_E, at) = E;
        AT(L_U, at) = u;
        AT(L_V, at) = v;
        AT(L_W, at) = w;
        AT(L_K, at) = ke;
        AT(L_T, at) = (E - ke) * inv;
    }
    lds_barrier();

#define LV(f, dz, dy, dx) AT(f, own + (dz) * PS + (dy) * RS + (dx))
#define TAPS_X(t, f) const double t[4] = {LV(f, 0, 0, -2), LV(f, 0, 0, -1), LV(f, 0, 0, 1), LV(f, 0, 0, 2)}
#define TAPS_Y(t, f) const double t[4] = {LV(f, 0, -2, 0), LV(f, 0, -1, 0), LV(f, 0, 1, 0), LV(f, 0, 2, 0)}
#define TAPS_Z(t, f) const double t[4] = {LV(f, -2, 0, 0), LV(f, -1, 0, 0), LV(f, 1, 0, 0), LV(f, 2, 0, 0)}
#define D1T(t) d1(t[0], t[1], t[2], t[3])
#define D2T(t, t0) d2(t[0], t[1], t0, t[2], t[3])
#define HALF_SUMS(s, u0, t, w4, wh)                                                               \
    const double s[4] = {(wh) * ((u0) + t[0]), (w4) * ((u0) + t[1]), (w4) * ((u0) + t[2]), (wh) * ((u0) + t[3])}

    // ---- in-plane gradients of the own columns with their z halo
    if (tid < GC) {
        const int at = (tid / GP) * PS + ((tid % GP) / BRX + 2) * RS + tid % BRX + 2;
        const double ux = d1(AT(L_U, at - 2), AT(L_U, at - 1), AT(L_U, at + 1), AT(L_U, at + 2));
        const double vy = d1(AT(L_V, at - 2 * RS), AT(L_V, at - RS), AT(L_V, at + RS), AT(L_V, at + 2 * RS));
        const double wx = d1(AT(L_W, at - 2), AT(L_W, at - 1), AT(L_W, at + 1), AT(L_W, at + 2));
        const double wy = d1(AT(L_W, at - 2 * RS), AT(L_W, at - RS), AT(L_W, at + RS), AT(L_W, at + 2 * RS));
        const double gxx = c1x * ux, gyy = c1y * vy;
        grad[G_A][tid] = gxx + gyy;
        grad[G_B][tid] = c1x * wx;
        grad[G_C][tid] = c1y * wy;
    }
    lds_barrier();

    // residuals of the own equations; what div u multiplies in them (group A rho
    // and E + p, B rho u_i); of B the terms with the planes above
    double R[3] = {0.0, 0.0, 0.0}, car[3] = {0.0, 0.0, 0.0}, up[3][2] = {};
    // diagnostics of the point: group A mass, energy and kinetic energy, B the
    // momenta, C enstrophy
    double dsum[4] = {0.0, 0.0, 0.0, 0.0};
    if (grp == 0) {
        // ------------------------------------------------------------ group A
        const double r = LV(L_R, 0, 0, 0), E = LV(L_E, 0, 0, 0), w = LV(L_W, 0, 0, 0), T = LV(L_T, 0, 0, 0);
        const double ke = LV(L_K, 0, 0, 0), u = LV(L_U, 0, 0, 0), v = LV(L_V, 0, 0, 0);
        double rm = 0.0, re = 0.0;
        {
            TAPS_X(ut, L_U);
            TAPS_X(rt, L_R);
            TAPS_X(et, L_E);
            TAPS_X(kt, L_K);
            TAPS_X(tt, L_T);
            HALF_SUMS(su, u, ut, k.x4, k.xh);
            double dE[4], dp[4];
            diffs(E, et, dE);
            pressure_diffs(dE, ke, kt, dp);
            rm = conv(rm, r, rt, su);
            re = conv(re, dE, su);
            re = __builtin_fma(-k.gx, d1_prod(dp, ut), re);
            re = __builtin_fma(k.kx, D2T(tt, T), re);
            vbuf[H_PX][pt] = k.gx * D1T(dp);
        }
        {
            TAPS_Y(vt, L_V);
            TAPS_Y(rt, L_R);
            TAPS_Y(et, L_E);
            TAPS_Y(kt, L_K);
            TAPS_Y(tt, L_T);
            HALF_SUMS(sv, v, vt, k.y4, k.yh);
            double dE[4], dp[4];
            diffs(E, et, dE);
            pressure_diffs(dE, ke, kt, dp);
            rm = conv(rm, r, rt, sv);
            re = conv(re, dE, sv);
            re = __builtin_fma(-k.gy, d1_prod(dp, vt), re);
            re = __builtin_fma(k.ky, D2T(tt, T), re);
            vbuf[H_PY][pt] = k.gy * D1T(dp);
        }
        {
            // terms between the point's plane and the two below and above, added
            // in the march's order
            TAPS_Z(wt, L_W);
            TAPS_Z(rt, L_R);
            TAPS_Z(et, L_E);
            TAPS_Z(kt, L_K);
            TAPS_Z(tt, L_T);
            double mf[4], ef[4], pf[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool below = t < 2, near = t == 1 || t == 2;
                const double st = (near ? k.z4 : k.zh) * (w + wt[t]);
                // from the lower to the upper plane of the pair
                const double dE = below ? E - et[t] : et[t] - E, dK = below ? ke - kt[t] : kt[t] - ke;
                const double h = (near ? k.kz16 : k.kz) * (below ? T - tt[t] : tt[t] - T);
                pf[t] = (near ? k.gz8 : k.gz) * (dE - dK);
                const double e = dE * st;
                mf[t] = (below ? r - rt[t] : rt[t] - r) * st;
                ef[t] = below ? __builtin_fma(pf[t], wt[t], e) + h : __builtin_fma(pf[t], wt[t], e) - h;
            }
            rm = rm - (mf[1] - mf[0]);
            rm -= mf[2];
            rm += mf[3];
            re = re - (ef[1] - ef[0]);
            re -= ef[2];
            re += ef[3];
            double pz = pf[1] - pf[0];
            pz += pf[2];
            pz -= pf[3];
            vbuf[H_PZ][pt] = pz;
        }
        R[0] = rm;
        R[1] = re;
        car[0] = r;
        car[1] = __builtin_fma(c.gm1, E - ke, E);
        if constexpr (DIAG) dsum[2] = ke;
    } else if (grp == 1) {
        // ------------------------------------------------------------ group B
        const double m[3] = {LV(L_M0, 0, 0, 0), LV(L_M1, 0, 0, 0), LV(L_M2, 0, 0, 0)};
        const double u = LV(L_U, 0, 0, 0), v = LV(L_V, 0, 0, 0), w = LV(L_W, 0, 0, 0);
        double rr[3];
        {
            TAPS_X(ut, L_U);
            TAPS_X(m0t, L_M0);
            TAPS_X(m1t, L_M1);
            TAPS_X(m2t, L_M2);
            HALF_SUMS(su, u, ut, k.x4, k.xh);
            rr[0] = conv(0.0, m[0], m0t, su);
            rr[1] = conv(0.0, m[1], m1t, su);
            rr[2] = conv(0.0, m[2], m2t, su);
        }
        {
            TAPS_Y(vt, L_V);
            TAPS_Y(m0t, L_M0);
            TAPS_Y(m1t, L_M1);
            TAPS_Y(m2t, L_M2);
            HALF_SUMS(sv, v, vt, k.y4, k.yh);
            rr[0] = conv(rr[0], m[0], m0t, sv);
            rr[1] = conv(rr[1], m[1], m1t, sv);
            rr[2] = conv(rr[2], m[2], m2t, sv);
        }
        {
            TAPS_Z(wt, L_W);
            double sz[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) sz[t] = (t == 1 || t == 2 ? k.z4 : k.zh) * (w + wt[t]);
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                TAPS_Z(mt, L_M0 + f);
                double fl[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) fl[t] = (t < 2 ? m[f] - mt[t] : mt[t] - m[f]) * sz[t];
                R[f] = rr[f] - (fl[1] - fl[0]);
                car[f] = m[f];
                up[f][0] = fl[2];
                up[f][1] = fl[3];
            }
        }
    } else {
        // ------------------------------------------------------------ group C
        const int gat = (tz + 2) * GP + ty * BRX + tx;
        const int hx = (tx < 2) ? -2 : (tx >= BRX - 2 ? 2 : 0);
        double phi, r0, r1, r2, a, bb, cc, oz;
        const double u = LV(L_U, 0, 0, 0), v = LV(L_V, 0, 0, 0), w = LV(L_W, 0, 0, 0);
        {
            TAPS_X(ux, L_U);
            TAPS_Y(uy, L_U);
            TAPS_X(vx, L_V);
            TAPS_Y(vy, L_V);
            TAPS_X(wx, L_W);
            TAPS_Y(wy, L_W);
            const double hu4[4] = {LV(L_U, 0, -2, hx), LV(L_U, 0, -1, hx), LV(L_U, 0, 1, hx), LV(L_U, 0, 2, hx)};
            const double hv4[4] = {LV(L_V, 0, -2, hx), LV(L_V, 0, -1, hx), LV(L_V, 0, 1, hx), LV(L_V, 0, 2, hx)};
            const double dyu = D1T(uy), dyv = D1T(vy);
            const double Gxx = c1x * D1T(ux), Gxy = c1y * dyu;
            const double Gyx = c1x * D1T(vx), Gyy = c1y * dyv;
            r0 = k.vx * D2T(ux, u) + c2y * D2T(uy, u);
            r1 = k.mxy * d1u_x_lanes<BRX>(dyu, D1T(hu4), tx);
            r1 += c2x * D2T(vx, v) + k.vy * D2T(vy, v);
            r0 += k.mxy * d1u_x_lanes<BRX>(dyv, D1T(hv4), tx);
            phi = 2.0 * (Gxx * Gxx + Gyy * Gyy) + Gxy * Gxy + Gyx * Gyx + 2.0 * Gxy * Gyx;
            const double Gzx = c1x * D1T(wx), Gzy = c1y * D1T(wy);
            r2 = c2x * D2T(wx, w) + c2y * D2T(wy, w);
            phi += Gzx * Gzx + Gzy * Gzy;
            a = Gxx + Gyy;
            bb = Gzx;
            cc = Gzy;
            oz = Gyx - Gxy;
        }
        TAPS_Z(uz, L_U);
        TAPS_Z(vz, L_V);
        TAPS_Z(wz, L_W);
#define GZ(f) d1(grad[f][gat - 2 * GP], grad[f][gat - GP], grad[f][gat + GP], grad[f][gat + 2 * GP])
        const double Gxz = c1z * D1T(uz), Gyz = c1z * D1T(vz), Gzz = c1z * D1T(wz);
        const double Vx = r0 + (c2z * D2T(uz, u) + k.mz * GZ(G_B));
        const double Vy = r1 + (c2z * D2T(vz, v) + k.mz * GZ(G_C));
        const double Vz = r2 + (k.vz * D2T(wz, w) + k.mz * GZ(G_A));
#undef GZ
        const double div = a + Gzz;
        const double phz = Gxz * Gxz + Gyz * Gyz + 2.0 * Gzz * Gzz
                           + 2.0 * (Gxz * bb + Gyz * cc) - (2.0 / 3.0) * div * div;
        vbuf[H_VX][pt] = Vx;
        vbuf[H_VY][pt] = Vy;
        vbuf[H_VZ][pt] = Vz;
        vbuf[H_EN][pt] = c.inv_re * (u * Vx + v * Vy + w * Vz + (phi + phz));
        vbuf[H_DIV][pt] = div;
        if constexpr (DIAG) {
            const double ox = cc - Gyz, oy = Gxz - bb;
            dsum[0] = 0.5 * LV(L_R, 0, 0, 0) * (ox * ox + oy * oy + oz * oz);
        }
    }
    lds_barrier();

    // ---- C's part of the equations, RK update, output
    if (grp < 2 && active) {
        const double div = vbuf[H_DIV][pt];
        if (grp == 0) {
            R[0] = __builtin_fma(-car[0], div, R[0]);
            R[1] = __builtin_fma(-car[1], div, R[1] + vbuf[H_EN][pt]);
        } else {
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                if (f < 2) R[f] -= vbuf[H_PX + f][pt];
                R[f] -= up[f][0];
                R[f] += up[f][1];
                R[f] = __builtin_fma(-car[f], div, R[f]);
                if (f == 2) R[f] -= vbuf[H_PZ][pt];
                R[f] = __builtin_fma(c.inv_re, vbuf[H_VX + f][pt], R[f]);
            }
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            if (grp == 0 && f == 2) continue;
            const int field = grp == 0 ? 4 * f : 1 + f;
            const int64_t at = field * N + pidx;
            if (s.mode == 0) {
                s.rout[at] = R[f];
            } else {
                ((double *)s.qout)[at] = acc[f] + s.a_dt * R[f];
                if (s.mode < 3) s.acc_out[at] = acc[f] + s.b_dt * R[f];
            }
        }
        if constexpr (DIAG) {
            dsum[0] = acc[0];
            dsum[1] = acc[1];
            if (grp == 1) dsum[2] = acc[2];
        }
    }
#undef AT
#undef LV
#undef TAPS_X
#undef TAPS_Y
#undef TAPS_Z
#undef D1T
#undef D2T
#undef HALF_SUMS

    if constexpr (DIAG) {
        // block sum of the diagnostics in a fixed order
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const double vsum = wave_sum(active ? dsum[d] : 0.0);
            if ((tid & 63) == 63) red[wave][d] = vsum;
        }
        lds_barrier();
        if (tid < kDiag) {
            // a record's slots by group: B 1 to 3, A 0, 4 and 5, C 6 and 7 (zero)
            const int g = tid >= 1 && tid < 4 ? 1 : tid < 6 ? 0 : 2;
            const int d = g == 1 ? tid - 1 : g == 0 ? (tid == 0 ? 0 : tid - 3) : tid - 6;
            const int64_t blin = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
            double t = 0.0;
#pragma unroll
            for (int wv = 0; wv < NW / 3; ++wv) t += red[g * (NW / 3) + wv][d];
            s.diag_partial[blin * kDiag + tid] = t;
        }
    }
}

int64_t brick_num_blocks(const Consts &c, int bz)
{
    return (int64_t)((c.nx + BRX - 1) / BRX) * ((c.ny + BRY - 1) / BRY) * ((c.nz + bz - 1) / bz);
}

template <int BRZ>
static hipError_t launch_brick_z(const Consts &c, const StageArgs &s, hipStream_t st)
{
    const dim3 block(3 * BRX * BRY * BRZ);
    const dim3 grid((c.nx + BRX - 1) / BRX, (c.ny + BRY - 1) / BRY,
                    (c.nz + BRZ - 1) / BRZ + (s.fin_out != nullptr));
    const Coef64 k = make_coef64(c);
    if (s.diag_partial != nullptr)
        hipLaunchKernelGGL((brick_stage_kernel<BRZ, true>), grid, block, 0, st, c, k, s);
    else
        hipLaunchKernelGGL((brick_stage_kernel<BRZ, false>), grid, block, 0, st, c, k, s);
    return hipGetLastError();
}

hipError_t launch_brick_stage(const Consts &c, const StageArgs &s, int bz, hipStream_t st)
{
    return bz == 2 ? launch_brick_z<2>(c, s, st) : launch_brick_z<4>(c, s, st);
}

}  // namespace ns
