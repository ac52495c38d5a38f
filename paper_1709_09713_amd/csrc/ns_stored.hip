// ns_stored.hip -- the stored-derivative (baseline, BL) algorithm class.
//
// As in the baseline-algorithm section every derivative of the governing
// equations is computed first and stored in its own global work array, and a
// pointwise pass assembles the residual from those arrays and applies the
// Runge-Kutta update.  Derivative census: 42 first derivatives, 12 second
// derivatives and the 6 mixed derivatives d/dx_i (d u_k/dx_k), i != k, first
// derivatives of the velocity gradients (in either order of the two
// stencils): 60 arrays.
#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

// Derivative arrays (units of N doubles).  The work space has room for 20 more,
// the primitives and products of the former sweeps, which are formed on chip
// now: ns_workspace_bytes keeps the size that callers were told.
enum { W_TOTAL = 80 };
enum {
    D_RHO = 0,    // d rho / dx_j                      (3)
    D_M = 3,      // d m_i / dx_j,     3 i + j         (9)
    D_U = 12,     // d u_i / dx_j,     3 i + j         (9)
    D_MU = 21,    // d (m_i u_j) / dx_j, 3 i + j       (9)
    D_E = 30,     // d rhoE / dx_j                     (3)
    D_EU = 33,    // d (rhoE u_j) / dx_j               (3)
    D_PU = 36,    // d (p u_j) / dx_j                  (3)
    D_P = 39,     // d p / dx_i                        (3)
    D2_U = 42,    // d2 u_i / dx_j^2,  3 i + j         (9)
    D2_T = 51,    // d2 T / dx_j^2                     (3)
    D_MIX = 54,   // d/dx_i (d u_k / dx_k), i != k, (i, k) = (0,1) (0,2) (1,0) (1,2) (2,0) (2,1)
    D_COUNT = 60
};

size_t stored_workspace_doubles(const Consts &c) { return (size_t)W_TOTAL * (size_t)c.N; }

namespace {

constexpr int BL_BX = 32, BL_BY = 8, BL_NT = BL_BX * BL_BY;

}  // namespace

// All 60 derivative arrays in one pass.  A block owns a 32 x 8 column tile
// and marches along z: each plane with its halo of two goes through LDS as
// primitives, the x and y derivatives of the plane and the two in-plane mixed
// ones are stored in its step, the z derivatives of plane zp - 2 from a ring
// of five planes of the own column.
//
// Bound by memory: 40 B read and 480 B written per point (one sweep per
// derivative, primitives and products through global arrays: 1.4 KB), so the
// rings are shifted by moves and two waves per SIMD are enough.  256^3: 1.84
// ms, 4.74 TB/s; with the pointwise pass (2.07 ms, 5.2 TB/s) an RK3 step
// takes 11.8 ms where 62 sweeps per stage took 22.0, and 0.05 ms instead of
// 0.6 at 16^3, where the launches counted.  Taking the two passes slab by slab
// (32 to 300 MB of derivatives at a time, for the cache behind L2) was 3% to
// 70% slower.
__global__ void __launch_bounds__(BL_NT)
bl_derivatives_kernel(Consts c, const double *__restrict__ Q, double *__restrict__ D, int zchunk)
{
    // Products at the taps are rounded once, alike for every point that uses
    // a tap, so that periodic sums of the flux differences telescope.
#pragma clang fp contract(on)
    constexpr int HX = BL_BX + 4, HY = BL_BY + 4, HP = HX * HY;
    static_assert(HP <= 2 * BL_NT, "one halo point per thread");
    enum { RHO, M0, M1, M2, EN, U, V, W, P, T, NF };
    enum { GXX = NF, GYY, GZX, GZY, NR };       // in-plane gradients differentiated along z
    __shared__ double lds[2][NF][HP];
    const int tid = threadIdx.x, tx = tid % BL_BX, ty = tid / BL_BX;
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz);
    const int x0 = tbx * BL_BX, y0 = tby * BL_BY;
    const int z0 = tbz * zchunk, z1 = min(z0 + zchunk, c.nz);
    const bool active = x0 + tx < c.nx && y0 + ty < c.ny;
    const int64_t N = c.N;
    const int own = (ty + 2) * HX + tx + 2;
    // Own column, wrapped beyond the grid (a partial tile's last columns read
    // their halo there), and this thread's point of the radius-2 ring: two
    // rows above and below, then two columns on each side.
    const int ocol = ((y0 + ty) % c.ny) * c.nx + (x0 + tx) % c.nx;
    const bool halo = tid < HP - BL_NT;
    int hx = 2, hy = 2;
    if (tid < 4 * HX) {
        const int row = tid / HX;
        hx = tid % HX;
        hy = row < 2 ? row : HY - 4 + row;
    } else if (halo) {
        const int q = tid - 4 * HX, cc = q % 4;
        hx = cc < 2 ? cc : HX - 4 + cc;
        hy = 2 + q / 4;
    }
    const int hcell = hy * HX + hx;
    int hxx = (x0 + hx - 2) % c.nx, hyy = (y0 + hy - 2) % c.ny;
    if (hxx < 0) hxx += c.nx;
    if (hyy < 0) hyy += c.ny;
    const int hcol = hyy * c.nx + hxx;

    double po[5], ph[5];        // conserved values of the next plane: own and halo point
    auto load = [&](int zp) {
        int zw = zp % c.nz;
        if (zw < 0) zw += c.nz;
        const double *q = Q + (int64_t)zw * c.nxy;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            po[f] = q[f * N + ocol];
            ph[f] = q[f * N + hcol];
        }
    };
    auto primitives = [&](const double (&q)[5], double (&v)[NF]) {
        const double inv = recip_f64(q[0]);
        v[RHO] = q[0];
        v[M0] = q[1];
        v[M1] = q[2];
        v[M2] = q[3];
        v[EN] = q[4];
        v[U] = quotient_f64(q[1], q[0], inv);
        v[V] = quotient_f64(q[2], q[0], inv);
        v[W] = quotient_f64(q[3], q[0], inv);
        v[P] = c.gm1 * (q[4] - 0.5 * (q[1] * v[U] + q[2] * v[V] + q[3] * v[W]));
        v[T] = quotient_f64(c.gM2 * v[P], q[0], inv);
    };
    double r[5][NR];            // planes zp - 4 .. zp of the own column
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int f = 0; f < NR; ++f) r[k][f] = 0.0;

    load(z0 - 2);
    for (int zp = z0 - 2; zp < z1 + 2; ++zp) {
        const int b = (zp - z0) & 1;
        double v[NF];
        primitives(po, v);
#pragma unroll
        for (int f = 0; f < NF; ++f) lds[b][f][own] = v[f];
        if (halo) {
            double g[NF];
            primitives(ph, g);
#pragma unroll
            for (int f = 0; f < NF; ++f) lds[b][f][hcell] = g[f];
        }
        lds_barrier();
        if (zp + 1 < z1 + 2) load(zp + 1);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int f = 0; f < NR; ++f) r[k][f] = r[k + 1][f];
#pragma unroll
        for (int f = 0; f < NF; ++f) r[4][f] = v[f];

        const double c1x = c.c1[0], c1y = c.c1[1], c1z = c.c1[2];
        const bool out = active && zp >= z0 && zp < z1;
        double *o = D + (int64_t)(out ? zp : z0) * c.nxy + ocol;
#define LV(f, dy, dx) lds[b][f][own + (dy) * HX + (dx)]
#define TX(t, f) const double t[4] = {LV(f, 0, -2), LV(f, 0, -1), LV(f, 0, 1), LV(f, 0, 2)}
#define TY(t, f) const double t[4] = {LV(f, -2, 0), LV(f, -1, 0), LV(f, 1, 0), LV(f, 2, 0)}
#define D1(t) d1u(t[0], t[1], t[2], t[3])
#define D1P(t, g) d1u(t[0] * g[0], t[1] * g[1], t[2] * g[2], t[3] * g[3])
#define D2(t, t0) d2u(t[0], t[1], t0, t[2], t[3])
#define OUT(k, x)                       \
    do {                                \
        const double val = (x);         \
        if (out) o[(k) * N] = val;      \
    } while (0)
        // the gradients that the mixed derivatives differentiate, on every
        // lane and plane
        TX(ux, U);
        TX(vx, V);
        TX(wx, W);
        TY(uy, U);
        TY(vy, V);
        TY(wy, W);
        const double gxx = c1x * D1(ux), gyy = c1y * D1(vy);
        const double gzx = c1x * D1(wx), gzy = c1y * D1(wy);
        r[4][GXX] = gxx;
        r[4][GYY] = gyy;
        r[4][GZX] = gzx;
        r[4][GZY] = gzy;
        if (zp >= z0 && zp < z1) {
            const double dyu = D1(uy), dyv = D1(vy);
            // d_x d_y across the row's lanes (the end lanes take their halo
            // column's y-derivative; the others read their own column)
            const int ho = (tx < 2) ? -2 : (tx >= BL_BX - 2 ? 2 : 0);
            const double hu[4] = {LV(U, -2, ho), LV(U, -1, ho), LV(U, 1, ho), LV(U, 2, ho)};
            const double hv[4] = {LV(V, -2, ho), LV(V, -1, ho), LV(V, 1, ho), LV(V, 2, ho)};
            const double mxv = d1u_x_lanes<BL_BX>(dyv, D1(hv), tx), mxu = d1u_x_lanes<BL_BX>(dyu, D1(hu), tx);
            OUT(D_MIX + 0, c1x * c1y * mxv);
            OUT(D_MIX + 2, c1x * c1y * mxu);
            OUT(D_U + 0, gxx);
            OUT(D_U + 3, c1x * D1(vx));
            OUT(D_U + 6, gzx);
            OUT(D_U + 1, c1y * dyu);
            OUT(D_U + 4, gyy);
            OUT(D_U + 7, gzy);
            OUT(D2_U + 0, c.c2[0] * D2(ux, v[U]));
            OUT(D2_U + 3, c.c2[0] * D2(vx, v[V]));
            OUT(D2_U + 6, c.c2[0] * D2(wx, v[W]));
            OUT(D2_U + 1, c.c2[1] * D2(uy, v[U]));
            OUT(D2_U + 4, c.c2[1] * D2(vy, v[V]));
            OUT(D2_U + 7, c.c2[1] * D2(wy, v[W]));
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                TX(mx, M0 + a);
                TY(my, M0 + a);
                OUT(D_M + 3 * a, c1x * D1(mx));
                OUT(D_M + 3 * a + 1, c1y * D1(my));
                OUT(D_MU + 3 * a, c1x * D1P(mx, ux));
                OUT(D_MU + 3 * a + 1, c1y * D1P(my, vy));
            }
            {
                TX(tx4, RHO);
                TY(ty4, RHO);
                OUT(D_RHO + 0, c1x * D1(tx4));
                OUT(D_RHO + 1, c1y * D1(ty4));
            }
            {
                TX(tx4, EN);
                TY(ty4, EN);
                OUT(D_E + 0, c1x * D1(tx4));
                OUT(D_E + 1, c1y * D1(ty4));
                OUT(D_EU + 0, c1x * D1P(tx4, ux));
                OUT(D_EU + 1, c1y * D1P(ty4, vy));
            }
            {
                TX(tx4, P);
                TY(ty4, P);
                OUT(D_P + 0, c1x * D1(tx4));
                OUT(D_P + 1, c1y * D1(ty4));
                OUT(D_PU + 0, c1x * D1P(tx4, ux));
                OUT(D_PU + 1, c1y * D1P(ty4, vy));
            }
            {
                TX(tx4, T);
                TY(ty4, T);
                OUT(D2_T + 0, c.c2[0] * D2(tx4, v[T]));
                OUT(D2_T + 1, c.c2[1] * D2(ty4, v[T]));
            }
        }
#undef LV
#undef TX
#undef TY
#undef D1
#undef D1P
#undef D2
#undef OUT
        if (active && zp - 2 >= z0) {
            double *oz = D + (int64_t)(zp - 2) * c.nxy + ocol;
#define Z1(f) d1u(r[0][f], r[1][f], r[3][f], r[4][f])
#define Z1P(f, g) d1u(r[0][f] * r[0][g], r[1][f] * r[1][g], r[3][f] * r[3][g], r[4][f] * r[4][g])
#define Z2(f) d2u(r[0][f], r[1][f], r[2][f], r[3][f], r[4][f])
            oz[(D_RHO + 2) * N] = c1z * Z1(RHO);
            oz[(D_E + 2) * N] = c1z * Z1(EN);
            oz[(D_EU + 2) * N] = c1z * Z1P(EN, W);
            oz[(D_PU + 2) * N] = c1z * Z1P(P, W);
            oz[(D_P + 2) * N] = c1z * Z1(P);
            oz[(D2_T + 2) * N] = c.c2[2] * Z2(T);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                oz[(D_M + 3 * a + 2) * N] = c1z * Z1(M0 + a);
                oz[(D_U + 3 * a + 2) * N] = c1z * Z1(U + a);
                oz[(D_MU + 3 * a + 2) * N] = c1z * Z1P(M0 + a, W);
                oz[(D2_U + 3 * a + 2) * N] = c.c2[2] * Z2(U + a);
            }
            // d_z of the in-plane gradients; d_x and d_y of dw/dz as d_z of
            // dw/dx and dw/dy
            oz[(D_MIX + 1) * N] = c1z * Z1(GZX);
            oz[(D_MIX + 3) * N] = c1z * Z1(GZY);
            oz[(D_MIX + 4) * N] = c1z * Z1(GXX);
            oz[(D_MIX + 5) * N] = c1z * Z1(GYY);
#undef Z1
#undef Z1P
#undef Z2
        }
    }
}

// Residual assembled pointwise from the stored derivative arrays, and the
// Runge-Kutta update in the same pass (s.mode 0: residual only).
__global__ void __launch_bounds__(256) bl_stage_kernel(Consts c, StageArgs s, const double *__restrict__ D)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= c.N) return;
    const int64_t N = c.N;
    const double *__restrict__ Q = (const double *)s.qin;
#define DA(k) D[(int64_t)(k) * N + i]
    const double rho = Q[i], E = Q[4 * N + i];
    const double m[3] = {Q[N + i], Q[2 * N + i], Q[3 * N + i]};
    const double inv = recip_f64(rho);
    const double u[3] = {quotient_f64(m[0], rho, inv), quotient_f64(m[1], rho, inv), quotient_f64(m[2], rho, inv)};
    double G[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int j = 0; j < 3; ++j) G[a][j] = DA(D_U + 3 * a + j);
    const double div = G[0][0] + G[1][1] + G[2][2];
    double R[5];

    double r = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) r += DA(D_M + 3 * j + j) + rho * G[j][j] + u[j] * DA(D_RHO + j);
    R[0] = -0.5 * r;

    // viscous: lap u_i + (1/3)(d2 u_i/dx_i^2 + sum_{k != i} d/dx_i du_k/dx_k)
    double V[3];
    const int mix[3][2] = {{0, 1}, {2, 3}, {4, 5}};   // (i, k) pairs in D_MIX order
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double d2[3] = {DA(D2_U + 3 * a + 0), DA(D2_U + 3 * a + 1), DA(D2_U + 3 * a + 2)};
        V[a] = (d2[0] + d2[1] + d2[2]) + (d2[a] + DA(D_MIX + mix[a][0]) + DA(D_MIX + mix[a][1])) / 3.0;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double cv = 0.0;
#pragma unroll
        for (int j = 0; j < 3; ++j) cv += DA(D_MU + 3 * a + j) + m[a] * G[j][j] + u[j] * DA(D_M + 3 * a + j);
        R[1 + a] = -0.5 * cv - DA(D_P + a) + c.inv_re * V[a];
    }
    double ce = 0.0, pw = 0.0, ht = 0.0, wk = 0.0, phi = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        ce += DA(D_EU + j) + E * G[j][j] + u[j] * DA(D_E + j);
        pw += DA(D_PU + j);
        ht += DA(D2_T + j);
        wk += u[j] * V[j];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int j = 0; j < 3; ++j) phi += G[a][j] * (G[a][j] + G[j][a]);
    phi -= (2.0 / 3.0) * div * div;
    R[4] = -0.5 * ce - pw + c.inv_re * (wk + phi) + c.kappa * ht;
#undef DA
    if (s.mode == 0) {
#pragma unroll
        for (int f = 0; f < 5; ++f) s.rout[f * N + i] = R[f];
        return;
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        const double acc = s.mode == 1 ? Q[f * N + i] : s.acc_in[f * N + i];
        ((double *)s.qout)[f * N + i] = acc + s.a_dt * R[f];
        if (s.mode < 3) s.acc_out[f * N + i] = acc + s.b_dt * R[f];
    }
}

// Planes per block of the derivative pass: about 1024 blocks, two per compute
// unit at a time, so that few planes are read twice.
static int bl_zchunk(const Consts &c)
{
    const int64_t tiles = (int64_t)((c.nx + BL_BX - 1) / BL_BX) * ((c.ny + BL_BY - 1) / BL_BY);
    const int64_t chunks = (1024 + tiles - 1) / tiles;
    return (int)((c.nz + chunks - 1) / chunks);
}

hipError_t stored_stage(const Consts &c, const StageArgs &s, double *D, hipStream_t st)
{
    const int zc = bl_zchunk(c);
    const dim3 grid((c.nx + BL_BX - 1) / BL_BX, (c.ny + BL_BY - 1) / BL_BY, (c.nz + zc - 1) / zc);
    hipLaunchKernelGGL(bl_derivatives_kernel, grid, dim3(BL_NT), 0, st, c, (const double *)s.qin, D, zc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bl_stage_kernel, dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, st, c, s, D);
    return hipGetLastError();
}

}  // namespace ns
