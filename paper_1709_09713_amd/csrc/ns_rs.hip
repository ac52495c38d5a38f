// ns_rs.hip -- the intermediate-storage algorithm class (RS / SS of the
// algorithms section): only the nine velocity-gradient components
// du_i/dx_j are kept in global arrays, every other derivative is evaluated
// inline at the point that needs it.
//
// Per RK stage: rs_gradient_kernel evaluates the nine gradients and stores
// them; the three-group stage kernel (ns_trio.hip, GRAD) then evaluates the
// residual of the governing-equations section -- convective, pressure, heat
// conduction and second derivatives inline from LDS-staged planes; div u, the
// dissipation and the mixed viscous derivatives d/dx_i (du_k/dx_k) from the
// stored arrays -- and applies the low-storage RK update of the
// generic-algorithm figure in the same pass.  Small grids take one thread per
// point with every tap through the caches instead.  FP64 only.
#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

namespace {

constexpr int RS_BX = 32, RS_BY = 8, RS_NT = RS_BX * RS_BY;

// A block owns a 32 x 8 column tile and marches along z: each plane's
// velocities go through LDS for the x and y gradients, which are stored in
// the plane's step; the z gradients of plane zp - 2 come from a ring of five
// planes of the own column.  No corners: a gradient has taps in one direction
// only.
//
// Bound by memory: 32 B read and 72 B written per point (0.38 ms at 256^3,
// 4.6 TB/s; one thread per point, three divisions per tap: 0.75 ms).
__global__ void __launch_bounds__(RS_NT)
rs_gradient_kernel(Consts c, const double *__restrict__ Q, double *__restrict__ G, int zchunk)
{
    constexpr int HX = RS_BX + 4, HY = RS_BY + 4;
    constexpr int YH = 4 * RS_BX, XH = 4 * RS_BY;   // halo points above and below, left and right
    static_assert(YH + XH <= RS_NT, "one halo point per thread");
    __shared__ double lu[2][3][HY][HX];
    const int tid = threadIdx.x, tx = tid % RS_BX, ty = tid / RS_BX;
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz);
    const int x0 = tbx * RS_BX, y0 = tby * RS_BY;
    const int z0 = tbz * zchunk, z1 = min(z0 + zchunk, c.nz);
    const bool active = x0 + tx < c.nx && y0 + ty < c.ny;
    const int64_t N = c.N;
    // Own column, wrapped beyond the grid: a partial tile's last columns read
    // their halo there.
    const int ocol = ((y0 + ty) % c.ny) * c.nx + (x0 + tx) % c.nx;
    const bool halo = tid < YH + XH;
    int hx = 2, hy = 2;   // threads without a halo point read the tile's first point
    if (tid < YH) {
        const int row = tid / RS_BX;
        hx = tid % RS_BX + 2;
        hy = row < 2 ? row : RS_BY + row;
    } else if (halo) {
        const int q = tid - YH, cc = q % 4;
        hx = cc < 2 ? cc : RS_BX + cc;
        hy = q / 4 + 2;
    }
    int hxx = (x0 + hx - 2) % c.nx, hyy = (y0 + hy - 2) % c.ny;
    if (hxx < 0) hxx += c.nx;
    if (hyy < 0) hyy += c.ny;
    const int hcol = hyy * c.nx + hxx;

    double po[4], ph[4];   // rho and momenta of the next plane: own and halo point
    auto load = [&](int zp) {
        int zw = zp % c.nz;
        if (zw < 0) zw += c.nz;
        const double *q = Q + (int64_t)zw * c.nxy;
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            po[f] = q[f * N + ocol];
            ph[f] = q[f * N + hcol];
        }
    };
    double qz[5][3];       // u, v, w of planes zp - 4 .. zp
#pragma unroll
    for (int k = 0; k < 5; ++k) qz[k][0] = qz[k][1] = qz[k][2] = 0.0;

    load(z0 - 2);
    for (int zp = z0 - 2; zp < z1 + 2; ++zp) {
        const int b = (zp - z0) & 1;
        const double inv = recip_f64(po[0]);
        double u[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            u[a] = quotient_f64(po[1 + a], po[0], inv);
            lu[b][a][ty + 2][tx + 2] = u[a];
        }
        if (halo) {
            const double hinv = recip_f64(ph[0]);
#pragma unroll
            for (int a = 0; a < 3; ++a) lu[b][a][hy][hx] = quotient_f64(ph[1 + a], ph[0], hinv);
        }
        lds_barrier();
        if (zp + 1 < z1 + 2) load(zp + 1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int k = 0; k < 4; ++k) qz[k][a] = qz[k + 1][a];
            qz[4][a] = u[a];
        }
        if (active && zp >= z0 && zp < z1) {
            double *g = G + (int64_t)zp * c.nxy + ocol;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double(&l)[HY][HX] = lu[b][a];
                g[(3 * a) * N] = c.c1[0] * d1u(l[ty + 2][tx], l[ty + 2][tx + 1], l[ty + 2][tx + 3], l[ty + 2][tx + 4]);
                g[(3 * a + 1) * N] = c.c1[1] * d1u(l[ty][tx + 2], l[ty + 1][tx + 2], l[ty + 3][tx + 2], l[ty + 4][tx + 2]);
            }
        }
        if (active && zp - 2 >= z0) {
            double *g = G + (int64_t)(zp - 2) * c.nxy + ocol;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                g[(3 * a + 2) * N] = c.c1[2] * d1u(qz[0][a], qz[1][a], qz[3][a], qz[4][a]);
        }
    }
}

// Planes per block of the gradient sweep: about 2048 blocks (up to eight fit
// on a compute unit), so that few planes are read twice.
int gradient_zchunk(const Consts &c)
{
    const int64_t tiles = (int64_t)((c.nx + RS_BX - 1) / RS_BX) * ((c.ny + RS_BY - 1) / RS_BY);
    const int64_t chunks = (2048 + tiles - 1) / tiles;
    return (int)((c.nz + chunks - 1) / chunks);
}

// ---------------------------------------------------------------- small grids
// One thread per point, taps through the caches.
constexpr int PT_BX = 64, PT_BY = 4;

// Offsets of the four taps of direction d around (i, j, k), periodic.
struct Taps {
    int64_t m2, m1, p1, p2;
};

__device__ __forceinline__ Taps taps(const Consts &c, int i, int j, int k, int d)
{
    int co, n;
    int64_t stride;
    if (d == 0) { co = i; n = c.nx; stride = 1; }
    else if (d == 1) { co = j; n = c.ny; stride = c.nx; }
    else { co = k; n = c.nz; stride = c.nxy; }
    Taps t;
    t.m2 = (int64_t)(wrap1(co - 2, n) - co) * stride;
    t.m1 = (int64_t)(wrap1(co - 1, n) - co) * stride;
    t.p1 = (int64_t)(wrap1(co + 1, n) - co) * stride;
    t.p2 = (int64_t)(wrap1(co + 2, n) - co) * stride;
    return t;
}

// Primitive values at one stencil tap, from the conserved state.  Every
// point that uses a tap recomputes them, so they are evaluated without
// multiply-add contraction: each value is rounded once, identically in
// every context, and the periodic sums of the flux differences telescope
// exactly as with values stored once (discrete conservation).
struct TapVals {
    double rho, m[3], E, u[3], p, T;
};

__device__ __forceinline__ TapVals tap_vals(const Consts &c, const double *__restrict__ Q, int64_t at)
{
#pragma clang fp contract(off)
    const int64_t N = c.N;
    TapVals v;
    v.rho = Q[at];
    v.m[0] = Q[N + at];
    v.m[1] = Q[2 * N + at];
    v.m[2] = Q[3 * N + at];
    v.E = Q[4 * N + at];
    const double inv = 1.0 / v.rho;
#pragma unroll
    for (int a = 0; a < 3; ++a) v.u[a] = v.m[a] * inv;
    v.p = c.gm1 * (v.E - 0.5 * (v.m[0] * v.u[0] + v.m[1] * v.u[1] + v.m[2] * v.u[2]));
    v.T = c.gM2 * v.p * inv;
    return v;
}

// Product of two tap values, rounded once (see tap_vals).
__device__ __forceinline__ double tap_prod(double a, double b)
{
#pragma clang fp contract(off)
    return a * b;
}

__device__ __forceinline__ double tap_velocity(double m, double inv)
{
#pragma clang fp contract(off)
    return m * inv;
}

__global__ void __launch_bounds__(PT_BX * PT_BY)
rs_point_gradient_kernel(Consts c, const double *__restrict__ Q, double *__restrict__ G)
{
    const int i = blockIdx.x * PT_BX + threadIdx.x, j = blockIdx.y * PT_BY + threadIdx.y;
    const int k = blockIdx.z;
    if (i >= c.nx || j >= c.ny) return;
    const int64_t idx = (int64_t)k * c.nxy + (int64_t)j * c.nx + i;
    const int64_t N = c.N;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const Taps t = taps(c, i, j, k, d);
        const int64_t at[4] = {idx + t.m2, idx + t.m1, idx + t.p1, idx + t.p2};
        double u[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double inv = 1.0 / Q[at[q]];
#pragma unroll
            for (int a = 0; a < 3; ++a) u[q][a] = tap_velocity(Q[(1 + a) * N + at[q]], inv);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a)
            G[(3 * a + d) * N + idx] = c.c1[d] * d1u(u[0][a], u[1][a], u[2][a], u[3][a]);
    }
}

__global__ void __launch_bounds__(PT_BX * PT_BY) rs_point_stage_kernel(Consts c, StageArgs s)
{
    const int i = blockIdx.x * PT_BX + threadIdx.x, j = blockIdx.y * PT_BY + threadIdx.y;
    const int k = blockIdx.z;
    if (i >= c.nx || j >= c.ny) return;
    const int64_t idx = (int64_t)k * c.nxy + (int64_t)j * c.nx + i;
    const int64_t N = c.N;
    const double *__restrict__ Q = (const double *)s.qin;
    const double *__restrict__ G = s.grad;

    const TapVals o = tap_vals(c, Q, idx);
    double g[3][3];   // g[a][d] = du_a / dx_d (stored)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = 0; d < 3; ++d) g[a][d] = G[(3 * a + d) * N + idx];
    const double div = g[0][0] + g[1][1] + g[2][2];

    // Derivatives recomputed inline from the taps of each direction d.
    double dm_sum = 0.0;                 // sum_d D_d m_d
    double urho = 0.0, uE = 0.0;         // sum_d u_d D_d rho, sum_d u_d D_d rhoE
    double dEu = 0.0, dpu = 0.0;         // sum_d D_d (rhoE u_d), sum_d D_d (p u_d)
    double lapT = 0.0;                   // sum_d D2_d T
    double dmu[3] = {0.0, 0.0, 0.0};     // sum_d D_d (m_a u_d)
    double udm[3] = {0.0, 0.0, 0.0};     // sum_d u_d D_d m_a
    double lapu[3] = {0.0, 0.0, 0.0};    // sum_d D2_d u_a
    double d2ii[3];                      // D2_a u_a
    double dp[3];                        // D_a p
    double mixv[3];                      // sum_{k != a} D_a (du_k/dx_k)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const Taps t = taps(c, i, j, k, d);
        const TapVals a = tap_vals(c, Q, idx + t.m2), b = tap_vals(c, Q, idx + t.m1);
        const TapVals e = tap_vals(c, Q, idx + t.p1), f = tap_vals(c, Q, idx + t.p2);
        const double c1 = c.c1[d], c2 = c.c2[d];
#define D1(x) (c1 * d1u(a.x, b.x, e.x, f.x))
#define D2(x) (c2 * d2u(a.x, b.x, o.x, e.x, f.x))
        dm_sum += D1(m[d]);
        urho += o.u[d] * D1(rho);
        uE += o.u[d] * D1(E);
        dEu += c1 * d1u(tap_prod(a.E, a.u[d]), tap_prod(b.E, b.u[d]), tap_prod(e.E, e.u[d]),
                        tap_prod(f.E, f.u[d]));
        dpu += c1 * d1u(tap_prod(a.p, a.u[d]), tap_prod(b.p, b.u[d]), tap_prod(e.p, e.u[d]),
                        tap_prod(f.p, f.u[d]));
        lapT += D2(T);
        dp[d] = D1(p);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            dmu[q] += c1 * d1u(tap_prod(a.m[q], a.u[d]), tap_prod(b.m[q], b.u[d]),
                               tap_prod(e.m[q], e.u[d]), tap_prod(f.m[q], f.u[d]));
            udm[q] += o.u[d] * D1(m[q]);
            const double d2 = D2(u[q]);
            lapu[q] += d2;
            if (q == d) d2ii[q] = d2;
        }
#undef D1
#undef D2
        // mixed: D_d of the stored diagonal gradients of the other directions
        double mx = 0.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (q == d) continue;
            const double *Gq = G + (int64_t)(4 * q) * N;   // du_q / dx_q
            mx += c1 * d1u(Gq[idx + t.m2], Gq[idx + t.m1], Gq[idx + t.p1], Gq[idx + t.p2]);
        }
        mixv[d] = mx;
    }

    double R[5];
    R[0] = -0.5 * (dm_sum + o.rho * div + urho);
    double V[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        V[a] = lapu[a] + (d2ii[a] + mixv[a]) / 3.0;
        R[1 + a] = -0.5 * (dmu[a] + o.m[a] * div + udm[a]) - dp[a] + c.inv_re * V[a];
    }
    double phi = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = 0; d < 3; ++d) phi += g[a][d] * (g[a][d] + g[d][a]);
    phi -= (2.0 / 3.0) * div * div;
    const double work = o.u[0] * V[0] + o.u[1] * V[1] + o.u[2] * V[2];
    R[4] = -0.5 * (dEu + o.E * div + uE) - dpu + c.inv_re * (work + phi) + c.kappa * lapT;

    if (s.mode == 0) {
#pragma unroll
        for (int f = 0; f < 5; ++f) s.rout[f * N + idx] = R[f];
        return;
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        const double acc = (s.mode == 1) ? Q[f * N + idx] : s.acc_in[f * N + idx];
        ((double *)s.qout)[f * N + idx] = acc + s.a_dt * R[f];
        if (s.mode < 3) s.acc_out[f * N + idx] = acc + s.b_dt * R[f];
    }
}

dim3 point_grid(const Consts &c) { return dim3((c.nx + PT_BX - 1) / PT_BX, (c.ny + PT_BY - 1) / PT_BY, c.nz); }

// The marching kernels' blocks step through at least five planes one after
// another, which small grids cannot hide.  ms per RK3 step, one thread per
// point | marching: 16^3 0.033 | 0.052, 64^3 0.092 | 0.110, 101x77x53 (412,000
// points) 0.170 | 0.159, 128^3 0.786 | 0.476, 256^3 6.14 | 3.46.
constexpr int64_t kMarchPoints = 400000;

}  // namespace

size_t rs_workspace_doubles(const Consts &c) { return 9 * (size_t)c.N; }

hipError_t rs_stage(const Consts &c, const double *qin, double *G, const double *acc_in, double *acc_out,
                    double *qout, double *rout, double a_dt, double b_dt, int mode, int zchunk, hipStream_t st)
{
    StageArgs a = {};
    a.qin = qin;
    a.grad = G;
    a.acc_in = acc_in;
    a.acc_out = acc_out;
    a.qout = qout;
    a.rout = rout;
    a.a_dt = a_dt;
    a.b_dt = b_dt;
    a.mode = mode;
    a.zchunk = zchunk;
    if (c.N < kMarchPoints) {
        hipLaunchKernelGGL(rs_point_gradient_kernel, point_grid(c), dim3(PT_BX, PT_BY, 1), 0, st, c, qin, G);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(rs_point_stage_kernel, point_grid(c), dim3(PT_BX, PT_BY, 1), 0, st, c, a);
        return hipGetLastError();
    }
    const int gz = gradient_zchunk(c);
    const dim3 grid((c.nx + RS_BX - 1) / RS_BX, (c.ny + RS_BY - 1) / RS_BY, (c.nz + gz - 1) / gz);
    hipLaunchKernelGGL(rs_gradient_kernel, grid, dim3(RS_NT), 0, st, c, qin, G, gz);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_trio_grad(c, a, st);
}

}  // namespace ns
