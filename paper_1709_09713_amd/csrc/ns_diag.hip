// ns_diag.hip -- Taylor-Green initial state and the FP64 diagnostics.
//
// tgv_init writes the initial condition of the results section.
// The diagnostics are the kinetic-energy / enstrophy quantities of the
// validation data set that the results section compares against, plus the
// conserved totals: per-block partial sums (wave64 reduction by DPP moves, then
// LDS across waves) and a one-block final pass in a fixed order, so the
// result is bitwise reproducible for a given grid.
#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

__global__ void tgv_init_kernel(Consts c, double gamma, double mach, double *__restrict__ Q)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= c.N) return;
    const int i = (int)(idx % c.nx);
    const int j = (int)((idx / c.nx) % c.ny);
    const int k = (int)(idx / c.nxy);
    // x / L with L = length / (2 pi) and h = length / n: x / L = 2 pi i / n
    const double two_pi = 6.283185307179586476925286766559;
    const double x = (double)i * (two_pi / c.nx);
    const double y = (double)j * (two_pi / c.ny);
    const double z = (double)k * (two_pi / c.nz);
    double sx, cx, sy, cy, sz, cz;
    sincos(x, &sx, &cx);
    sincos(y, &sy, &cy);
    sincos(z, &sz, &cz);
    (void)sz;
    const double u = sx * cy * cz;
    const double v = -cx * sy * cz;
    const double gM2 = gamma * mach * mach;
    const double p = 1.0 / gM2 + (cos(2.0 * x) + cos(2.0 * y)) * (2.0 + cos(2.0 * z)) / 16.0;
    const double rho = gM2 * p;
    const int64_t N = c.N;
    Q[idx] = rho;
    Q[N + idx] = rho * u;
    Q[2 * N + idx] = rho * v;
    Q[3 * N + idx] = 0.0;
    Q[4 * N + idx] = p / (gamma - 1.0) + 0.5 * rho * (u * u + v * v);
}

hipError_t launch_tgv_init(const Consts &c, const ns_params *p, double *state, hipStream_t st)
{
    hipLaunchKernelGGL(tgv_init_kernel, dim3((unsigned)((c.N + 255) / 256)), dim3(256), 0, st, c,
                       p->gamma, p->mach, state);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Diagnostics partials: a block owns a 32 x 8 column tile and marches along z
// through a chunk of planes.  Each plane's velocities go through LDS for the
// x and y stencils (fd); u and v also keep a ring of five planes of the own
// column for the z stencils.  w has no z derivative in the vorticity, u no x
// and v no y derivative, so the halo is two rows (u, w) and two columns (v, w)
// on each side and no corners.
//
// Bound by memory: 40 B per point must be read; the halo rows and columns add
// about 30% of L2 reads and the planes above and below a chunk 4 / chunk.
// Whole diagnostics() calls: 256^3 561 -> 177 us, 512^3 5.03 -> 1.21 ms (4.4
// TB/s) against one thread per point gathering its neighbours through the
// caches with a division per velocity.
constexpr int kDiagBX = 32, kDiagBY = 8, kDiagThreads = kDiagBX * kDiagBY;

// Planes per block of the march.  A block steps through its chunk and four
// halo planes, and the grid runs in rounds of the 768 blocks that the device
// holds (three on each of 256 compute units): the chunk with the least rounds x
// planes, the longest of equals.  Where one layer of tiles is more than that,
// memory bounds the march whatever the rounds, and about 2048 blocks are as
// good.  Against about 2048 blocks for every grid, us per diagnostics(): 128^3
// 62 -> 49, 161x97x119 62 -> 50, 192^3 101 -> 86, 256^3 197 -> 179, 320^3 and
// above the same.
static int diag_zchunk(const Consts &c)
{
    constexpr int kResident = 768;
    const int tiles = ((c.nx + kDiagBX - 1) / kDiagBX) * ((c.ny + kDiagBY - 1) / kDiagBY);
    if (tiles > kResident) {
        const int chunks = (2048 + tiles - 1) / tiles;
        return (c.nz + chunks - 1) / chunks;
    }
    int best = c.nz;
    int64_t best_cost = INT64_MAX;
    // k chunks of z planes, for each z the smallest k
    for (int k = 1;;) {
        const int z = (c.nz + k - 1) / k;
        const int64_t cost = (int64_t)((tiles * k + kResident - 1) / kResident) * (z + 4);
        if (cost < best_cost) {
            best_cost = cost;
            best = z;
        }
        if (z <= 1) break;
        k = (c.nz + z - 2) / (z - 1);
    }
    return best;
}

// Grids of fewer points than this take one thread per point instead
// (diag_point_kernel): a march is at least five dependent plane loads, which
// a small grid cannot hide.  diagnostics() calls, point kernel | march: 16^3
// 29.8 | 32.1, 64^3 35.5 | 40.0, 101x77x53 43.5 | 43.6, 128^3 (as it was) 86 | 61 us.
constexpr int64_t kDiagMarchPoints = (int64_t)1 << 19;

static bool diag_march(const Consts &c) { return c.N >= kDiagMarchPoints; }

static dim3 diag_grid(const Consts &c)
{
    if (!diag_march(c)) return dim3((unsigned)((c.N + kDiagThreads - 1) / kDiagThreads));
    const int zc = diag_zchunk(c);
    return dim3((c.nx + kDiagBX - 1) / kDiagBX, (c.ny + kDiagBY - 1) / kDiagBY, (c.nz + zc - 1) / zc);
}

int64_t diag_num_blocks(const Consts &c)
{
    const dim3 g = diag_grid(c);
    return (int64_t)g.x * g.y * g.z;
}

// Block sum of the seven per-thread sums in a fixed order, into the block's
// partial record.
__device__ __forceinline__ void diag_block_sum(double (&s)[7], double *__restrict__ partial, int64_t blin)
{
    __shared__ double red[kDiagThreads / 64][kDiag];
#pragma unroll
    for (int q = 0; q < 7; ++q) s[q] = wave_sum(s[q]);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 63)
        for (int q = 0; q < 7; ++q) red[wave][q] = s[q];
    __syncthreads();
    if (threadIdx.x < kDiag) {
        double t = 0.0;
        for (int wv = 0; wv < kDiagThreads / 64 && threadIdx.x < 7; ++wv) t += red[wv][threadIdx.x];
        partial[blin * kDiag + threadIdx.x] = t;
    }
}

// One thread per point, neighbours through the caches.
__global__ void __launch_bounds__(kDiagThreads)
diag_point_kernel(Consts c, const double *__restrict__ Q, double *__restrict__ partial)
{
    const int64_t idx = (int64_t)blockIdx.x * kDiagThreads + threadIdx.x;
    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    if (idx < c.N) {
        const int64_t N = c.N;
        const int i = (int)(idx % c.nx);
        const int j = (int)((idx / c.nx) % c.ny);
        const int k = (int)(idx / c.nxy);
        const int co[3] = {i, j, k};
        const int nn[3] = {c.nx, c.ny, c.nz};
        const int64_t st[3] = {1, c.nx, c.nxy};
        // G[d][e] = D_d of the two velocities other than u_d: (d + 1) % 3 and (d + 2) % 3
        double G[3][2];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int off[4] = {-2, -1, 1, 2};
            double t[2][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t at = idx + (int64_t)(wrap1(co[d] + off[q], nn[d]) - co[d]) * st[d];
                const double rho = Q[at], inv = recip_f64(rho);
#pragma unroll
                for (int e = 0; e < 2; ++e) t[e][q] = quotient_f64(Q[(1 + (d + 1 + e) % 3) * N + at], rho, inv);
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) G[d][e] = c.c1[d] * d1u(t[e][0], t[e][1], t[e][2], t[e][3]);
        }
        const double rho = Q[idx];
        const double m0 = Q[N + idx], m1 = Q[2 * N + idx], m2 = Q[3 * N + idx];
        const double ox = G[1][0] - G[2][1], oy = G[2][0] - G[0][1], oz = G[0][0] - G[1][1];
        s[0] = rho;
        s[1] = m0;
        s[2] = m1;
        s[3] = m2;
        s[4] = Q[4 * N + idx];
        s[5] = 0.5 * (m0 * m0 + m1 * m1 + m2 * m2) / rho;
        s[6] = 0.5 * rho * (ox * ox + oy * oy + oz * oz);
    }
    diag_block_sum(s, partial, blockIdx.x);
}

// Three waves per SIMD and no more: a fourth has larger grids' planes leave L2
// before the neighbouring blocks have read them (512^3 1221 -> 1340 us).
__global__ void __launch_bounds__(kDiagThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
diag_march_kernel(Consts c, const double *__restrict__ Q, double *__restrict__ partial, int zchunk)
{
    constexpr int BX = kDiagBX, BY = kDiagBY, HX = BX + 4, HY = BY + 4;
    constexpr int YH = 4 * BX, XH = 4 * BY;      // halo points above and below, left and right
    static_assert(YH + XH <= kDiagThreads, "one halo point per thread");
    __shared__ double lu[2][HY][BX];             // u: own columns, two halo rows each side
    __shared__ double lv[2][BY][HX];             // v: own rows, two halo columns each side
    __shared__ double lw[2][HY][HX];             // w: both
    const int tid = threadIdx.x, tx = tid % BX, ty = tid / BX;
    int tbx, tby, tbz;
    xcd_tile(&tbx, &tby, &tbz);
    const int x0 = tbx * BX, y0 = tby * BY;
    const int z0 = tbz * zchunk, z1 = min(z0 + zchunk, c.nz);
    const bool active = x0 + tx < c.nx && y0 + ty < c.ny;
    const int64_t N = c.N;
    // Own column (wrapped, valid memory beyond the grid: a partial tile's
    // last columns read their halo there) and this thread's halo point.
    const int ox = (x0 + tx) % c.nx, oy = (y0 + ty) % c.ny;
    const int ocol = oy * c.nx + ox;
    const bool yhalo = tid < YH, xhalo = tid >= YH && tid < YH + XH;
    int hx = 0, hy = 0;                          // cell in the tile with its halo
    if (yhalo) {
        const int row = tid / BX;
        hx = tid % BX + 2;
        hy = row < 2 ? row : BY + row;
    } else if (xhalo) {
        const int q = tid - YH, cc = q % 4;
        hx = cc < 2 ? cc : BX + cc;
        hy = q / 4 + 2;
    }
    int hxx = (x0 + hx - 2) % c.nx, hyy = (y0 + hy - 2) % c.ny;
    if (hxx < 0) hxx += c.nx;
    if (hyy < 0) hyy += c.ny;
    const int hcol = hyy * c.nx + hxx;
    const int64_t hf = yhalo ? N : 2 * N;        // the halo point's second velocity: u or v

    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    double qu[5], qv[5];                         // u, v of the own column, planes zp-4 .. zp
    double qx[3], qy[3], qr[3];                  // D_x w, D_y w, rho of planes zp-2 .. zp
#pragma unroll
    for (int k = 0; k < 5; ++k) qu[k] = qv[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) qx[k] = qy[k] = qr[k] = 0.0;

    double p0[5], ph[3];                         // next plane: own point, halo point
    auto load = [&](int zp) {
        int zw = zp % c.nz;
        if (zw < 0) zw += c.nz;
        const double *q = Q + (int64_t)zw * c.nxy;
#pragma unroll
        for (int f = 0; f < 5; ++f) p0[f] = q[f * N + ocol];
        // threads without a halo point read the tile's first one
        ph[0] = q[hcol];
        ph[1] = q[hf + hcol];
        ph[2] = q[3 * N + hcol];
    };

    load(z0 - 2);
    for (int zp = z0 - 2; zp < z1 + 2; ++zp) {
        const int b = (zp - z0) & 1;
        const double rho = p0[0], m0 = p0[1], m1 = p0[2], m2 = p0[3], E = p0[4];
        const double inv = recip_f64(rho);
        const double u = quotient_f64(m0, rho, inv), v = quotient_f64(m1, rho, inv), w = quotient_f64(m2, rho, inv);
        lu[b][ty + 2][tx] = u;
        lv[b][ty][tx + 2] = v;
        lw[b][ty + 2][tx + 2] = w;
        if (yhalo || xhalo) {
            const double hinv = recip_f64(ph[0]);
            const double hv = quotient_f64(ph[1], ph[0], hinv);
            if (yhalo)
                lu[b][hy][hx - 2] = hv;
            else
                lv[b][hy - 2][hx] = hv;
            lw[b][hy][hx] = quotient_f64(ph[2], ph[0], hinv);
        }
        lds_barrier();
        if (zp + 1 < z1 + 2) load(zp + 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            qu[k] = qu[k + 1];
            qv[k] = qv[k + 1];
        }
        qu[4] = u;
        qv[4] = v;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            qx[k] = qx[k + 1];
            qy[k] = qy[k + 1];
            qr[k] = qr[k + 1];
        }
        qr[2] = rho;
        if (zp >= z0 && zp < z1) {
            qx[2] = c.c1[0] * d1u(lw[b][ty + 2][tx], lw[b][ty + 2][tx + 1], lw[b][ty + 2][tx + 3], lw[b][ty + 2][tx + 4]);
            qy[2] = c.c1[1] * d1u(lw[b][ty][tx + 2], lw[b][ty + 1][tx + 2], lw[b][ty + 3][tx + 2], lw[b][ty + 4][tx + 2]);
            const double oz = c.c1[0] * d1u(lv[b][ty][tx], lv[b][ty][tx + 1], lv[b][ty][tx + 3], lv[b][ty][tx + 4])
                              - c.c1[1] * d1u(lu[b][ty][tx], lu[b][ty + 1][tx], lu[b][ty + 3][tx], lu[b][ty + 4][tx]);
            if (active) {
                s[0] += rho;
                s[1] += m0;
                s[2] += m1;
                s[3] += m2;
                s[4] += E;
                s[5] += 0.5 * (m0 * u + m1 * v + m2 * w);
                s[6] += 0.5 * rho * (oz * oz);
            }
        }
        // the vorticity components with z derivatives of plane zp - 2
        if (active && zp - 2 >= z0) {
            const double wx = qy[0] - c.c1[2] * d1u(qv[0], qv[1], qv[3], qv[4]);
            const double wy = c.c1[2] * d1u(qu[0], qu[1], qu[3], qu[4]) - qx[0];
            s[6] += 0.5 * qr[0] * (wx * wx + wy * wy);
        }
    }
    diag_block_sum(s, partial, ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
}

hipError_t launch_diag_partials(const Consts &c, const double *state, double *partial, hipStream_t st)
{
    if (diag_march(c))
        hipLaunchKernelGGL(diag_march_kernel, diag_grid(c), dim3(kDiagThreads), 0, st, c, state, partial,
                           diag_zchunk(c));
    else
        hipLaunchKernelGGL(diag_point_kernel, diag_grid(c), dim3(kDiagThreads), 0, st, c, state, partial);
    return hipGetLastError();
}

// Fixed-order final reduction: thread t sums partials t, t+256, ... in
// order; then a fixed pairwise tree over the 256 thread sums.
__global__ void __launch_bounds__(256)
diag_finalize_kernel(Consts c, const double *__restrict__ partial, int64_t nblocks, ns_diag *out)
{
    __shared__ double red[256][7];
    const int t = threadIdx.x;
    double s[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t b = t; b < nblocks; b += 256)
#pragma unroll
        for (int q = 0; q < 7; ++q) s[q] += partial[b * kDiag + q];
#pragma unroll
    for (int q = 0; q < 7; ++q) red[t][q] = s[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w)
#pragma unroll
            for (int q = 0; q < 7; ++q) red[t][q] += red[t + w][q];
        __syncthreads();
    }
    if (t == 0) {
        const double v[7] = {red[0][0], red[0][1], red[0][2], red[0][3], red[0][4], red[0][5], red[0][6]};
        write_diag(c, v, out);
    }
}

hipError_t launch_diag_finalize(const Consts &c, const double *partial, int64_t nblocks, ns_diag *out,
                                hipStream_t st)
{
    hipLaunchKernelGGL(diag_finalize_kernel, dim3(1), dim3(256), 0, st, c, partial, nblocks, out);
    return hipGetLastError();
}

}  // namespace ns
