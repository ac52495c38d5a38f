// ns_fp64.hpp -- arithmetic shared by the FP64 stage kernels that split a
// point's work over groups of waves (ns_trio.hip, ns_brick.hip): both evaluate
// the same expressions in the same order, so a point's result does not depend
// on which of them computed it.
#pragma once

#include "ns_common.hpp"

namespace ns {

// Coefficients of the stencils with their weights and physical constants
// folded in on the host: uniform double products formed in the kernel would
// be held in two vector registers each for the whole march.
struct Coef64 {
    double x4, xh, y4, yh, z4, zh;   // 4 c1 and c1 / 2 of each direction
    double gx, gy, gz, gz8;          // (gamma - 1) c1 of each direction, 8 (gamma - 1) c1_z
    double kx, ky, kz, kz16;         // kappa T / e c2 of each direction, 16 times that of z; T = gamma (gamma - 1) M^2 e
    double vx, vy, vz;               // 4/3 c2 of each direction
    double mx, my, mz, mxy;          // c1 / 3 of each direction, c1_x c1_y / 3
};

inline Coef64 make_coef64(const Consts &c)
{
    Coef64 k;
    k.x4 = 4.0 * c.c1[0];
    k.xh = 0.5 * c.c1[0];
    k.y4 = 4.0 * c.c1[1];
    k.yh = 0.5 * c.c1[1];
    k.z4 = 4.0 * c.c1[2];
    k.zh = 0.5 * c.c1[2];
    k.gx = c.gm1 * c.c1[0];
    k.gy = c.gm1 * c.c1[1];
    k.gz = c.gm1 * c.c1[2];
    k.gz8 = 8.0 * k.gz;
    const double ke = c.kappa * c.gM2 * c.gm1;
    k.kx = ke * c.c2[0];
    k.ky = ke * c.c2[1];
    k.kz = ke * c.c2[2];
    k.kz16 = 16.0 * k.kz;
    k.vx = 4.0 * c.c2[0] / 3.0;
    k.vy = 4.0 * c.c2[1] / 3.0;
    k.vz = 4.0 * c.c2[2] / 3.0;
    k.mx = c.c1[0] / 3.0;
    k.my = c.c1[1] / 3.0;
    k.mxy = c.c1[0] * c.c1[1] / 3.0;
    k.mz = c.c1[2] / 3.0;
    return k;
}

// Unscaled first- and second-derivative stencils with the multiply-adds
// written out: a product left to the compiler (30 f_0, say) can be shared
// with another plane's step, fused in one phase of the march and not in
// another, and a point's rounding would depend on its place in a z-chunk.
__device__ __forceinline__ double d1(double fm2, double fm1, double fp1, double fp2)
{
    return __builtin_fma(8.0, fp1 - fm1, fm2 - fp2);
}
__device__ __forceinline__ double d2(double fm2, double fm1, double f0, double fp1, double fp2)
{
    return __builtin_fma(-30.0, f0, __builtin_fma(16.0, fm1 + fp1, -(fm2 + fp2)));
}

// Differences f_k - f_0 of the taps k = -2, -1, 1, 2 to the point's own value.
__device__ __forceinline__ void diffs(double f0, const double (&t)[4], double (&d)[4])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = t[q] - f0;
}

// acc - sum_k c_k (f_k - f_0) (u_0 + u_k) / 2 with the differences d[] of f and
// the weighted velocity sums s[k] = |c_k| (u_0 + u_k) / 2.
__device__ __forceinline__ double conv(double acc, const double (&d)[4], const double (&s)[4])
{
    acc = __builtin_fma(-d[0], s[0], acc);
    acc = __builtin_fma(d[1], s[1], acc);
    acc = __builtin_fma(-d[2], s[2], acc);
    return __builtin_fma(d[3], s[3], acc);
}
__device__ __forceinline__ double conv(double acc, double f0, const double (&t)[4], const double (&s)[4])
{
    double d[4];
    diffs(f0, t, d);
    return conv(acc, d, s);
}

// (p_k - p_0) / (gamma - 1) of the taps from the differences of energy and
// kinetic energy.
__device__ __forceinline__ void pressure_diffs(const double (&dE)[4], double K, const double (&kt)[4], double (&d)[4])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = dE[q] - (kt[q] - K);
}

// unscaled first derivative of the product of two fields at the taps
__device__ __forceinline__ double d1_prod(const double (&f)[4], const double (&g)[4])
{
    const double far = __builtin_fma(f[0], g[0], -(f[3] * g[3]));
    const double near = __builtin_fma(f[2], g[2], -(f[1] * g[1]));
    return __builtin_fma(8.0, near, far);
}

}  // namespace ns
