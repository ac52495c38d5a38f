"""FP64 residuals of states far from any uniform reference state: density and
energy a small or large multiple of the Taylor-Green vortex's, an inviscid gas
whose energy the Mach number does not tell, and a fast mean flow.  All storage
and arithmetic is in double, so the error of every class, tile and grid size is
bounded by the rounding of the state's own values.

Bound: a point's residual is a sum of products of staged values, and no term
passes more than 32 roundings (reciprocal 3, velocity 1, kinetic energy 4,
pressure 2, temperature 2, stencil 5, weights 3, at most 12 additions of
terms), so |R - R_exact| <= 32 u B, with u = 2^-53 and B the sum of the terms'
magnitudes at the point.  R_exact and B are NumPy in 80-bit arithmetic."""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import numpy_ref

pytestmark = pytest.mark.gpu

LD = np.longdouble
GAMMA, PRANDTL = 1.4, 0.71


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


def state(kind, n):
    """(Q, Reynolds, Mach)"""
    Q = synth.random_state(n[::-1], seed=n[0] + n[2])
    if kind.startswith("scaled"):
        return Q * float(kind.split()[1]), 1600.0, 0.1
    if kind == "inviscid":
        # p about 1 where the reference state of this Mach number has 7e5
        Q[4] = Q[4] - 180.0 + 5.0
        return Q, math.inf, 1e-3
    # mean flow
    rho = Q[0].copy()
    for a, u in enumerate((5.0, 3.0, -2.0)):
        Q[1 + a] += rho * u
    Q[4] += 40.0
    return Q, math.inf, 0.3


def abs1(f, d, h):
    """Sum of the magnitudes of the first-derivative stencil's terms."""
    return sum(w * numpy_ref._sh(f, d, s) for w, s in ((8, -1), (8, 1), (1, -2), (1, 2))) / (12 * h[d])


def abs2(f, d, h):
    return (sum(w * numpy_ref._sh(f, d, s) for w, s in ((16, -1), (16, 1), (1, -2), (1, 2))) + 30 * f) / (12 * h[d] ** 2)


def magnitude(Q, h, re, mach):
    """Sum of the magnitudes of a residual's terms."""
    rho, m, E = Q[0], np.abs(Q[1:4]), Q[4]
    u = m / rho
    p = (GAMMA - 1) * (E + 0.5 * (m * u).sum(axis=0))
    T = GAMMA * mach ** 2 * p / rho
    inv_re = 0.0 if math.isinf(re) else 1.0 / re
    kappa = inv_re / ((GAMMA - 1) * mach ** 2 * PRANDTL)
    B = np.zeros_like(Q)
    V = [np.zeros_like(rho) for _ in range(3)]
    g = [[abs1(u[i], j, h) for j in range(3)] for i in range(3)]
    for f, q in enumerate((rho, m[0], m[1], m[2], E)):
        for j in range(3):
            B[f] += 0.5 * (abs1(q * u[j], j, h) + q * g[j][j] + u[j] * abs1(q, j, h))
    for i in range(3):
        for j in range(3):
            V[i] += abs2(u[i], j, h)
            V[i] += (abs2(u[i], i, h) if i == j else abs1(g[j][j], i, h)) / 3
        B[1 + i] += abs1(p, i, h) + inv_re * V[i]
        B[4] += abs1(p * u[i], i, h) + inv_re * u[i] * V[i] + kappa * abs2(T, i, h)
        for j in range(3):
            B[4] += inv_re * g[i][j] * (g[i][j] + g[j][i]) + inv_re * (2.0 / 3.0) * g[i][i] * g[j][j]
    return B


def check(ns, algo, n, kind, tiles):
    Q, re, mach = state(kind, n)
    h = [LD(2 * math.pi) / k for k in n]
    QL = Q.astype(LD)
    want = numpy_ref.residual(QL, h, LD(GAMMA), LD(PRANDTL), LD(re), LD(mach))
    bound = 32 * LD(2.0) ** -53 * magnitude(QL, h, re, LD(mach))
    p = ns.make_params(n, reynolds=re, mach=mach)
    Qd = torch.as_tensor(Q, device="cuda")
    work = torch.empty(ns.ns_workspace_bytes(p, ns.ALGOS[algo], ns.NS_FP64), dtype=torch.uint8, device="cuda")
    for tile in tiles:
        print(f"reference free {algo} n={n} {kind} tile={tile}", flush=True)
        R = torch.empty_like(Qd)
        ns.ns_set_fused_config(tile, 0)
        try:
            ns.ns_residual(p, ns.ALGOS[algo], Qd, R, work)
            torch.cuda.synchronize()
        finally:
            ns.ns_set_fused_config(-1, 0)
        err = np.abs(R.cpu().numpy().astype(LD) - want)
        worst = [float((err[f] / bound[f]).max()) for f in range(5)]
        print("  error over bound", ["%.2f" % w for w in worst], flush=True)
        assert max(worst) <= 1.0, (tile, worst)


KINDS = ["scaled 1", "scaled 1e-2", "scaled 1e-4", "scaled 1e4", "inviscid", "mean flow"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [(16, 12, 10), (33, 18, 20), (64, 40, 28)])
def test_fused(ns, n, kind):
    """Bricks of two and four planes or the march, and the tiles."""
    check(ns, "fused", n, kind, (-1, 4, 8, 9, 10))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("algo,n", [("stored", (33, 18, 20)), ("some", (33, 18, 20)), ("some", (80, 80, 63))])
def test_classes(ns, algo, n, kind):
    check(ns, algo, n, kind, (-1,))
