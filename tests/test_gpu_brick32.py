"""The brick kernel of small FP32-storage grids (automatic launch shape) against
the one-thread march it stands in for: the same expressions summed in the same
order, so states are equal bit for bit.  Extents below, at and one above a
brick in each direction, the smallest grid, and sizes on both sides of the
switches between bricks of two planes, of four, and the march.

The per-step record is reduced by the launch of the next stage; on every route
(precision and tile) it must agree with diagnostics() of the same state.  The
sums of at most 2^18 doubles agree to 1e-13 of the sum of magnitudes.  FP32
storage forms kinetic energy and enstrophy from single-precision velocities and
their differences, whose rounding (a unit u = 2^-24 each, 18 units in a stencil
of weights 1, 8, 8, 1) is n / (2 pi) times larger against the gradient of a
wave that fills n points and enters the square twice: 2 * 18 * n / (2 pi) u <
6 n u."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


def _steps(ns, p, prec, Q, tile, steps, diag):
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, prec), dtype=torch.uint8, device="cuda")
    S = torch.as_tensor(Q, device="cuda")
    d = torch.full((steps, 8), float("nan"), dtype=torch.float64, device="cuda")
    ns.ns_set_fused_config(tile, 0)
    try:
        ns.rk3_step(p, ns.NS_ALGO_FUSED, prec, 5e-4, steps, S, work, diag_dev=d if diag else None)
        torch.cuda.synchronize()
    finally:
        ns.ns_set_fused_config(-1, 0)
    return S, d.cpu().numpy()


@pytest.mark.parametrize("n", [(5, 5, 5), (8, 5, 8), (9, 8, 5), (7, 9, 6), (16, 16, 16), (31, 33, 12), (32, 32, 32),
                               (2048, 5, 5), (5, 6, 257), (33, 40, 41), (48, 48, 48), (65, 48, 48)])
def test_automatic_fp32_shape_gives_the_marching_kernels_bits(ns, n):
    print(f"brick32 n={n}", flush=True)
    Q = synth.random_state(n[::-1], seed=n[0] + 2 * n[1])
    p = ns.make_params(n, reynolds=700.0, mach=0.25)
    want, _ = _steps(ns, p, ns.NS_FP32_STORE, Q, 0, 3, False)
    for diag in (False, True):
        got, _ = _steps(ns, p, ns.NS_FP32_STORE, Q, -1, 3, diag)
        assert torch.equal(got, want)


@pytest.mark.parametrize("n", [(16, 16, 16), (32, 32, 32), (37, 24, 19), (40, 44, 48), (80, 37, 52)])
@pytest.mark.parametrize("prec,tile", [("fp64", -1), ("fp64", 0), ("fp64", 7), ("fp64", 9), ("fp64", 10),
                                       ("fp32", -1), ("fp32", 0), ("fp32", 7), ("fp32", 8)])
def test_step_record_is_the_diagnostics_of_the_input(ns, n, prec, tile):
    print(f"record n={n} {prec} tile={tile}", flush=True)
    Q = synth.random_state(n[::-1], seed=3 * n[0] + n[2])
    p = ns.make_params(n, reynolds=700.0, mach=0.25)
    code = ns.NS_FP64 if prec == "fp64" else ns.NS_FP32_STORE
    _, d = _steps(ns, p, code, Q, tile, 1, True)
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, code), dtype=torch.uint8, device="cuda")
    ref = ns.diagnostics(p, torch.as_tensor(Q, device="cuda"), work)
    ref = np.array([ref[k] for k in ("mass", "momentum_x", "momentum_y", "momentum_z", "energy", "kinetic_energy",
                                     "enstrophy", "dissipation")])
    vol = float(np.prod([2 * np.pi / k for k in n]))
    scale = np.abs(ref)
    scale[1:4] = [vol * np.abs(Q[f]).sum() for f in (1, 2, 3)]
    tol = np.full(8, 1e-13)
    if prec == "fp32":
        tol[5:] = 6 * max(n) * 2.0 ** -24
    assert (np.abs(d[0] - ref) <= tol * scale).all(), (d[0], ref)
