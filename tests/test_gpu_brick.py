"""The brick kernel of small FP64 grids (automatic launch shape) against the
marching kernel it stands in for, bit for bit, and the oracle: extents below,
at and one above a brick in each direction, the smallest grid, and sizes on
both sides of the switches between brick, 16x8 and 32x8 tiles.  States and
residuals are the same expressions in the same order, so equality is exact;
diagnostics sum in another order (at most 2^18 terms: 1e-13 of the sum of
magnitudes)."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


@pytest.mark.parametrize("n", [(5, 5, 5), (8, 5, 8), (9, 8, 5), (7, 9, 6), (16, 16, 16), (31, 33, 12), (32, 32, 32),
                               (2048, 5, 5), (5, 6, 257), (33, 32, 32), (48, 48, 48), (101, 37, 23)])
def test_automatic_shape_gives_the_marching_kernels_bits(ns, n):
    print(f"brick n={n}", flush=True)
    re, mach, dt, steps = 700.0, 0.25, 5e-4, 3
    Q = synth.random_state(n[::-1], seed=n[0] + 2 * n[1])
    p = ns.make_params(n, reynolds=re, mach=mach)
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, ns.NS_FP64), dtype=torch.uint8, device="cuda")
    out = {}
    for tile in (-1, 9):
        ns.ns_set_fused_config(tile, 0)
        try:
            S = torch.as_tensor(Q, device="cuda")
            R = torch.empty_like(S)
            ns.ns_residual(p, ns.NS_ALGO_FUSED, S, R)
            P = S.clone()
            d = torch.zeros((steps, 8), dtype=torch.float64, device="cuda")
            ns.rk3_step(p, ns.NS_ALGO_FUSED, ns.NS_FP64, dt, steps, S, work, diag_dev=d)
            ns.rk3_step(p, ns.NS_ALGO_FUSED, ns.NS_FP64, dt, steps, P, work)
            torch.cuda.synchronize()
        finally:
            ns.ns_set_fused_config(-1, 0)
        assert torch.equal(S, P)          # diagnostics do not touch the state
        out[tile] = (R.cpu().numpy(), S.cpu().numpy(), d.cpu().numpy())
    assert np.array_equal(out[-1][0], out[9][0])
    assert np.array_equal(out[-1][1], out[9][1])
    vol = float(np.prod([2 * np.pi / k for k in n]))
    mag = np.array([vol * np.abs(Q[f]).sum() for f in range(5)])
    for k in range(8):
        scale = 2 * mag[k] if k < 5 else np.abs(out[9][2][:, k]).max()
        assert np.abs(out[-1][2][:, k] - out[9][2][:, k]).max() <= 1e-13 * scale, k
    want = oracle.rk3(oracle.Physics(n=n, reynolds=re, mach=mach), Q, dt, steps)
    sc = [np.abs(want[v]).max() for v in range(5)]
    sc[1:4] = [max(sc[1:4])] * 3
    assert max(np.abs(out[-1][1][v] - want[v]).max() / sc[v] for v in range(5)) < 1e-12
