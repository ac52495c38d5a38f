"""Grids on which two-plane bricks would outnumber the blocks that the workspace
has diagnostic partials for (an odd number of planes, extents just above a
multiple of the tile), and their neighbours on which they do not: with per-step
diagnostics under the automatic shape the state keeps the bits of the march, and
each record agrees with the march's (another order of at most 2^15 terms: 1e-13
of the sum of magnitudes)."""
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


@pytest.mark.parametrize("n", [(48, 56, 5), (47, 53, 5), (16, 165, 5), (16, 25, 5), (48, 56, 6), (33, 34, 7)])
@pytest.mark.parametrize("prec,tile", [("fp64", 9), ("fp32", 0)])
def test_bricks_fit_the_partials(ns, n, prec, tile):
    print(f"partials n={n} {prec}", flush=True)
    code = ns.NS_FP64 if prec == "fp64" else ns.NS_FP32_STORE
    p = ns.make_params(n, reynolds=700.0, mach=0.25)
    Q = synth.random_state(n[::-1], seed=n[0] + n[1])
    out = {}
    for t in (-1, tile):
        work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, code), dtype=torch.uint8, device="cuda")
        S = torch.as_tensor(Q, device="cuda")
        d = torch.zeros((3, 8), dtype=torch.float64, device="cuda")
        ns.ns_set_fused_config(t, 0)
        try:
            ns.rk3_step(p, ns.NS_ALGO_FUSED, code, 2e-4, 3, S, work, diag_dev=d)
            torch.cuda.synchronize()
        finally:
            ns.ns_set_fused_config(-1, 0)
        out[t] = (S, d.cpu().numpy())
    assert torch.equal(out[-1][0], out[tile][0])
    vol = float(np.prod([2 * np.pi / k for k in n]))
    scale = np.abs(out[tile][1]).max(axis=0)
    scale[1:4] = [vol * np.abs(Q[f]).sum() for f in (1, 2, 3)]
    assert (np.abs(out[-1][1] - out[tile][1]) <= 1e-13 * scale).all()
