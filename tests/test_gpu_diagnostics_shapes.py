"""Standalone diagnostics on both of their kernels: grids just below and just
above the switch to the marching kernel (2^19 points), ragged in every
direction, shorter than a tile, and of few or many planes.

Tolerance: both sides form the same stencils in double and sum at most 6e5
terms in blocks, so sums of positive terms agree to far better than 1e-12
relative; a momentum total is compared relative to the sum of |m|."""
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


@pytest.mark.parametrize("n", [(5, 5, 5), (33, 9, 6), (64, 64, 127), (128, 64, 64), (81, 83, 79),
                               (33, 9, 1999), (2047, 53, 5), (7, 2041, 38)])
def test_diagnostics_at_both_kernels_edges(ns, n):
    print(f"diagnostics n={n}", flush=True)
    Q = synth.random_state(n[::-1], seed=n[0] + n[2])
    p = ns.make_params(n)
    Qd = torch.as_tensor(Q, device="cuda")
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, ns.NS_FP64), dtype=torch.uint8, device="cuda")
    got = ns.diagnostics(p, Qd, work)
    want = oracle.diagnostics(oracle.Physics(n=n), Q)
    assert got["status"] == ns.NS_OK
    vol = float(np.prod([2 * np.pi / k for k in n]))
    for name in oracle.DIAG_NAMES:
        if name.startswith("momentum"):
            scale = vol * np.abs(Q[1 + "xyz".index(name[-1])]).sum()
        else:
            scale = abs(want[name])
        assert abs(got[name] - want[name]) < 1e-12 * scale, (name, got[name], want[name])
    again = ns.diagnostics(p, Qd, work)
    assert again == got
