"""Grids of more four-plane bricks than compute units, up to and just above as
many as the device holds at once: the automatic shape keeps the march's bits,
with diagnostics and without."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


@pytest.mark.parametrize("n", [(36, 36, 36), (40, 40, 40), (41, 40, 40), (39, 37, 41), (64, 40, 28), (80, 40, 16)])
@pytest.mark.parametrize("prec,tile", [("fp64", 9), ("fp32", 0)])
def test_bricks_above_one_per_unit(ns, n, prec, tile):
    print(f"limits n={n} {prec}", flush=True)
    code = ns.NS_FP64 if prec == "fp64" else ns.NS_FP32_STORE
    p = ns.make_params(n, reynolds=700.0, mach=0.25)
    Q = torch.as_tensor(synth.random_state(n[::-1], seed=sum(n)), device="cuda")
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, code), dtype=torch.uint8, device="cuda")
    out = []
    for t, diag in ((tile, False), (-1, False), (-1, True)):
        S, d = Q.clone(), torch.zeros((2, 8), dtype=torch.float64, device="cuda")
        ns.ns_set_fused_config(t, 0)
        try:
            ns.rk3_step(p, ns.NS_ALGO_FUSED, code, 2e-4, 2, S, work, diag_dev=d if diag else None)
            torch.cuda.synchronize()
        finally:
            ns.ns_set_fused_config(-1, 0)
        out.append(S)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
