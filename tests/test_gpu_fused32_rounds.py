"""FP32 storage in the one-thread march: chunks of every length modulo the five
planes of a round, shorter and longer than one round, give the bits of the
automatic shape (a brick kernel at this size, which has no rounds)."""
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


@pytest.mark.parametrize("n", [(33, 9, 13), (16, 12, 6)])
def test_chunks_of_every_length(ns, n):
    Q = synth.random_state(n[::-1], seed=n[2])
    p = ns.make_params(n, mach=0.2)
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, ns.NS_FP32_STORE), dtype=torch.uint8, device="cuda")
    out = {}
    for tile, zc in [(-1, 0)] + [(t, z) for t in (0, 6) for z in range(1, n[2] + 1)]:
        print(f"rounds n={n} tile={tile} zchunk={zc}", flush=True)
        S = torch.as_tensor(Q, device="cuda")
        ns.ns_set_fused_config(tile, zc)
        try:
            ns.rk3_step(p, ns.NS_ALGO_FUSED, ns.NS_FP32_STORE, 5e-4, 2, S, work)
            torch.cuda.synchronize()
        finally:
            ns.ns_set_fused_config(-1, 0)
        out[tile, zc] = S.cpu().numpy()
        assert np.array_equal(out[tile, zc], out[-1, 0]), (tile, zc)
