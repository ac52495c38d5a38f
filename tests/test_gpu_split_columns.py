"""The kernels that split a column over groups of waves (tiles 8-10) at the
edges of their tiles and of the march: extents one below, at and one above a
tile, the shortest grid, and a chunk of every length modulo the ring's five
phases, for other gas constants than the Taylor-Green vortex's.

Tolerance: the residual-level bar of the parity tests, 1e-12 of max|R| per
field on these grids (none above 68 points), where two independent correct
double evaluations differ by less than 1e-12."""
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


@pytest.mark.parametrize("n", [(5, 5, 5), (31, 7, 6), (32, 8, 8), (33, 9, 5), (68, 17, 7), (16, 5, 11)])
@pytest.mark.parametrize("gamma,mach,re", [(1.4, 0.1, 1600.0), (1.67, 0.5, 300.0)])
def test_residual_at_tile_and_chunk_edges(ns, n, gamma, mach, re):
    Q = synth.random_state(n[::-1], seed=n[0] + 3 * n[2], energy_mean=1.0 / (gamma * (gamma - 1.0) * mach ** 2))
    p = ns.make_params(n, gamma=gamma, mach=mach, reynolds=re)
    want = oracle.residual(oracle.Physics(n=n, gamma=gamma, mach=mach, reynolds=re), Q)
    scale = [np.abs(want[v]).max() for v in range(5)]
    scale[1:4] = [max(scale[1:4])] * 3
    Qd = torch.as_tensor(Q, device="cuda")
    first = None
    try:
        for tile in (8, 9, 10):
            for zc in (0, 1, 2, 3, 4, 5, 6):
                print(f"split columns n={n} tile={tile} zchunk={zc}", flush=True)
                ns.ns_set_fused_config(tile, zc)
                R = torch.empty_like(Qd)
                ns.ns_residual(p, ns.NS_ALGO_FUSED, Qd, R)
                torch.cuda.synchronize()
                got = R.cpu().numpy()
                err = max(np.abs(got[v] - want[v]).max() / scale[v] for v in range(5))
                assert err < 1e-12, (tile, zc, err)
                if first is None:
                    first = got
                assert np.array_equal(got, first), (tile, zc)
    finally:
        ns.ns_set_fused_config(-1, 0)
