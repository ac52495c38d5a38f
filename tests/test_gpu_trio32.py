"""The three-group FP32-storage kernel (tiles 8-10) against the one-thread kernel
(tile 0): the same expressions summed in the same order, so states are equal
bit for bit, whatever the z-chunk.  Extents below, at and one above a tile, odd
and even nx (single and paired loads), chunks of every length modulo the ring's
five phases, and the automatic shape on both sides of its switches.  The
direction-grouped order stays accepted under the automatic shape, which then
takes a one-thread tile."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


def _steps(ns, n, Q, tile, zchunk, steps=2, order=0):
    p = ns.make_params(n, reynolds=700.0, mach=0.25)
    work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, ns.NS_FP32_STORE), dtype=torch.uint8, device="cuda")
    S = torch.as_tensor(Q, device="cuda")
    ns.ns_set_fused_config(tile, zchunk)
    ns.ns_set_fused_order(order)
    try:
        ns.rk3_step(p, ns.NS_ALGO_FUSED, ns.NS_FP32_STORE, 5e-4, steps, S, work)
        torch.cuda.synchronize()
    finally:
        ns.ns_set_fused_config(-1, 0)
        ns.ns_set_fused_order(0)
    return S


@pytest.mark.parametrize("n", [(5, 5, 5), (31, 7, 6), (32, 8, 8), (33, 9, 7), (68, 17, 11), (16, 5, 13)])
def test_three_groups_give_the_one_thread_bits(ns, n):
    print(f"trio32 n={n}", flush=True)
    Q = synth.random_state(n[::-1], seed=n[0] + 3 * n[2])
    want = _steps(ns, n, Q, 0, 0)
    for tile in (8, 9, 10):
        for zc in (0, 1, 2, 3, 4, 5, 6):
            assert torch.equal(_steps(ns, n, Q, tile, zc), want), (tile, zc)


@pytest.mark.parametrize("n", [(56, 56, 56), (64, 64, 64), (101, 77, 53), (112, 112, 112), (161, 97, 119)])
def test_automatic_shape_and_order(ns, n):
    print(f"trio32 automatic n={n}", flush=True)
    Q = synth.random_state(n[::-1], seed=n[0])
    for order in (0, 1):
        assert torch.equal(_steps(ns, n, Q, -1, 0, order=order), _steps(ns, n, Q, 0, 0, order=order)), order
