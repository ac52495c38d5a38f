"""A batch balances its members over its streams anew in every call: members
that are added, run out of steps or are removed between calls move the others
to different streams.  Every member still ends with the bits of its own
rk3_step, eagerly and through replayed graphs."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ns():
    import paper_1709_09713_amd as ns
    assert torch.cuda.is_available()
    return ns


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nstreams", [1, 2, 3, 8])
@pytest.mark.parametrize("graphs", [False, True])
def test_members_keep_their_bits_when_streams_change(ns, precision, nstreams, graphs):
    print(f"balance {precision} streams={nstreams} graphs={graphs}", flush=True)
    # (extent, steps, the call before which it is added)
    plan = [(16, 9, 0), (40, 26, 0), (24, 17, 0), (56, 26, 0), (20, 26, 0), (48, 17, 1), (32, 8, 1), (64, 9, 2)]
    calls = (9, 8, 9)
    prec = ns.NS_FP32_STORE if precision == "fp32" else ns.NS_FP64
    b = ns.Batch(len(plan), precision, nstreams=nstreams, graphs=graphs)
    states = {}
    for call, k in enumerate(calls):
        for i, (n, steps, when) in enumerate(plan):
            if when == call:
                Q = torch.as_tensor(synth.random_state((n,) * 3, seed=n), device="cuda")
                states[i] = Q
                b.add(n, reynolds=700.0, mach=0.25, dt=2e-4, steps=steps, state=Q, init_tgv=False)
        b.step(k)
    torch.cuda.synchronize()
    for i, (n, steps, when) in enumerate(plan):
        p = ns.make_params((n,) * 3, reynolds=700.0, mach=0.25)
        S = torch.as_tensor(synth.random_state((n,) * 3, seed=n), device="cuda")
        work = torch.empty(ns.ns_workspace_bytes(p, ns.NS_ALGO_FUSED, prec), dtype=torch.uint8, device="cuda")
        ns.rk3_step(p, ns.NS_ALGO_FUSED, prec, 2e-4, min(steps, sum(calls[when:])), S, work)
        torch.cuda.synchronize()
        assert torch.equal(states[i], S), (i, n)
