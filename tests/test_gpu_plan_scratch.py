"""A plan request's scratch is held once: a batch of such requests takes theirs instead of as much again, and gives the
standalone results, before and after the requests are evaluated alone."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,capture", [("c1", False), ("c2", False), ("c2", True)])
def test_batch_uses_the_requests_scratch(kind, capture):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0, stream=torch.cuda.Stream())
    w = W.structured_workload(kind)
    m, n = w.model, 12
    reqs = [api.Request(ctx, m.n_qubits, m.K, m.M, w.seqs.offsets, w.seqs.gates, w.counts) for _ in range(n)]
    assert all(r.plan_info()["plan_used"] for r in reqs)
    gs = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    held = [r.footprint() for r in reqs]
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    batches = [api.Batch(ctx, reqs[x:], [gs] * (n - x), capture_graph=capture) for x in (0, 1)]
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken < 48 << 20, taken   # descriptors and outputs, not as much scratch again for each batch
    alone = None
    for _ in range(2):
        for b in batches:
            b.run()
            ctx.sync()
            got = [(o.clone(), g.clone()) for o, g in zip(b.obj, b.grad)]
            o, _, g = reqs[0].eval(gs)
            ctx.sync()
            alone = alone or (o, g)
            assert torch.equal(o, alone[0]) and torch.equal(g, alone[1])
            assert all(torch.equal(a, alone[0]) and torch.equal(c, alone[1]) for a, c in got)
    assert [r.footprint() for r in reqs] == held
    for b in batches:
        b.close()
    for r in reqs:
        r.close()
