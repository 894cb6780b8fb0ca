"""Probabilities of a three-qubit list allocate nothing: a context's first call can be recorded into a graph (as it could
before the grouped schedules), and replays give the eager call's bits."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [3, 700])
def test_first_probabilities_under_capture(oracle_lib, S):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    stream = torch.cuda.Stream()
    ctx = api.Context(0, stream=stream)
    rng = np.random.default_rng(S)
    m = W.noisy_gateset("3q", W.LAMBDA, W.SIGMA, rng)
    sl = W.random_list(S, m.K, 1, 40, rng)
    req = api.Request(ctx, 3, m.K, m.M, sl.offsets, sl.gates)
    assert req.plan_info()["plan_used"] == 0
    gs = api.DeviceGateSet.from_numpy(3, m.rho, m.effects, m.gates)
    out = torch.zeros((S, m.M), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        req.probs(gs, out=out)
    want = oracle_lib.probs(m.rho, m.effects, m.gates, sl.offsets, sl.gates)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
        eager = req.probs(gs)
        ctx.sync()
        assert np.array_equal(eager.cpu().numpy(), want)
    req.close()
