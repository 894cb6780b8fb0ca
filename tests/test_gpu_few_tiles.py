"""The team kernel's two variants (rows loaded ahead or not) on both sides of the switch, three tiles of sixteen words per
CU, against the oracle: probabilities bit-identical, objective and gradient within 1e-10 relative."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more", [0, 1])
def test_both_sides(oracle_lib, more):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    S = 3 * torch.cuda.get_device_properties(0).multi_processor_count * 16 + more
    rng = np.random.default_rng(S)
    m = W.noisy_gateset("2q", W.LAMBDA, W.SIGMA, rng)
    sl = W.random_list(S, m.K, 1, 12, rng)
    counts = rng.integers(0, 50, size=(S, m.M)).astype(np.int32)
    counts[oracle_lib.probs(m.rho, m.effects, m.gates, sl.offsets, sl.gates) <= 0] = 0
    F, p_or, g_or, _, rc = oracle_lib.loglik(m.rho, m.effects, m.gates, sl.offsets, sl.gates, counts)
    assert rc == 0
    gs = api.DeviceGateSet.from_numpy(2, m.rho, m.effects, m.gates)
    req = api.Request(ctx, 2, m.K, m.M, sl.offsets, sl.gates, counts)
    assert req.plan_info()["plan_used"] == 0
    obj, p, g = req.eval(gs, want_probs=True)
    ctx.sync()
    assert np.array_equal(p.cpu().numpy(), p_or)
    assert abs(float(obj.cpu()[0]) - F) <= 1e-10 * abs(F)
    assert np.abs(g.cpu().numpy() - g_or).max() <= 1e-10 * np.abs(g_or).max()
    req.close()
