"""The gradient of steps inside germ-power jumps: groups of up to sixteen jumps of one pattern and length, against
the oracle.  Patterns of one to four gates (also with a gate twice), jumps of 2 to 64 steps, groups partly filled."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    return api, api.Context(0)


@pytest.mark.parametrize("kind,n_fid,germs,powers", [
    ("1q", 6, [(0,), (0, 1), (0, 0, 1), (0, 1, 2, 1)], [1, 2, 4, 8, 16, 32, 64, 100]),
    ("2q", 7, [(0,), (3,), (0, 3), (0, 1, 3), (0, 3, 1, 3)], [1, 5, 16, 63, 128]),
    ("2q", 17, [(2, 5)], [90]), ("2q", 4, [(4, 4, 1)], [31, 47]),
])
@pytest.mark.parametrize("reps", [0, 2, 8, 16])
def test_jump_gradient(oracle_lib, gpu, kind, n_fid, germs, powers, reps):
    import torch
    api, ctx = gpu
    api.set_plan_jump(ctx, reps)
    try:
        rng = np.random.default_rng(n_fid)
        m = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, rng)
        fids = W.shortlex_words((0, 1), n_fid)
        sl = W.structured_list(fids, fids, germs, powers)
        counts = rng.integers(0, 40, size=(sl.S, m.M)).astype(np.int32)
        counts[oracle_lib.probs(m.rho, m.effects, m.gates, sl.offsets, sl.gates) <= 1e-9] = 0
        F, _, g_or, _, rc = oracle_lib.loglik(m.rho, m.effects, m.gates, sl.offsets, sl.gates, counts)
        assert rc == 0
        req, req2 = (api.Request(ctx, m.n_qubits, m.K, m.M, sl.offsets, sl.gates, counts) for _ in range(2))
    finally:
        api.set_plan_jump(ctx, 8)
    gs = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    bt = api.Batch(ctx, [req, req2], [gs, gs])
    obj, _, g = req.eval(gs)
    bt.run()
    ctx.sync()
    for o, h in ((obj, g), (bt.obj[0], bt.grad[0]), (bt.obj[1], bt.grad[1])):
        assert abs(float(o.cpu()[0]) - F) <= 1e-10 * abs(F)
        assert np.abs(h.cpu().numpy() - g_or).max() <= 1e-10 * np.abs(g_or).max()
    w = rng.standard_normal((sl.S, m.M))
    v = req.vjp(gs, torch.as_tensor(w, device="cuda"))
    ctx.sync()
    v_or = oracle_lib.vjp(m.rho, m.effects, m.gates, sl.offsets, sl.gates, w)
    assert np.abs(v.cpu().numpy() - v_or).max() <= 1e-10 * np.abs(v_or).max()
    bt.close()
    req.close()
    req2.close()
