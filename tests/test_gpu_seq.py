"""The 16-lane-team kernels of lists without shared prefixes, against the oracle.

Word lengths at the edges of a chunk of 16 steps, a segment of 8 and the half
segments whose (adjoint, state) pairs are added together; four words of one
length (no step selects a state) and of four; groups of fewer than four words;
gate counts on both sides of the accumulators of six gates; lists on both sides
of the launch that fills more than two workgroups per CU.  Probabilities must be
bit-identical, the objective within 1e-10 relative, the gradient within 1e-10
of its largest entry.
"""
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


def _model(kind, K, rng):
    m = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, rng)
    g = np.concatenate([m.gates, W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, rng).gates])
    m.gates = np.ascontiguousarray(np.concatenate([g, g])[:K])
    return m


@pytest.mark.parametrize("kind,K,S,lengths", [
    ("2q", 6, 5, (16,)), ("2q", 6, 8, (8, 24)), ("2q", 1, 6, (4, 5, 12, 0)), ("2q", 6, 13, (33, 31, 1, 40)),
    ("2q", 7, 9, (17,)), ("2q", 8, 64, (7, 9, 23, 32)), ("2q", 6, 8208, (9,)), ("2q", 6, 8191, (8, 6, 7, 2)),
    ("2q", 8, 8300, (5, 3)), ("1q", 8, 21, (16, 15, 8)), ("1q", 3, 18, (16, 5, 8)),
])
def test_team_kernels(oracle_lib, gpu, kind, K, S, lengths):
    import torch
    api, ctx = gpu
    rng = np.random.default_rng([K, S, len(lengths)])
    m = _model(kind, K, rng)
    sl = W.from_words([rng.integers(0, K, size=lengths[s % len(lengths)]).tolist() for s in range(S)])
    counts = rng.integers(0, 40, size=(S, m.M)).astype(np.int32)
    counts[oracle_lib.probs(m.rho, m.effects, m.gates, sl.offsets, sl.gates) <= 0] = 0
    F, p_or, g_or, _, rc = oracle_lib.loglik(m.rho, m.effects, m.gates, sl.offsets, sl.gates, counts)
    assert rc == 0
    gs = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    req = api.Request(ctx, m.n_qubits, K, m.M, sl.offsets, sl.gates, counts)
    seqs = api.DeviceSeqs.from_numpy(sl.offsets, sl.gates)
    calls = [("plain", lambda: ctx.loglik(gs, seqs, torch.as_tensor(counts, device="cuda"), want_probs=True))]
    if not req.plan_info()["plan_used"]:   # one gate: the words share their prefixes
        calls.append(("request", lambda: req.eval(gs, want_probs=True)))
    for label, call in calls:
        obj, p, g = call()
        ctx.sync()
        assert np.array_equal(p.cpu().numpy(), p_or), label
        assert abs(float(obj.cpu()[0]) - F) <= 1e-10 * abs(F), label
        assert np.abs(g.cpu().numpy() - g_or).max() <= 1e-10 * np.abs(g_or).max(), label
    req.close()


@pytest.mark.parametrize("K,S,lengths", [
    (1, 63, (9, 3)), (2, 64, (16,)), (3, 65, (8, 7, 0, 1)), (4, 130, (17, 24, 16, 40)), (3, 200, (33,)),
    (2, 1, (15,)), (4, 256, (8,)), (4, 1000, (31, 32, 33)),
])
def test_lane_kernel(oracle_lib, gpu, K, S, lengths):
    """One chain per lane: tiles of 64 words, full and not; segments of 8 that all words of a tile run through and not."""
    api, ctx = gpu
    rng = np.random.default_rng([K, S, len(lengths)])
    m = _model("1q", K, rng)
    sl = W.from_words([rng.integers(0, K, size=lengths[s % len(lengths)]).tolist() for s in range(S)])
    counts = rng.integers(0, 40, size=(S, m.M)).astype(np.int32)
    counts[oracle_lib.probs(m.rho, m.effects, m.gates, sl.offsets, sl.gates) <= 0] = 0
    F, p_or, g_or, _, rc = oracle_lib.loglik(m.rho, m.effects, m.gates, sl.offsets, sl.gates, counts)
    assert rc == 0
    gs = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    req = api.Request(ctx, m.n_qubits, K, m.M, sl.offsets, sl.gates, counts)
    bt = api.Batch(ctx, [req], [gs], want_probs=True, want_grad=True)

    def batch():
        bt.run()
        return bt.obj[0], bt.probs[0], bt.grad[0]
    for label, call in (("batch", batch), ("request", lambda: req.eval(gs, want_probs=True))):
        obj, p, g = call()
        ctx.sync()
        assert np.array_equal(p.cpu().numpy(), p_or), label
        assert abs(float(obj.cpu()[0]) - F) <= 1e-10 * abs(F), label
        assert np.abs(g.cpu().numpy() - g_or).max() <= 1e-10 * np.abs(g_or).max(), label
    bt.close()
    req.close()
