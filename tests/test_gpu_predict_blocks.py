"""Predictions on both sides of the split of a chain of blocks over the wave's four teams (eight blocks of 32
repetitions), and ragged counts of blocks, against the oracle: the first block bit-identical, later ones within
1e-11 (probabilities)."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["1q", "2q"])
@pytest.mark.parametrize("r_max", [223, 224, 255, 256, 287, 319, 351, 1000])
def test_blocks(oracle_lib, kind, r_max):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    m = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, np.random.default_rng(r_max))
    preps, gates = [[], [0], [1, 0, 1]], list(range(int(m.K)))
    dg = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    p = api.predict(ctx, dg, preps, gates, r_max).cpu().numpy()
    want = oracle_lib.predict(m.rho, m.effects, m.gates, preps, gates, r_max)
    assert np.array_equal(p[:, :, :32], want[:, :, :32])
    assert np.abs(p - want).max() <= 1e-11


@pytest.mark.parametrize("n_prep,length,n_gates", [(1, 0, 1), (64, 8, 6), (65, 1, 6), (9, 57, 2), (8, 64, 2), (3, 2, 64), (3, 2, 65)])
def test_words_in_the_arguments(oracle_lib, n_prep, length, n_gates):
    """Preparation words and gate lists on both sides of what the kernels' arguments hold (64 words, 512 gates in
    them, 64 gates)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    rng = np.random.default_rng([n_prep, length])
    m = W.noisy_gateset("2q", W.LAMBDA, W.SIGMA, rng)
    preps = [rng.integers(0, m.K, size=length).tolist() for _ in range(n_prep)]
    gates = rng.integers(0, m.K, size=n_gates).tolist()
    dg = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    p = api.predict(ctx, dg, preps, gates, 40).cpu().numpy()
    want = oracle_lib.predict(m.rho, m.effects, m.gates, preps, gates, 40)
    assert np.array_equal(p[:, :, :32], want[:, :, :32])
    assert np.abs(p - want).max() <= 1e-11
