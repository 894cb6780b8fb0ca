"""Predictions do not depend on r_max: those up to r are the same bits whatever follows them, on both sides of the
chain's steps (blocks of 32 repetitions, the first four one after the other, later ones 128 repetitions apart)."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["1q", "2q"])
def test_an_r_does_not_depend_on_r_max(kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    m = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, np.random.default_rng(5))
    preps, gates = [[], [0], [1, 0, 1]], list(range(int(m.K)))
    dg = api.DeviceGateSet.from_numpy(m.n_qubits, m.rho, m.effects, m.gates)
    longest = api.predict(ctx, dg, preps, gates, 1000).cpu().numpy()
    for r_max in (0, 31, 32, 127, 128, 159, 160, 191, 192, 223, 224, 255, 256, 500):
        p = api.predict(ctx, dg, preps, gates, r_max).cpu().numpy()
        assert np.array_equal(p, longest[:, :, :r_max + 1]), r_max
