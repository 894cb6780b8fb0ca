"""Memory of three-qubit lists without shared prefixes: a recorded state is 512 bytes, one per step, however few chains the
tiles and entries of the schedule hold."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,longest", [(1, 500), (8, 500), (200, 300), (512, 300), (700, 200), (1000, 128), (3000, 64)])
def test_bytes_per_step(S, longest):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    rng = np.random.default_rng([S, longest])
    m = W.noisy_gateset("3q", W.LAMBDA, W.SIGMA, rng)
    sl = W.random_list(S, m.K, 1, longest, rng)
    counts = rng.integers(0, 50, size=(S, m.M)).astype(np.int32)
    req = api.Request(ctx, 3, m.K, m.M, sl.offsets, sl.gates, counts)
    assert req.plan_info()["plan_used"] == 0
    steps = int(sl.offsets[-1])
    # a state, two schedule entries and the index of a step; per sequence its final state, its share of the readout's
    # partial rows (4.6 KB for 16) and its inputs; the gradient of each of at most 256 workgroups, and its row
    bound = steps * (512 + 8 + 1) + S * (512 + 1200) + min(S, 256) * (m.K * 32768 + 5000) + (1 << 17)
    assert req.footprint() <= bound, (req.footprint(), bound)
    req.close()
