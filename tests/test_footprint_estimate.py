"""What admission counts with: the estimate of a request's bytes before it is created covers what it then holds, for lists
without shared prefixes (fewer three-qubit words than workgroups, more two-qubit words than tiles of sixteen to a round)."""
import numpy as np
import pytest

from paper_2008_13490_amd import serving as SV
from paper_2008_13490_amd import workloads as W

LISTS = [("1q", 1, 5), ("1q", 5000, 64), ("2q", 1, 1), ("2q", 3001, 100), ("2q", 30000, 16), ("2q", 65536, 4),
         ("2q", 66000, 4), ("2q", 150000, 4), ("3q", 1, 500), ("3q", 100, 300), ("3q", 512, 200), ("3q", 513, 100),
         ("3q", 4000, 64), ("3q", 20000, 16)]


@pytest.mark.parametrize("S,tiles", [(16, 1), (17, 2), (16385, 1025), (30000, 1875), (65536, 4096), (65537, 2049)])
def test_two_qubit_tiles(S, tiles):
    """A row of partial sums per tile: sixteen words up to 65,536 of them, then as many more as keep the rows in bounds."""
    row = 8 * (1 + 16 + 4 * 16 + 6 * 256)
    b = SV.footprint_estimate(2, 6, 4, S, 10 * S)
    rest = 16 * (S + 1) + 10 * S + 16 * S
    assert tiles * row + rest <= b <= tiles * (row + 64) + rest + 16384


@pytest.mark.parametrize("S,L", [(1, 1000), (512, 1000), (2000, 100), (100000, 20)])
def test_three_qubit_states(S, L):
    """A recorded state and a final state are 512 bytes."""
    assert SV.footprint_estimate(3, 5, 8, S, S * L) >= 512 * S * (L + 1)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,S,longest", LISTS)
def test_estimate_covers_the_request(kind, S, longest):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2008_13490_amd import api
    ctx = api.Context(0)
    rng = np.random.default_rng([S, longest])
    m = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, rng)
    sl = W.random_list(S, m.K, 1, longest, rng)
    counts = rng.integers(0, 50, size=(S, m.M)).astype(np.int32)
    for tuned in (0, 16):
        api.tune_set(ctx, m.n_qubits, tuned, 0)
        req = api.Request(ctx, m.n_qubits, m.K, m.M, sl.offsets, sl.gates, counts)
        if req.plan_info()["plan_used"] or req.plan_info()["grouped"]:
            pytest.skip("a list with a sharing plan")
        est = SV.footprint_estimate(m.n_qubits, m.K, m.M, S, int(sl.offsets[-1]), ctx)
        assert req.footprint() <= est <= 2 * req.footprint() + (1 << 16)
        req.close()
