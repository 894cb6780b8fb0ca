"""The order of a grouped-chain plan's levels when the list has long chains: before the long
level only what leads to it; the plan still executes to the oracle's numbers."""
import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W
from test_plan64 import TC, get_plan, plib, run_plan, small_structured  # noqa: F401


@pytest.mark.parametrize("n_fid,spec,powers", [(5, [(2, 3), (3, 2)], [1, 2, 4, 8, 16]), (6, [(2, 2)], [16, 32]),
                                               (3, [(2, 1)], [64])])
def test_short_chains_wait_for_the_long_level(oracle_lib, plib, n_fid, spec, powers):  # noqa: F811
    gs, sl = small_structured("3q", 5, n_fid, spec, powers)
    P = get_plan(plib, sl, gs.K, ratio=10.0)
    assert P["used"]
    ltp, row0, length = P["level_tile_ptr"], P["row0"], P["len"]
    longest = [length[ltp[v]:ltp[v + 1]].max() for v in range(P["n_levels"])]
    last_long = max(v for v in range(P["n_levels"]) if longest[v] >= 32)
    # rows of the tiles up to the last long level that a later tile of those levels starts from
    T = ltp[last_long + 1]
    leads = set(int(a) for t in range(T) for a in P["anchor"][t * TC:t * TC + P["cols"][t]])
    for t in range(ltp[last_long]):
        if length[t] < 32:
            for c in range(P["cols"][t]):
                assert any(int(row0[t] + s * TC + c) in leads for s in range(length[t]))
    rng = np.random.default_rng(6)
    counts = W.sample_counts(oracle_lib.probs(gs.rho, gs.effects, gs.gates, sl.offsets, sl.gates), 1000, rng)
    F, p, g = run_plan(P, gs, counts)
    F_or, p_or, g_or, _, rc = oracle_lib.loglik(gs.rho, gs.effects, gs.gates, sl.offsets, sl.gates, counts)
    assert rc == 0
    assert np.abs(p - p_or).max() <= 1e-12 * np.abs(p_or).max()
    assert abs(F - F_or) <= 1e-10 * abs(F_or)
    assert np.abs(g - g_or).max() <= 1e-10 * np.abs(g_or).max()
