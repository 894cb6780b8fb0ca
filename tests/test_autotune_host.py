"""The autotuner's candidates: different policies to the library, and for three qubits the library's own rule is the
default (it depends on the list; a fixed tile size replaces it only where it is faster)."""
from paper_2008_13490_amd import autotune


def test_three_qubit_candidates():
    cands = autotune.CANDIDATES[3]
    assert cands[0] == (0, 0)
    # a three-qubit tile takes at most 16 sequences, and the workgroups per CU do not matter
    assert len({min(t, 16) for t, _ in cands}) == len(cands)
