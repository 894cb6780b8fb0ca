"""The grouped schedules' builder, the program of its wave run lane by lane on the CPU: no access outside the staged
window of 512 steps, and the schedule applies every word's gates once, in order, with the chain and the parity of the
step in each column and different chains in the two entries of a round."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_13490_amd", "csrc")
NONE = 16


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("sched") / "libschedprobe.so")
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O2", "-fPIC", "-shared", "-I", CSRC,
                    os.path.join(ROOT, "tests", "sched_probe.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    P = ctypes.c_void_p
    lib.sched_cpu.argtypes = [P, P, P, ctypes.c_int64, ctypes.c_int, ctypes.c_int, P, P, P]
    lib.sched_cpu.restype = lib.sched_at.restype = ctypes.c_int64
    lib.sched_at.argtypes = [ctypes.c_int64, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("K,tile,lengths", [
    (5, 16, [513, 3, 0]), (5, 1, [520, 0, 7, 2]), (5, 16, [35]), (2, 3, [530, 513, 512, 511, 1, 0, 0]), (1, 16, [9] * 17),
    (5, 16, list(range(20, 41))), (4, 5, [24, 23, 1, 1, 0, 520, 40]),
])
def test_schedule(lib, K, tile, lengths):
    rng = np.random.default_rng([K, tile, len(lengths)])
    words = [rng.integers(0, K, size=n).astype(np.uint8) for n in lengths]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    gates = np.concatenate(words + [np.zeros(1, np.uint8)])
    S = len(lengths)
    order = np.argsort(-np.asarray(lengths), kind="stable").astype(np.int64)
    n_tiles = (S + tile - 1) // tile
    rec = np.array([sum(lengths[q] for q in order[:t * tile]) for t in range(n_tiles + 1)], np.int64)
    at = [lib.sched_at(int(rec[t]), t) for t in range(n_tiles + 1)]
    count = np.full(n_tiles, -1, np.int32)
    entries = np.full(at[-1] + 1, 0xffffffff, np.uint32)
    args = [x.ctypes.data for x in (off, gates, order)] + [S, K, tile]
    assert lib.sched_cpu(*args, rec.ctypes.data, count.ctypes.data, entries.ctypes.data) == 0
    assert entries[-1] == 0xffffffff
    for t in range(n_tiles):
        chains = order[t * tile:(t + 1) * tile]
        pos = [0] * len(chains)
        es = entries[at[t]:at[t] + count[t]]
        assert len(es) % 4 == 0 and at[t] + len(es) <= at[t + 1]
        assert (entries[at[t] + len(es):at[t + 1]] == 0xffffffff).all()
        for x in range(0, len(es), 2):
            seen = set()
            for e in es[x:x + 2]:
                fields = [int(e) >> (6 * r) & 63 for r in range(4)]
                live = [f for f in fields if f >> 1 != NONE]
                assert fields == live + [2 * NONE] * (4 - len(live))   # columns are filled from the first
                for f in live:
                    c = f >> 1
                    assert c not in seen and (f & 1) == (pos[c] & 1)
                    assert words[chains[c]][pos[c]] == int(e) >> 24
                    seen.add(c)
            for c in seen:
                pos[c] += 1
        assert pos == [len(words[q]) for q in chains]
