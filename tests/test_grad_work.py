"""The gradient's work of a sharing plan (records outside germ-power jumps, groups of sixteen jumps): unrolled
as the kernel runs it, it is every (gate, adjoint row, state row) of the plan once, and every tile has one writer."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2008_13490_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_13490_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("grad") / "libgradprobe.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-I", CSRC, os.path.join(ROOT, "tests", "grad_work_probe.cpp"),
                    os.path.join(CSRC, "gst_plan.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    P = ctypes.c_void_p
    lib.grad_work.argtypes = [P, P, ctypes.c_int64, ctypes.c_int, P]
    lib.grad_work.restype = ctypes.c_int64
    lib.grad_work_copy.argtypes = [P, P]
    return lib


@pytest.mark.parametrize("kind,n_fid,germs,powers", [
    ("1q", 6, [(0,), (0, 1), (0, 0, 1), (0, 1, 2)], [1, 2, 4, 8, 16, 32, 64, 100]),
    ("2q", 7, [(0,), (3,), (0, 3), (0, 1, 3), (0, 3, 1, 3), (4, 4, 0, 4)], [1, 5, 16, 63, 128, 256]),
    ("2q", 17, [(2, 5)], [300]), ("2q", 5, [(0, 1)], [1, 2]),
])
def test_every_step_once(lib, kind, n_fid, germs, powers):
    K = W.noisy_gateset(kind, W.LAMBDA, W.SIGMA, np.random.default_rng(1)).K
    fids = W.shortlex_words((0, 1), n_fid)
    sl = W.structured_list(fids, fids, germs, powers)
    off, g = np.ascontiguousarray(sl.offsets, np.int64), np.ascontiguousarray(sl.gates, np.uint8)
    info = np.zeros(3, np.int64)
    n = lib.grad_work(off.ctypes.data, g.ctypes.data, sl.S, int(K), info.ctypes.data)
    assert n > 0 and info[0] == 0 and info[2] == n
    assert info[1] > 0 or max(powers) < 5
    plan, work = np.zeros((n, 3), np.int64), np.zeros((n, 3), np.int64)
    lib.grad_work_copy(plan.ctypes.data, work.ctypes.data)
    assert np.array_equal(plan[np.lexsort(plan.T)], work[np.lexsort(work.T)])
