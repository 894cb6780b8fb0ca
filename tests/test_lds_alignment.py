"""Arrays in LDS that are accessed two doubles at a time are declared 16-byte aligned: where the compiler places an array
of doubles is otherwise any multiple of eight."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_13490_amd", "csrc")

@pytest.mark.parametrize("function,arrays", [
    ("chain64_fwd_kernel", ["V"]), ("chain64_bwd_kernel", ["V"]), ("plan64_fwd_long", ["Vs"]), ("plan64_bwd_long", ["Bs"]),
    ("gemm64_ts_body", ["Sb", "Sf"]), ("readout64_body", ["Fs"]),
])
def test_wide_arrays(function, arrays):
    src = open(os.path.join(CSRC, "gst_kernels64.hip")).read()
    body = next(f for f in re.split(r"\n(?=(?:template|__global__|__device__))", src) if re.search(r"\b%s\(const" % function, f))
    for name in arrays:
        decl = re.search(r"__shared__ ([^;]*)\b%s\[" % name, body)
        assert decl and "__align__(16)" in decl.group(1), (function, name)
