"""The FP64 d = 10 path kernels keep next to nothing in scratch memory across
their path loops (the compiler's report written by the build): what is kept there
is read back on every path, and with few Euler steps a path that is the launch."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RES = os.path.join(ROOT, "paper_1102_4666_amd", "_build", "resources.txt")


@pytest.mark.parametrize("eta,most", [(2, 140), (3, 24)])
def test_scratch_of_the_d10_fp64_kernels(eta, most):
    if not os.path.exists(RES):
        pytest.skip("library not built in this tree")
    rows = [ln.split() for ln in open(RES) if "path_kernelILi10ELi%dEd" % eta in ln]
    assert len(rows) == 4
    for name, vgprs, scratch in rows:
        assert int(scratch.split("=")[1]) <= most, (name, scratch)
