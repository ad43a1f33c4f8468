"""The kernel operator's path kernels for plain rows (uniform points, more time
nodes than a product table holds) keep the registers of their own loop, apart
from the product form's: 512 vector registers a SIMD lane give the waves named
here (the compiler's report written by the build)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RES = os.path.join(ROOT, "paper_1102_4666_amd", "_build", "resources.txt")
# kernel-name pattern (d, precision, operator) -> most registers
MOST = {"path_kernelILi1ELi1Ef%sELi10ELi1E": 64,   # eight waves
        "path_kernelILi1ELi1Ed%sELi10ELi1E": 128,  # four
        "path_kernelILi2ELi1Ef%sELi10ELi1E": 128,  # four
        "path_kernelILi2ELi1Ed%sELi10ELi1E": 168}  # three


@pytest.mark.parametrize("vol", ["Li0", "Li1"])
@pytest.mark.parametrize("kernel", sorted(MOST))
def test_plain_rows_keep_their_waves(kernel, vol):
    if not os.path.exists(RES):
        pytest.skip("library not built in this tree")
    rows = [ln.split() for ln in open(RES) if kernel % vol in ln]
    assert len(rows) == 1
    assert int(rows[0][1].split("=")[1]) <= MOST[kernel], rows[0]
