"""The sparse hyperbolic sets of d = 10 (eta = 4, q = 0.6; eta = 5, q = 0.5) have
fewer live channel entries than the cubic form has products and run in the
channels: their batch kernels keep the registers of four waves a SIMD, the
denser sets' those of three (the compiler's report written by the build)."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RES = os.path.join(ROOT, "paper_1102_4666_amd", "_build", "resources.txt")


@pytest.mark.parametrize("eta,q10,vol,channels", [
    (4, 6, 0, True), (4, 6, 1, True), (5, 5, 0, True), (5, 6, 0, False), (5, 6, 1, False),
    (5, 7, 0, False), (5, 7, 1, False)])
def test_form_of_a_hyperbolic_set(eta, q10, vol, channels):
    if not os.path.exists(RES):
        pytest.skip("library not built in this tree")
    name = "batch_path_kernelILi10ELi%dEfLi%dELi%dE" % (eta, vol, q10)
    rows = [ln.split() for ln in open(RES) if name in ln]
    assert len(rows) == 1
    assert (int(rows[0][1].split("=")[1]) <= 128) == channels, rows[0]
