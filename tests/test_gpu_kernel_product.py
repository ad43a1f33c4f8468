"""The kernel operator's product table (points that are every spatial point
at every time node) at the edges of its rule: two and sixteen time nodes,
seventeen (plain rows again), one spatial point, rows that need no padding and
rows that need three, a window that puts most pairs at the clamp; per point
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close_c, run_gpu
from workloads import problem

pytestmark = pytest.mark.gpu

# the bounds of the kernel operator's other parity cases
TOL = {"fp64": 1e-8, "fp32": 2e-3}
CASES = [(1, dict(n_t=2, n_x=9), 0.4), (1, dict(n_t=3, n_x=1), 0.5),
         (1, dict(n_t=16, n_x=5), 0.15), (1, dict(n_t=17, n_x=5), 0.15),
         (1, dict(n_t=4, n_x=12), 0.06), (2, dict(n_t=2, n_x=4), 0.4),
         (2, dict(n_t=16, n_x=3), 0.3), (2, dict(grid="random", n_t=7, n_x=11), 0.3)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d,grid,bw", CASES)
def test_product_points(d, grid, bw, prec):
    cfg = problem(d=d, vol_kind="bump", vol_level=0.2, bump_a=0.25, rho=0.0 if d == 1 else 0.3,
                  S0=100.0, eta=2, M=130, N=5, K_it=2, omega=1.0, kernel_bw=bw, precision=prec,
                  seed=8, **grid)
    print("kernel product d=%d %s bw=%g %s" % (d, grid, bw, prec), flush=True)
    ref = oracle.solve(cfg)
    got = run_gpu(cfg)
    assert_close_c(got["c"], ref["c"], TOL[prec], "c")
    assert_close_c(got["alpha"], ref["alpha"], 3 * TOL[prec], "y")
    assert np.all(np.isfinite(got["var"]))
