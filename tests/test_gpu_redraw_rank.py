"""A redrawn basis that fails its rank test: the solve reports it, and the
problem is left with the points and the pseudo-inverse of the last iteration
that ran, the ones get_points returns and fit_values fits at; with one and with
two sets of buffers, the failing draw the first, a middle and the last one."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu

# (seed, first draw that fails): nine spatial points for degree 8, so that two of
# them close together make the basis singular.  Smallest pivot over the largest
# column: below 5e-10 in the failing draw, so that one of the two rank tests
# refuses it whatever the rounding of the Gram matrix, and above 1e-4 in those
# before it (the tests' limits are 1e-7 and 1e-3)
DRAWS = [(9910, 1), (14339, 2), (33064, 3), (32542, 4)]


# (2e7 asset steps an iteration and more take two sets of buffers)
@pytest.mark.parametrize("M,N", [(50, 4), (22000, 20)])
@pytest.mark.parametrize("seed,bad", DRAWS)
def test_rank_deficient_draw(seed, bad, M, N):
    cfg = problem(d=1, S0=100.0, vol_level=0.2, grid="random", redraw=1, n_t=9, n_x=9, eta=8,
                  M=M, N=N, K_it=5, omega=1.0, seed=seed)
    print("rank-deficient draw %d M=%d" % (bad, M), flush=True)
    pts = oracle.points(cfg, bad - 1)
    y = pts[:, 0] + 0.5 * pts[:, 1] ** 2
    with bsde.Problem(cfg) as P:
        for _ in range(2):
            with pytest.raises(bsde.BsdeError) as e:
                P.solve()
            assert e.value.status == 3
            with pytest.raises(bsde.BsdeError) as e:
                P.corrections(0)          # no iteration counts as done
            assert e.value.status == 5
            assert np.abs(P.points() - pts).max() <= 1e-12
            P.fit_values(y, 0)
            price, _ = P.price_delta(pts[:, 0], np.exp(pts[:, 1:]))
            # kappa is at most 1e5 and y below 16
            assert np.abs(price - y).max() <= 1e-8
