"""The cubic form of the iterate (total degree 3, d = 3, 5, 10) at the edges
of its waves and step groups: path counts around a wavefront and a workgroup
and a single path (FP32 paths run whole wavefronts on the matrix cores), Euler
step counts that leave every remainder of a step group, and points at T, per
point against the FP64 oracle from an iterate with every monomial present."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu

# per-point corrections relative to 1 + |c| + standard deviation + |u|
TOL = {"fp64": 1e-8, "fp32": 2e-3}
SHAPES = [(3, 1, 1), (3, 63, 6), (3, 257, 7), (5, 64, 1), (5, 65, 2), (5, 255, 3),
          (10, 1, 2), (10, 65, 3)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("d,M,N", SHAPES)
def test_corrections_of_a_cubic_iterate(d, M, N, prec):
    cfg = problem(d=d, vol_kind="bump", vol_level=[0.15 + 0.02 * j for j in range(d)],
                  bump_a=0.25, rho=0.2, payoff="put", S0=100.0, grid="random",
                  n_t=5, n_x={3: 30, 5: 80, 10: 330}[d], eta=3, M=M, N=N, K_it=2, omega=1.0,
                  precision=prec, seed=21)
    nu = oracle.index_set(d + 1, 3)
    deg = nu.sum(axis=1)
    alpha = np.random.default_rng(9).normal(size=len(nu)) * np.array([4.0, 1.5, 0.5, 0.15])[deg]
    alpha[0] = 6.0
    y = oracle.basis_matrix(cfg) @ alpha
    print("cubic iterate d=%d M=%d N=%d %s" % (d, M, N, prec), flush=True)
    with bsde.Problem(cfg) as P:
        P.fit_values(y, 1)
        P.solve()
        c, var = P.corrections(1)
        pts = P.points()
    # points at both ends of the time axis, and some between
    idx = [0, 1, len(pts) // 2, len(pts) // 2 + 7, len(pts) - 2, len(pts) - 1]
    assert pts[idx[-1], 0] == cfg["T"]
    for i in idx:
        rc, rv = (float(v[0]) for v in oracle.corrections(cfg, alpha, 1, i, i + 1))
        scale = 1.0 + abs(rc) + np.sqrt(rv) + abs(y[i])
        assert abs(c[i] - rc) <= TOL[prec] * scale, (i, c[i], rc)
        assert abs(var[i] - rv) <= 4 * TOL[prec] * scale ** 2, (i, var[i], rv)
