"""FP32 path corrections per point against the FP64 oracle, held to FP32
rounding: every form of the iterate (channels, the cubic form, the cubic form
with single-variate terms of degree 5), from an iterate with every function
present, in the narrow and the wide domain."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu

# A path's log-prices, below 8 here, are rounded twice in each of ten steps and a
# few times at tau: 24 roundings of 8 x 2^-25 come to 6e-6 if all have one sign.
# They enter payoff and iterate with the price, at most some three times the scale
# below, and the sums of a path's term add a few 2^-24 of its size
TOL = 2e-5
SETS = [(1, 4, 1.0), (2, 5, 1.0), (3, 3, 1.0), (5, 2, 1.0), (5, 3, 1.0), (10, 3, 1.0), (10, 4, 0.6),
        (10, 5, 0.5), (10, 5, 0.6), (10, 5, 0.7)]


@pytest.mark.parametrize("width", [1.0, 4.0])
@pytest.mark.parametrize("d,eta,q", SETS)
def test_corrections_to_fp32_rounding(d, eta, q, width):
    nu = oracle.index_set(d + 1, eta, q)
    cfg = problem(d=d, vol_kind="bump", vol_level=[0.15 + 0.02 * j for j in range(d)], bump_a=0.25,
                  rho=0.2 if d > 1 else 0.0, payoff="put", S0=100.0, grid="uniform", n_t=2,
                  n_x=max(60, 3 * len(nu)), eta=eta, q=q, width=width, M=65, N=10, K_it=2, omega=1.0,
                  precision="fp32", seed=37)
    size = np.array([8.0, 3.0, 1.0, 0.4, 0.2, 0.1])[nu.sum(axis=1)]
    alpha = np.random.default_rng(4).normal(size=len(nu)) * size
    y = oracle.basis_matrix(cfg) @ alpha
    print("fp32 rounding d=%d eta=%d q=%g width=%g" % (d, eta, q, width), flush=True)
    with bsde.Problem(cfg) as P:
        P.fit_values(y, 1)
        P.solve()
        c, var = P.corrections(1)
    for i in np.linspace(0, len(y) - 1, 8).astype(int):
        rc, rv = (float(v[0]) for v in oracle.corrections(cfg, alpha, 1, i, i + 1))
        scale = 1.0 + abs(rc) + np.sqrt(rv) + abs(y[i])
        assert abs(c[i] - rc) <= TOL * scale, (i, c[i], rc)
        assert abs(var[i] - rv) <= 4 * TOL * scale ** 2, (i, var[i], rv)
