"""Redrawn points whose set-up runs beside the iteration before it: the same
numbers as with one iteration a solve, where nothing can run ahead, and the
problem left with the last iteration's points and pseudo-inverse, whichever of
the two sets of buffers they were formed in."""
import numpy as np
import pytest

import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu


# (more than 2e7 asset steps an iteration; the last but one more than 1e9)
@pytest.mark.parametrize("d,n,eta,q,M,N,prec", [
    (3, 400, 2, 1.0, 9000, 4, "fp64"), (5, 600, 3, 1.0, 3000, 4, "fp32"),
    (5, 600, 3, 0.8, 3000, 4, "fp64"), (10, 900, 5, 0.6, 1000, 3, "fp32"),
    (5, 1000, 3, 1.0, 30000, 10, "fp32"), (2, 90, 3, 1.0, 200, 3, "fp64")])
@pytest.mark.parametrize("K", [3, 4])
def test_set_up_ahead_gives_the_same_iterations(d, n, eta, q, M, N, prec, K):
    def config(k_it):
        return problem(d=d, vol_kind="const" if d == 10 else "bump", vol_level=0.2,
                       bump_a=0.0 if d == 10 else 0.25, rho=0.2, payoff="put", S0=100.0,
                       grid="uniform", n_t=2, n_x=n, redraw=1, width=1.0, eta=eta, q=q, M=M, N=N,
                       K_it=k_it, omega=1.0, precision=prec, seed=5)
    print("redraw d=%d n=%d eta=%d q=%g K=%d" % (d, n, eta, q, K), flush=True)
    stepped = None
    for k in range(K):
        with bsde.Problem(config(k + 1)) as P:
            if k:
                P.set_coefficients(stepped, k)
            P.solve()
            stepped, pts = P.coefficients(), P.points()
    with bsde.Problem(config(K)) as P:
        for start in (0, 1):
            P.set_coefficients(np.zeros(P.p), start)
            P.solve()
            if start == 0:
                whole = P.coefficients()
        assert np.array_equal(P.points(), pts)
        # the pseudo-inverse fits the points it is left with
        S = P.points()
        P.fit_values(S[:, 0] + 0.5 * S[:, 1] ** 2, K)
        t, x = S[:25, 0], S[:25, 1:]
        price, _ = P.price_delta(t, np.exp(x))
    assert np.all(np.abs(whole - stepped) <= 1e-11 * np.max(np.abs(stepped)))
    ref = S[:25, 0] + 0.5 * S[:25, 1] ** 2
    assert np.all(np.abs(price - ref) <= 1e-9 * np.max(np.abs(ref)))
