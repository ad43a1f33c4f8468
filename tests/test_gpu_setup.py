"""The least-squares set-up on the device (basis matrix, Gram matrices,
blocked factorisations, products) at the edges of its 16-column tiles and of
its one-workgroup form: coefficients of a polynomial in the span come back
from its values at the points, and rank-deficient grids are refused."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu

# (d, eta, q, grid): p = 6, 15, 28, 45 (one to three tiles), 56 and 84 (the
# last one-workgroup and the first global-memory factorisation), 70, 78, 100,
# 111, 221, 364, 386; point counts off the 64-row padding
SETS = [(1, 2, 1.0, dict(n_t=4, n_x=5)), (1, 4, 1.0, dict(n_t=7, n_x=9)),
        (1, 6, 1.0, dict(n_t=9, n_x=21)), (1, 8, 1.0, dict(n_t=13, n_x=37)),
        (2, 5, 1.0, dict(n_t=7, n_x=9)), (3, 4, 1.0, dict(n_t=6, n_x=6)),
        (5, 3, 1.0, dict(grid="random", n_t=6, n_x=211)),
        (10, 2, 1.0, dict(grid="uniform", n_x=403)),
        (10, 4, 0.6, dict(grid="uniform", n_x=701)),
        (10, 5, 0.5, dict(grid="uniform", n_x=705)),
        (10, 5, 0.6, dict(grid="uniform", n_x=1501)),
        (10, 3, 1.0, dict(grid="uniform", n_x=2049)),
        (10, 5, 0.7, dict(grid="uniform", n_x=2600))]


@pytest.mark.parametrize("d,eta,q,grid", SETS)
def test_polynomial_comes_back_from_its_values(d, eta, q, grid):
    cfg = problem(d=d, S0=100.0, vol_level=0.2, eta=eta, q=q, M=1, N=1, K_it=1,
                  precision="fp32" if q < 1 else "fp64", seed=3, **grid)
    print("set-up d=%d eta=%d q=%g" % (d, eta, q), flush=True)
    B = oracle.basis_matrix(cfg)  # monomials: the same span
    a = np.random.default_rng(5).normal(size=B.shape[1])
    y = B @ a
    with bsde.Problem(cfg) as P:
        assert B.shape == (P.n, P.p)
        P.fit_values(y, 1)
        rng = np.random.default_rng(6)
        t = rng.uniform(0.0, 1.0, 8)
        S = 100.0 * np.exp(rng.uniform(-0.3, 0.3, (8, d)))
        price, _ = P.price_delta(t, S)
        alpha = P.coefficients(1)
    # the oracle's values of the same polynomial at the query points
    ref, _ = oracle.price_delta(cfg, a, t, S)
    # a least-squares solution is off by a few kappa 2^-52 of the data's size
    # (kappa of the Chebyshev basis the library solves in is at most that of
    # the monomials), and a value sums p coefficients
    kappa = np.linalg.cond(B)
    tol = 64 * P.p * kappa * 2.0 ** -52 * np.abs(y).max()
    print("  p=%d kappa %.3g error %.3g tolerance %.3g" % (len(a), kappa, np.abs(price - ref).max(), tol))
    assert np.all(np.isfinite(alpha))
    assert np.abs(price - ref).max() <= tol


@pytest.mark.parametrize("d,eta,grid", [
    (1, 4, dict(n_t=3, n_x=20)),                  # degree 4 in time on 3 nodes
    (3, 4, dict(n_t=3, n_x=6)),                   # the same beyond 64 columns
    (10, 3, dict(grid="random", n_t=3, n_x=300))])
def test_rank_deficient_grid_is_refused(d, eta, grid):
    cfg = problem(d=d, S0=100.0, vol_level=0.2, eta=eta, M=1, N=1, K_it=1, **grid)
    with pytest.raises(bsde.BsdeError) as e:
        bsde.Problem(cfg)
    assert e.value.status == 3
