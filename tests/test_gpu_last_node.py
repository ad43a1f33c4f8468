"""The last time node of a tensor or random grid is T itself for any T and
number of nodes, also where a T / (n_t - 1) rounds to a neighbour of T: paths
that start there do not move, and none starts after T."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

# (n_t - 1) T / (n_t - 1) is above T for the first three, below T for the others
# but the last, where it is T
NODES = [(0.1, 4), (0.9, 14), (90.0 / 365.0, 6), (0.7, 4), (0.9, 10), (1.0, 5)]


def _config(T, n_t, grid="tensor", **kw):
    return problem(d=1, vol_kind="bump", bump_a=0.25, vol_level=0.2, S0=100.0, T=T, grid=grid,
                   n_t=n_t, n_x=9, eta=3, M=300, N=7, K_it=1, omega=1.0, seed=11, **kw)


@pytest.mark.parametrize("grid", ["tensor", "random"])
@pytest.mark.parametrize("T,n_t", NODES)
def test_oracle_nodes_end_at_T(T, n_t, grid):
    t = oracle.points(_config(T, n_t, grid))[:, 0]
    assert np.all(t[-9:] == T) and np.all(t <= T)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("T,n_t", NODES)
def test_paths_from_the_last_node_do_not_move(T, n_t, prec):
    cfg = _config(T, n_t, precision=prec)
    print("last node T=%g n_t=%d %s" % (T, n_t, prec), flush=True)
    with bsde.Problem(cfg) as P:
        P.solve()
        c, var = P.corrections(0)
        t = P.points()[:, 0]
    assert np.all(t == oracle.points(cfg)[:, 0])
    assert np.all(var[t == T] == 0.0) and np.count_nonzero(t == T) == 9
    for i in (0, len(t) // 2, len(t) - 9, len(t) - 1):
        rc = float(oracle.corrections(cfg, np.zeros(10), 0, i, i + 1)[0][0])
        # u^0 = 0: the path term is the payoff; the log-price below 6 is rounded
        # twice in each of N steps, in 24 or 53 bits, and prices are below 300
        assert abs(c[i] - rc) <= 300 * 8 * 2 * 7 * 2.0 ** (-24 if prec == "fp32" else -53), (i, c[i], rc)
