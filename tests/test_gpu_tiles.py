"""How a point's paths are cut into tiles: points at T, whose paths do not
move, and numbers of paths around a wavefront and a workgroup in one and
several groups."""
import numpy as np
import pytest

import oracle
import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu

# per-point corrections relative to 1 + |c| + standard deviation + |u|
TOL = {"fp64": 1e-8, "fp32": 2e-3}


def _config(d, M, N, prec, **kw):
    shape = {1: dict(grid="tensor", n_t=6, n_x=9, eta=3), 2: dict(grid="tensor", n_t=7, n_x=8, eta=4),
             3: dict(grid="random", n_t=5, n_x=30, eta=2), 5: dict(grid="random", n_t=5, n_x=80, eta=3),
             10: dict(grid="random", n_t=5, n_x=120, eta=2)}[d]
    return problem(d=d, vol_kind="bump", vol_level=[0.15 + 0.02 * j for j in range(d)], bump_a=0.25,
                   rho=0.2 if d > 1 else 0.0, payoff="put", S0=100.0, M=M, N=N, K_it=2, omega=1.0,
                   precision=prec, seed=21, **dict(shape, **kw))


def _iterate(cfg):
    nu = oracle.index_set(cfg["d"] + 1, cfg["eta"])
    alpha = np.random.default_rng(9).normal(size=len(nu)) * 3.0 * 0.4 ** nu.sum(axis=1)
    return alpha, oracle.basis_matrix(cfg) @ alpha


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("d", [1, 2, 3, 5, 10])
def test_points_at_the_end_have_no_spread(d, prec):
    cfg = _config(d, 700, 7, prec)
    alpha, y = _iterate(cfg)
    print("points at T d=%d %s" % (d, prec), flush=True)
    with bsde.Problem(cfg) as P:
        P.fit_values(y, 1)
        P.solve()
        c, var = P.corrections(1)
        last = np.flatnonzero(P.points()[:, 0] == cfg["T"])
    assert len(last) == len(c) // cfg["n_t"]
    assert np.all(var[last] == 0.0)
    for i in last[[0, len(last) // 2, -1]]:
        rc, rv = (float(v[0]) for v in oracle.corrections(cfg, alpha, 1, i, i + 1))
        assert rv <= 1e-20
        assert abs(c[i] - rc) <= TOL[prec] * (1.0 + abs(rc) + abs(y[i])), (i, c[i], rc)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("M,tilings", [(1, [(1, 1), (3, 1)]), (64, [(1, 1)]), (65, [(1, 1), (2, 1)]),
                                       (256, [(1, 1), (8, 1)]), (777, [(1, 4), (2, 2), (4, 1), (8, 2)]),
                                       (1300, [(1, 6), (3, 2), (5, 2)])])
def test_moments_do_not_depend_on_the_tiling(M, tilings, prec):
    cfg = _config(2, M, 5, prec)
    alpha, y = _iterate(cfg)
    print("tilings of M=%d %s" % (M, prec), flush=True)
    with bsde.Problem(cfg) as P:
        got = []
        for t in [None] + tilings:
            P.set_tiling(*(t or (0, 0)))
            P.fit_values(y, 1)
            P.solve()
            got.append(P.corrections(1))
    # the paths' terms are the same numbers in every tiling; their moments
    # differ by the rounding of FP64 sums of at most 1300 terms
    c0, v0 = got[0]
    for c, v in got[1:]:
        assert np.all(np.abs(c - c0) <= 1e-12 * (1.0 + np.abs(c0) + np.sqrt(v0)))
        assert np.all(np.abs(v - v0) <= 1e-11 * (v0 + 1e-12 * (1.0 + c0 ** 2)))
    for i in (3, len(y) // 2 + 1):
        rc, rv = (float(v[0]) for v in oracle.corrections(cfg, alpha, 1, i, i + 1))
        scale = 1.0 + abs(rc) + np.sqrt(rv) + abs(y[i])
        assert abs(c0[i] - rc) <= TOL[prec] * scale
        assert abs(v0[i] - rv) <= 4 * TOL[prec] * scale ** 2


# points, functions, tilings and table entries around the sizes of the
# one-workgroup update (16 waves, strides of 512 and 1024, 32 K entries)
@pytest.mark.parametrize("d,n_t,n_x,eta,M,tiling", [
    (1, 3, 3, 2, 40, None), (1, 9, 57, 4, 300, None), (1, 9, 57, 8, 2500, (7, 2)),
    (1, 16, 128, 4, 500, (2, 1)), (1, 16, 128, 4, 600, (3, 1)), (2, 6, 11, 4, 300, None),
    (2, 8, 16, 5, 70, None), (5, 8, 60, 3, 90, None), (10, 4, 70, 2, 40, None)])
def test_update_in_one_workgroup_and_in_three_launches(d, n_t, n_x, eta, M, tiling):
    cfg = _config(d, M, 4, "fp64", n_t=n_t, n_x=n_x, eta=eta)
    print("update d=%d n_t=%d n_x=%d eta=%d M=%d" % (d, n_t, n_x, eta, M), flush=True)
    got = []
    for level in (1, 2):  # level 2 times the three kernels
        with bsde.Problem(cfg) as P:
            P.set_timing(level)
            if tiling:
                P.set_tiling(*tiling)
            P.solve()
            got.append((P.coefficients(),) + P.corrections(1))
    # the same sums in the same order
    for x, y in zip(*got):
        assert np.all(np.abs(x - y) <= 1e-13 * np.max(np.abs(y)))


# points around one segment of the projection, several, and the most of them
@pytest.mark.parametrize("n_t,n_x", [(16, 256), (17, 241), (9, 911), (7, 19000)])
def test_fit_over_segments_of_points(n_t, n_x):
    cfg = _config(1, 1, 1, "fp64", n_t=n_t, n_x=n_x, eta=2)
    print("segments n_t=%d n_x=%d" % (n_t, n_x), flush=True)
    with bsde.Problem(cfg) as P:
        S = P.points()
        P.fit_values(1.0 + S[:, 0] * S[:, 1] - 0.3 * S[:, 1] ** 2, 1)
        t, x = S[::97, 0], S[::97, 1:]
        price, _ = P.price_delta(t, np.exp(x))
    ref = 1.0 + t * x[:, 0] - 0.3 * x[:, 0] ** 2
    assert np.all(np.abs(price - ref) <= 1e-10 * np.max(np.abs(ref)))
