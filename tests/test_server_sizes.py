"""Requests whose numbers are out of range: the server's admission estimate
takes them (a process of its own each, which an arithmetic trap would end), and
on a GPU their tickets report BSDE_EINVAL as bsde_create_problem does."""
import os
import subprocess
import sys

import pytest

import paper_1102_4666_amd as bsde
from workloads import problem

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BAD = [dict(n_x=0), dict(n_x=-3), dict(n_t=0), dict(n_t=-1), dict(M=0), dict(M=-600), dict(N=0),
       dict(K_it=0), dict(d=2, n_x=65536), dict(d=10, n_x=64, eta=3),
       dict(grid="uniform", n_x=1 << 27), dict(grid="random", n_t=1 << 20, n_x=1 << 20)]

ESTIMATE = r"""
import ctypes, sys
import paper_1102_4666_amd as bsde
from workloads import problem
cfg = problem(**dict(dict(eta=3, vol_level=0.2, S0=100.0), **eval(sys.argv[1])))
f = bsde.lib()._ZN4bsde20problem_device_bytesEiPK9bsde_gridiii
f.restype = ctypes.c_size_t
d, sigma, payoff, grid, keep = bsde._marshal(cfg)
print(f(d, ctypes.byref(grid), cfg["M"], cfg["N"], cfg["K_it"]))
"""


def _estimate(kw):
    r = subprocess.run([sys.executable, "-c", ESTIMATE, repr(kw)], cwd=ROOT, capture_output=True,
                       text=True)
    assert r.returncode == 0, (kw, r.returncode, r.stderr[-500:])
    return int(r.stdout.split()[-1])


@pytest.mark.parametrize("kw", BAD)
def test_estimate_of_a_refused_request_is_zero(kw):
    assert _estimate(kw) == 0


def test_estimate_of_a_request():
    assert _estimate(dict(n_t=8, n_x=64)) > 8 * 64 * 8


def _class(b):
    c = 256
    while c < b:
        c *= 2
    return c


# (d, eta, points, basis functions) on either side of the factorisation's two forms
@pytest.mark.parametrize("d,eta,n_x,p", [(1, 4, 100, 15), (5, 3, 1000, 84), (10, 3, 8192, 364)])
def test_estimate_holds_every_buffer(d, eta, n_x, p):
    kw = dict(d=d, eta=eta, grid="uniform", n_x=n_x, M=100, N=5, K_it=4)
    # the problem's own: points, coefficients and tables in one block (at most p C
    # table entries and 16 p C non-zeros of the update), then W, beta, c, var and
    # the paths' moments
    entries = p * (2 + d + d * (d + 1) // 2)
    block = 8 * n_x * (d + 1) + 12 * 16 * entries + 8 * 5 * p + 16 * entries
    own = [block, 8 * p * n_x, 8 * p * -(-n_x // 4096), 8 * 4 * n_x, 8 * 4 * n_x, 16 * n_x]
    # the set-up's: basis matrix and Q, Gram partials, Gram matrix and factors
    pap, ld = (p + 15) // 16 * 16, ((n_x + 63) // 64 | 1) * 64
    blocks = (pap + 63) // 64
    rows = max(64, (-(-ld // (2048 // (blocks * (blocks + 1) // 2))) + 15) // 16 * 16)
    work = 3 * pap * pap + pap // 16 * 256 if pap > 64 else 0
    setup = [8 * ld * pap] * 2 + [8 * -(-ld // rows) * pap * pap, 8 * (3 * pap * pap + work)]
    assert _estimate(kw) >= sum(_class(b) for b in own + setup)


@pytest.mark.gpu
def test_kernel_operator_keeps_no_least_squares_buffers():
    import torch
    torch.cuda.init()
    cfg = problem(d=1, grid="uniform", n_x=1 << 18, eta=2, M=1, N=1, K_it=1, kernel_bw=0.3)
    with bsde.Problem(dict(cfg, n_x=64)):  # what the first use of the library takes
        free = torch.cuda.mem_get_info()[0]
    with bsde.Problem(cfg):
        taken = free - torch.cuda.mem_get_info()[0]
    # 2 MB a column: points, values and table in a block of 32 MB, corrections,
    # variances and moments; the projection's segments would be another 64
    assert taken <= 48 << 20


@pytest.mark.gpu
def test_refused_requests_get_a_ticket():
    with bsde.Server(1 << 30) as S:
        tickets = [S.submit(problem(**dict(dict(eta=3, vol_level=0.2, S0=100.0), **kw)))
                   for kw in BAD]
        assert [S.poll(t)["status"] for t in tickets] == [1] * len(BAD)
        good = S.poll(S.submit(problem(eta=3)))
        assert good["status"] == 0
