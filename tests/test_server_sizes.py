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


@pytest.mark.gpu
def test_refused_requests_get_a_ticket():
    with bsde.Server(1 << 30) as S:
        tickets = [S.submit(problem(**dict(dict(eta=3, vol_level=0.2, S0=100.0), **kw)))
                   for kw in BAD]
        assert [S.poll(t)["status"] for t in tickets] == [1] * len(BAD)
        good = S.poll(S.submit(problem(eta=3)))
        assert good["status"] == 0
