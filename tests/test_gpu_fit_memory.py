"""bsde_fit_values takes no device memory of its own, and fits the same values
on either side of the sizes it reads in place and of those it can pin."""
import numpy as np
import pytest

import paper_1102_4666_amd as bsde
from workloads import problem

pytestmark = pytest.mark.gpu


def _config(n_x, eta):
    return problem(d=1, vol_level=0.2, S0=100.0, grid="uniform", n_x=n_x, eta=eta, M=1, N=1, K_it=1,
                   seed=3)


def test_fit_takes_no_device_memory():
    import torch
    torch.cuda.init()
    with bsde.Problem(_config(5000, 2)) as P:  # what the first fit takes
        P.fit_values(P.points()[:, 0], 0)
    with bsde.Problem(_config(1 << 20, 2)) as P:
        y = P.points()[:, 0]
        free = torch.cuda.mem_get_info()[0]
        P.fit_values(y, 0)
        assert torch.cuda.mem_get_info()[0] == free


# 16 384 entries of W (1092 points of 15 functions) and 16 MB of values (2^21)
@pytest.mark.parametrize("n_x,eta", [(6, 2), (1092, 4), (1093, 4), (4097, 4), ((1 << 21) + 5, 2)])
def test_fit_of_a_polynomial(n_x, eta):
    print("fit n=%d eta=%d" % (n_x, eta), flush=True)
    with bsde.Problem(_config(n_x, eta)) as P:
        S = P.points()
        for sign in (1.0, -1.0):  # the buffers a second time
            P.fit_values(sign * (1.0 + S[:, 0] * S[:, 1] - 0.3 * S[:, 1] ** 2), 1)
            t, x = S[::max(1, n_x // 50), 0], S[::max(1, n_x // 50), 1:]
            price, _ = P.price_delta(t, np.exp(x))
            ref = sign * (1.0 + t * x[:, 0] - 0.3 * x[:, 0] ** 2)
            # kappa is 132 at the six points, and less at the others
            assert np.all(np.abs(price - ref) <= 1e-9 * np.max(np.abs(ref)))
