"""The FP32 adjoint's sums over the lanes of a wave are FP64 sums of the lanes' FP32 sums.

One query, and data points at two places at the same distance d from it, so that every pair has
the same weight and a pair's term is its value times one constant.  Point 0 has the value A, its
seven neighbours (which other lanes hold) A 2^-25, and a later point -A; the others have 0.  Added
in FP32 to A, the seven vanish in whole or in part; their FP64 sum is left when -A has cancelled A.
The only rounding of the query's sums is then that of the common factor, a few units in the last
place of FP32, so the bound is 1e-5 of the result itself."""
import numpy as np
import pytest
import torch

from gpu_helpers import points
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [2.0, 1.7, 8.0])
@pytest.mark.parametrize("dx", [False, True])
def test_sums_over_lanes_are_fp64(dim, p, dx):
    n, d = 8192, 0.25                                        # a box of side 1/2: the coordinates are not scaled
    x, z, q = np.zeros((n, dim)), np.zeros(n), np.zeros((1, dim))
    x[:, 0] = d
    x[9:-1:2, 0] = -d                                        # points of value 0, so that the box has a side
    z[0], z[1:8], z[-1] = 1.0, 2.0 ** -25, -1.0
    data, query = points(x, z, q, "aoas", "f32")
    one = torch.ones(1, dtype=torch.float32, device="cuda")
    den = torch.tensor([n * d ** -p], dtype=torch.float64, device="cuda")
    _, gp, gq = api.backward(data, query, p, one, torch.zeros_like(one), den, "f32", need_dx=dx)[:3]
    rest = 7 * 2.0 ** -25                                    # the sum of the values
    want_p = -np.log(d) * rest / n                           # -(1/D) w ln(d) rest
    want_q = p * rest / (n * d)                              # -(p/D) (w / d^2) (-d) rest
    got = gq.cpu().numpy().astype(np.float64)[0]
    assert abs(float(gp) - want_p) <= 1e-5 * want_p
    assert abs(got[0] - want_q) <= 1e-5 * want_q
    assert np.all(got[1:] == 0.0)
