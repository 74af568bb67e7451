"""FP64 forward forms at their edges against the oracle at 1e-12: four records per reciprocal
(p = 2, 4) at sizes around a group and a 64-record block, with coordinates small enough that
products of four squared distances leave no margin for an unscaled form, queries on and very
near data points, and a query far outside the box; the general-p series on both sides of the
exponent where it is shortened (p = 6)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, gpu_forward, rand_case, scaled_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [2.0, 4.0, 0.3, 5.999, 6.0, 6.001])
@pytest.mark.parametrize("n", [3, 64, 67, 577])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -60])
def test_f64_forward_forms(dim, p, n, scale):
    x, z, q = rand_case(n, n, 130, dim, "f64")
    q[0] = x[0]                       # exact hit
    q[1] = x[1] + 1e-9                # near-coincident
    q[2] = 1e3                        # outside the box
    q[3] = x[2] * (1.0 + 2e-16)
    x, q = x * scale, q * scale
    Z, D = gpu_forward(x, z, q, p, prec="f64")
    ref = oracle.forward(x, z, q, p)
    assert Z[0] == z[0] and np.isinf(D[0])
    assert np.max(scaled_err(Z, ref)) <= TOL["f64"]


@pytest.mark.parametrize("p", [2.0, 4.0])
def test_f64_far_query_leaves_the_product_range(p):
    # squared distances whose product of four passes the FP64 range: recomputed in the fix-up
    x, z, q = rand_case(9, 200, 4, 2, "f64")
    q[1] = 1e50
    Z, D = gpu_forward(x, z, q, p, prec="f64")
    ref = oracle.forward(x, z, q, p)
    assert np.max(scaled_err(Z, ref)) <= TOL["f64"]
    assert np.max(np.abs(D - ref["D"]) / ref["D"]) <= TOL["f64"]
