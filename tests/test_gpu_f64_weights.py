"""The FP64 forward's weights at p = 4, where four records of a query share one reciprocal.

One data point is at the origin and 63 at a distance of 1/2 or more; the queries lie 1e-5 to 4e-5
from the origin on the first axis.  The near point's weight, 1e20 or so, is then the whole
denominator (the others are below half a unit in its last place and are added after it), and
r^2 is exact, since the coordinates have 24 bits.  So the relative error of D is that of w = t^2,
twice the error of the reciprocal t and one rounding.

The bound: six roundings lead to t (two products, their product, the refined reciprocal and two
more products), each at most 2^-53 relative and taken as uniform, rms 0.58 2^-53.  Their rms is
sqrt(6) 0.58 = 1.42, doubled by the square 2.84, with its own rounding 2.9: 3.0 in units of 2^-53.
A reciprocal with one Newton step and the same products has 3.9, one of its own per record 3.5."""
import numpy as np
import pytest

from gpu_helpers import gpu_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("m", [4096, 70000])
def test_weights_are_as_accurate_as_their_roundings(dim, m):
    r = np.random.default_rng(dim)
    x = np.zeros((64, dim))
    x[1:] = r.uniform(0.5, 1.0, (63, dim))
    q = np.zeros((m, dim))
    q[:, 0] = np.exp(r.uniform(np.log(1e-5), np.log(4e-5), m)).astype(np.float32)
    _, D = gpu_forward(x, r.normal(size=64), q, 4.0, "aoas", "f64")
    e = (D.astype(np.longdouble) * q[:, 0].astype(np.longdouble) ** 4 - 1) * np.longdouble(2.0 ** 53)
    assert float(np.sqrt(np.mean(e * e))) <= 3.0
