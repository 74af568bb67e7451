"""Data points with a coordinate that is not finite, in FP64, whose sweeps take their weights from
tables: a point at infinity has weight 0 in every form and leaves the other points' dz alone; a NaN
coordinate makes every query NaN, as in the oracle, whatever its sign bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, TOL, points, rand_case, scaled_err
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [0.7, 1.7, 2.0, 4.0, 6.5])
@pytest.mark.parametrize("n,at", [(5, 4), (700, 3), (700, 690)])
@pytest.mark.parametrize("m", [130, 16390])
def test_f64_point_at_infinity(p, n, at, m):
    x, z, q = rand_case(n + at, n, m, 2, "f64")
    x[at, 1] = np.inf
    d, qq = points(x, z, q, "aoas", "f64")
    Z, D = api.forward(d, qq, p, "f64")
    ref = oracle.forward(x, z, q[:130], p)
    assert np.all(np.isfinite(ref["Z"]))
    assert np.max(scaled_err(Z.cpu().numpy()[:130], ref)) <= TOL["f64"]
    if m == 130:
        g = np.random.default_rng(n).normal(size=m)
        refb = oracle.backward(x, z, q, p, g)
        for need_dp in (False, True):
            dz = api.backward(d, qq, p, torch.from_numpy(g).cuda(), Z, D, "f64", True, need_dp, False)[0].cpu().numpy()
            keep = np.arange(n) != at
            assert np.all(np.abs(dz - refb["dz"])[keep] <= GTOL["f64"] * refb["dz_scale"][keep])


@pytest.mark.parametrize("p", [0.7, 1.7, 2.0, 6.5])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("m", [130, 16390])
def test_f64_nan_point(p, sign, m):
    x, z, q = rand_case(11, 700, m, 2, "f64")
    x[650, 0] = np.copysign(np.nan, sign)
    d, qq = points(x, z, q, "aoas", "f64")
    Z, _ = api.forward(d, qq, p, "f64")
    assert np.all(np.isnan(Z.cpu().numpy()))
