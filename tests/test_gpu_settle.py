"""Settling of the routes at the edges of its kernels: one workgroup owns up to 65,536 queries in
runs of 16,384, beyond that blocks of 4,096 are counted and listed; the bounding box of up to
16,384 data points is taken by one workgroup; few queries' partials are merged by four threads
each.  Exact hits sit on the first and last query of every such unit: they return their data
value bit for bit, the others agree with the FP64 oracle, and the adjoint's fix-up sums, which
follow the list's order, repeat bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, TOL, points, rand_case, scaled_err
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("p", [0.6, 2.0])
@pytest.mark.parametrize("n,m", [(64, 1), (300, 17), (1025, 4097), (16384, 300), (16385, 16385), (700, 65536),
                                 (700, 65537)])
def test_hits_at_unit_edges(prec, p, n, m):
    x, z, q = rand_case(n + m, n, m, 2, prec)
    edges = [e for u in (16, 4096, 16384, 65536) for k in (0, u, 2 * u) for e in (k - 1, k) if 0 <= e < m]
    rows = np.unique(np.array(edges + [m - 1]))
    pick = np.arange(len(rows)) % n
    q[rows] = x[pick]
    d, qq = points(x, z, q, "hybrid", prec)
    Z, D = api.forward(d, qq, p, prec)
    got = Z.cpu().numpy().astype(np.float64)
    assert np.array_equal(got[rows], z[pick])
    assert np.all(np.isinf(D.cpu().numpy()[rows]))
    some = np.unique(np.r_[rows, np.random.default_rng(m).integers(0, m, 200)])
    ref = oracle.forward(x, z, q[some], p)
    assert np.max(scaled_err(got[some], ref)) <= TOL[prec]
    g = np.random.default_rng(n).normal(size=m).astype(np.float32 if prec == "f32" else np.float64)
    gt = torch.from_numpy(g).cuda()
    a = api.backward(d, qq, p, gt, Z, D, prec)
    b = api.backward(d, qq, p, gt, Z, D, prec)
    assert all(torch.equal(u, v) for u, v in zip(a, b))
    if m <= 4097:
        ref = oracle.backward(x, z, q, p, g.astype(np.float64))
        dz = a[0].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(dz - ref["dz"]) <= GTOL[prec] * ref["dz_scale"])
        assert abs(float(a[1]) - ref["dp"]) <= GTOL[prec] * ref["dp_cond"]
