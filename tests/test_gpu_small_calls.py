"""Small calls at the limits of their kernels, against the FP64 oracle.  A forward of few pairs
(both sets up to 16,384, up to 2^26 pairs) is ended by one kernel that merges, checks the nearest
distances and recomputes the queries sent to FP64; beyond either limit the general kernels do it.
A third of the queries sit on or next to a data point, so every stage has work, at exponents
below and above the one under which the FP32 sweep asks for a distance check.  The adjoint's
FP64 pass over such queries is one kernel up to 4,096 data points and two above, and dp is summed
in its last kernel or, without dz, in one of its own: whichever outputs are asked for together,
each agrees with the oracle and repeats bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, TOL, dp_errors, dq_errors, oracle_forward_par, points, rand_case, scaled_err
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


def near_case(n, m, dim, prec):
    x, z, q = rand_case(3 * n + m, n, m, dim, prec)
    t = np.float64 if prec == "f64" else np.float32
    step = 1e-7 if prec == "f64" else 2.0 ** -22
    q[::6] = x[np.arange(0, m, 6) % n]
    k = np.arange(3, m, 6)
    q[k] = (x[k % n] + step).astype(t)
    return x, z, q


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dim,p", [(2, 0.4), (2, 2.0), (3, 3.1)])
@pytest.mark.parametrize("n,m", [(1, 5), (63, 4), (4099, 7), (16384, 67), (16385, 67), (67, 16384), (67, 16385),
                                 (16384, 2048), (16384, 4096), (16384, 4097)])
def test_forward_limits(prec, dim, p, n, m):
    x, z, q = near_case(n, m, dim, prec)
    d, qq = points(x, z, q, "aoas", prec)
    some = np.unique(np.r_[np.arange(min(m, 130)), np.arange(max(0, m - 130), m)])
    ref = oracle_forward_par(x, z, q[some], p)
    for split in (0, 3):
        Z, D = api.forward(d, qq, p, prec, split=split)
        got, den = Z.cpu().numpy().astype(np.float64)[some], D.cpu().numpy()
        assert np.all(np.isinf(den[::6])) and np.all(np.isfinite(np.delete(den, np.arange(0, m, 6))))
        assert np.max(scaled_err(got, ref)) <= TOL[prec]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("p", [2.0, 2.7])
@pytest.mark.parametrize("n,m", [(4096, 61), (4097, 61), (700, 1500)])
def test_adjoint_outputs_apart_and_together(prec, p, n, m):
    x, z, q = near_case(n, m, 2, prec)
    t = np.float32 if prec == "f32" else np.float64
    g = np.random.default_rng(n).normal(size=m).astype(t)
    ref = oracle.backward(x, z, q, p, g.astype(np.float64))
    d, qq = points(x, z, q, "aoas", prec)
    Z, D = api.forward(d, qq, p, prec)
    gt = torch.from_numpy(g).cuda()
    T, F = True, False
    for need in ((T, F, F), (F, T, F), (F, F, T), (T, T, F), (F, T, T), (T, T, T)):
        for separate in (False, True):
            a, b = (api.backward(d, qq, p, gt, Z, D, prec, *need, separate=separate)[:3] for _ in range(2))
            assert all(torch.equal(u, v) for want, u, v in zip(need, a, b) if want)
            dz, dp, dq = (v.cpu().numpy().astype(np.float64) if v is not None else None for v in a)
            if need[0]:
                assert np.all(np.abs(dz - ref["dz"]) <= GTOL[prec] * ref["dz_scale"])
            if need[1]:
                assert dp_errors(float(dp), ref)[0] <= GTOL[prec]
            if need[2]:
                assert np.max(dq_errors(dq, ref)[0]) <= GTOL[prec]
