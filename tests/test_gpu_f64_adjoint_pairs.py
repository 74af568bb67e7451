"""The FP64 adjoint at p = 2 and 4, where two queries (the fused sweep) or two data points of a lane
(the data sweeps) share one reciprocal.

Accuracy: dz_j = sum g_i w_ij / D_i over uniform points at p = 4, where the weights of the nearest
points decide.  The bounds are the errors with a reciprocal per record and one Newton step in both
directions, on the same inputs, in units of 2^-53 of the sum of absolute terms; with the forward's
reciprocals shared and the adjoint's not they were above them.

Partners: one of the two lies past the end of the points, is a hit, the leave-one-out self pair, a
point at infinity, or so far away that the product would overflow; the other must not notice."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, dp_errors, dq_errors, points, rand_case
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu

ASKED = [dict(need_dp=False, need_dq=False), dict(), dict(need_dx=True), dict(separate=True),
         dict(need_dx=True, separate=True)]


def dz_error(dim, p, seed=3, n=4096, m=1024):
    """dz over all points, its exact value and sum of absolute terms (80 bits)."""
    r = np.random.default_rng(seed)
    x, z, q, g = r.random((n, dim)), r.normal(size=n), r.random((m, dim)), r.normal(size=m)
    d, qq = points(x, z, q, "aoas", "f64")
    Z, D = api.forward(d, qq, p, "f64")
    want, scale = np.zeros(n, np.longdouble), np.zeros(n, np.longdouble)
    for s in range(0, m, 128):
        r2 = ((q[s:s + 128, None].astype(np.longdouble) - x[None].astype(np.longdouble)) ** 2).sum(-1)
        w = r2 ** (-int(p) // 2)
        t = g[s:s + 128, None] / w.sum(1)[:, None] * w
        want += t.sum(0)
        scale += np.abs(t).sum(0)
    out = []
    for asked in ASKED[:3]:
        dz = api.backward(d, qq, p, torch.from_numpy(g).cuda(), Z, D, "f64", **asked)[0].cpu().numpy()
        out.append(float(np.sqrt(np.mean(((dz - want) / scale * np.longdouble(2.0 ** 53)) ** 2))))
    return out


@pytest.mark.parametrize("dim,p,alone,fused", [(2, 2.0, 1.038, 1.100), (2, 4.0, 2.936, 2.925), (3, 2.0, 0.467, 0.489),
                                               (3, 4.0, 1.981, 2.021)])
def test_dz_is_no_further_off_than_with_single_reciprocals(dim, p, alone, fused):
    for got, most in zip(dz_error(dim, p), (alone, fused, fused)):
        assert got <= most


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [2.0, 4.0])
@pytest.mark.parametrize("n,m,kind", [(1, 5, "plain"), (3, 600, "hits"), (257, 300, "hits"), (513, 700, "plain"),
                                      (258, 258, "loo"), (777, 777, "loo"), (257, 40, "inf"), (514, 600, "inf"),
                                      (100, 70, "far"), (515, 520, "far")])
def test_partners_do_not_notice(dim, p, n, m, kind):
    x, z, q = rand_case(31 * n + m, n, m, dim, "f64", -0.5, 0.5)
    q[0] = 0.0                                        # where a point without coordinates would lie
    loo = kind == "loo"
    if kind == "hits":
        q[1::3] = x[np.arange(len(q[1::3])) % n]
    if loo:
        q = x.copy()
    if kind == "far":
        q[2::4] *= 1e100 if p == 2.0 else 1e76        # products of two r^2 past 2^1024
    there = np.ones(n, bool)
    if kind == "inf":
        x[n // 2, 0], x[n - 1, dim - 1] = np.inf, -np.inf
        there[[n // 2, n - 1]] = False
    g = np.random.default_rng(n).normal(size=m)
    si = np.arange(n) if loo else None
    ref = oracle.backward(x[there], z[there], q, p, g, self_index=si)
    refx = oracle.backward_x(x[there], z[there], q, p, g, self_index=si)
    d, qq = points(x, z, q, "hybrid", "f64")
    Z, D = api.forward(d, qq, p, "f64", exclude_self=loo)
    for asked in ASKED:
        out = [None if v is None else v.cpu().numpy() for v in
               api.backward(d, qq, p, torch.from_numpy(g).cuda(), Z, D, "f64", exclude_self=loo, **asked)]
        assert np.all(np.abs(out[0][there] - ref["dz"]) <= GTOL["f64"] * ref["dz_scale"]), asked
        if kind != "inf" and out[1] is not None:
            assert dp_errors(float(out[1]), ref)[0] <= GTOL["f64"], asked
            assert np.max(dq_errors(out[2], ref)[0]) <= GTOL["f64"], asked
        if len(out) == 4:
            got = out[3][there]
            assert np.all(np.max(np.abs(got - refx["dx"]), axis=1) <= GTOL["f64"] * refx["dx_cond"] + 2.0 ** -1074), asked
