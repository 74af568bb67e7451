"""The FP32 fused adjoint, whose waves own 8 or 16 queries and sweep 64 points at a time, at the
edges of its decomposition: a point set of one batch, of a tile and one more, of several tiles
across the 4096-point additions over lanes; fewer queries than a wave owns, and one more than
a workgroup owns; leave-one-out, whose self pairs are taken apart; against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, dp_errors, dq_errors, points, rand_case
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu

FLT_FLOOR = 2.0 ** -126  # a weight below it relative to its query's largest may be flushed


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [2.0, 1.7, 7.0])
@pytest.mark.parametrize("n,m,loo", [(1, 1, False), (64, 17, False), (513, 129, False), (4097, 130, False),
                                     (9001, 257, False), (2, 2, True), (513, 513, True), (4610, 4610, True)])
def test_fused_adjoint_edges(dim, p, n, m, loo):
    x, z, q = rand_case(5 + n, n, m, dim)
    if loo:
        q = x.copy()
    g = np.random.default_rng(n).normal(size=m).astype(np.float32).astype(np.float64)
    si = np.arange(n) if loo else None
    ref = oracle.backward(x, z, q, p, g, self_index=si)
    refx = oracle.backward_x(x, z, q, p, g, self_index=si)
    d, qq = points(x, z, q, "aoas", "f32")
    Z, D = api.forward(d, qq, p, "f32", exclude_self=loo)
    gt = torch.from_numpy(g.astype(np.float32)).cuda()
    for dx in (False, True):
        r = api.backward(d, qq, p, gt, Z, D, "f32", exclude_self=loo, need_dx=dx)
        dz, dp, dq = (t.cpu().numpy().astype(np.float64) for t in r[:3])
        floor = FLT_FLOOR * np.abs(g).sum()
        assert np.all(np.abs(dz - ref["dz"]) <= GTOL["f32"] * ref["dz_scale"] + floor)
        assert dp_errors(float(dp), ref)[0] <= GTOL["f32"]
        assert np.max(dq_errors(dq, ref)[0]) <= GTOL["f32"]
        if dx:
            got = r[3].cpu().numpy().astype(np.float64)
            bound = GTOL["f32"] * refx["dx_cond"] + 2.0 ** -149
            assert np.all(np.max(np.abs(got - refx["dx"]), axis=1) <= bound)
