"""dz alone at p >= 6 in FP32: the fused adjoint's build without query sums, 16 queries per wave and
128 per workgroup, at the edges of its decomposition, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, points, rand_case
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [6.0, 9.5])
@pytest.mark.parametrize("n,m,loo", [(1, 1, False), (64, 17, False), (513, 127, False), (513, 129, False),
                                     (9001, 257, False), (15, 15, True), (513, 513, True), (4610, 4610, True)])
def test_dz_alone_with_relative_weights(dim, p, n, m, loo):
    x, z, q = rand_case(9 + n, n, m, dim)
    if loo:
        q = x.copy()
    g = np.random.default_rng(n).normal(size=m).astype(np.float32).astype(np.float64)
    ref = oracle.backward(x, z, q, p, g, self_index=np.arange(n) if loo else None)
    d, qq = points(x, z, q, "aoas", "f32")
    Z, D = api.forward(d, qq, p, "f32", exclude_self=loo)
    dz, dp, dq = api.backward(d, qq, p, torch.from_numpy(g.astype(np.float32)).cuda(), Z, D, "f32", exclude_self=loo,
                              need_dp=False, need_dq=False)
    assert dp is None and dq is None
    floor = 2.0 ** -126 * np.abs(g).sum()  # a weight below it relative to its query's largest may be flushed
    assert np.all(np.abs(dz.cpu().numpy().astype(np.float64) - ref["dz"]) <= GTOL["f32"] * ref["dz_scale"] + floor)
