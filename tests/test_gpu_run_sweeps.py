"""The FP32 sweeps that evaluate full 512-record tiles in runs of transcendentals, at the
edges of their tiles: one tile, a tile and a remainder, several tiles split over workgroups,
with fewer queries than a workgroup holds and one more than it holds, for every weight form
and queries-per-lane build, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, TOL, dq_errors, gpu_forward, points, rand_case, scaled_err
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [1.0, 2.0, 2.5, 3.0, 4.0, 1.7, 8.0])
@pytest.mark.parametrize("n,m,split", [(512, 1, 0), (513, 257, 0), (1535, 1025, 1), (4096, 300, 3)])
def test_forward_tile_edges(dim, p, n, m, split):
    x, z, q = rand_case(11 + n + m, n, m, dim)
    ref = oracle.forward(x, z, q, p)
    for prec, lanes in (("f32", (0, 4) if p >= 6.0 else (0, 2, 4, 8)), ("f32_kahan", (0,))):
        for Q in lanes:
            Z, D = gpu_forward(x, z, q, p, prec=prec, queries_per_lane=Q, split=split)
            assert np.max(scaled_err(Z, ref)) <= TOL[prec], (prec, Q)
            assert np.max(np.abs(D - ref["D"]) / ref["D"]) <= TOL[prec], (prec, Q)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [1.0, 2.0, 2.5, 3.0, 4.0, 1.7])
@pytest.mark.parametrize("n,m", [(512, 1), (577, 513), (1535, 300)])
def test_single_direction_adjoint_tile_edges(dim, p, n, m):
    """dz alone (data sweep) and dp, dq or both without dz (query sweep)."""
    x, z, q = rand_case(31 + n + m, n, m, dim)
    g = np.random.default_rng(m).normal(size=m).astype(np.float32)
    ref = oracle.backward(x, z, q, p, g.astype(np.float64))
    d, qq = points(x, z, q, "soaos", "f32")
    Z, D = api.forward(d, qq, p, "f32")
    gt = torch.from_numpy(g).cuda()
    back = lambda dz, dp, dq: api.backward(d, qq, p, gt, Z, D, "f32", need_dz=dz, need_dp=dp, need_dq=dq)
    dz = back(True, False, False)[0].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(dz - ref["dz"]) <= GTOL["f32"] * ref["dz_scale"])
    dp1 = back(False, True, False)[1]
    dq1 = back(False, False, True)[2]
    _, dp2, dq2 = back(False, True, True)
    for dp in (dp1, dp2):
        assert abs(float(dp) - ref["dp"]) <= GTOL["f32"] * ref["dp_cond"]
    for dq in (dq1, dq2):
        assert np.max(dq_errors(dq.cpu().numpy().astype(np.float64), ref)[0]) <= GTOL["f32"]
