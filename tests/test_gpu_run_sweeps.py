"""The FP32 sweeps that evaluate full 512-record tiles in runs of transcendentals, at the
edges of their tiles: one tile, a tile and a remainder, several tiles split over workgroups,
with fewer queries than a workgroup holds and one more than it holds, for every weight form
and queries-per-lane build, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, gpu_forward, rand_case, scaled_err

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
