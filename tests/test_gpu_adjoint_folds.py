"""The FP32 fused adjoint where its workgroups take several tiles and several query blocks: a group
folds more than one block of 128 queries (64 with relative weights) into its rows of dz and dx, and
a range holds more than the eight 512-point tiles between two additions over the lanes, so that the
query sums are added to more than once (in 3-D with dx, in memory).  The planned groups are read off
the workspace, whose dx rows are one per group; the upstream gradient is non-zero on 150 queries, so
that the FP64 oracle needs just those.

   n       m       groups   blocks of 128   ranges   tiles of a range
   20,011  30,011  128      235             4        10
    9,001  60,013  256      469             2         9
   25,009  25,009  102      196             5        10     (leave-one-out)"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import GTOL, dp_errors, dq_errors, points, rand_case
from paper_1402_4986_amd import _lib, api

pytestmark = pytest.mark.gpu


def _groups(d, q):
    lib, size = _lib.load(), []
    for flags in (_lib.NEED_DZ, _lib.NEED_DX):
        out = ctypes.c_size_t()
        assert lib.idw_workspace_size(ctypes.byref(d.c()), ctypes.byref(q.c()), _lib.FP32, flags, None,
                                      ctypes.byref(out)) == 0
        size.append(out.value)
    return (size[1] - size[0]) // (8 * d.n * d.dim)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("p", [2.0, 1.7, 8.0])
@pytest.mark.parametrize("n,m,loo,groups", [(20011, 30011, False, 128), (9001, 60013, False, 256),
                                            (25009, 25009, True, 102)])
def test_rows_and_query_sums_are_folded(dim, p, n, m, loo, groups):
    x, z, q = rand_case(70 + dim, n, m, dim)
    if loo:
        q = x.copy()
    r = np.random.default_rng(n)
    sel = np.sort(r.choice(m, size=150, replace=False))
    g = np.zeros(m)
    g[sel] = r.normal(size=150).astype(np.float32)
    si = sel if loo else None
    ref = oracle.backward(x, z, q[sel], p, g[sel], self_index=si)
    refx = oracle.backward_x(x, z, q[sel], p, g[sel], self_index=si)
    d, qq = points(x, z, q, "soa", "f32")
    assert _groups(d, qq) == groups < -(-m // 128)
    Z, D = api.forward(d, qq, p, "f32", exclude_self=loo)
    gt = torch.from_numpy(g.astype(np.float32)).cuda()
    rest = np.setdiff1d(np.arange(m), sel)
    floor = 2.0 ** -126 * np.abs(g).sum()  # a weight below it relative to its query's largest may be flushed
    for dx in (False, True):
        out = api.backward(d, qq, p, gt, Z, D, "f32", exclude_self=loo, need_dx=dx)
        dz, dp, dq = (t.cpu().numpy().astype(np.float64) for t in out[:3])
        assert np.all(np.abs(dz - ref["dz"]) <= GTOL["f32"] * ref["dz_scale"] + floor)
        assert dp_errors(float(dp), ref)[0] <= GTOL["f32"]
        assert np.max(dq_errors(dq[sel], ref)[0]) <= GTOL["f32"] and np.all(dq[rest] == 0.0)
        if dx:
            got = out[3].cpu().numpy().astype(np.float64)
            assert np.all(np.max(np.abs(got - refx["dx"]), axis=1) <= GTOL["f32"] * refx["dx_cond"] + 2.0 ** -149)
