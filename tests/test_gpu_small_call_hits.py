"""Hits of neighbouring queries in a small forward.  The four queries that one workgroup of the
finishing kernel ends share their passes over the data: four hits side by side add less than 3.3
times what they add far apart, each in a workgroup of its own (passes in turn: 3.75 or more; two
in a pass at 1.0 to 1.6 times the price of one: 2.0 to 3.2).  Where a pass is long and the call is
not small otherwise (n^2 m above 5 2^37), the general kernels cut a query's data among workgroups:
there they add less than 1.5 times as much.  Every mixture of hits, near points and far queries in
a group, and both sides of that limit, agree with the oracle."""
import itertools
import time

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import TOL, oracle_forward_par, points, rand_case, scaled_err
from paper_1402_4986_amd import api

pytestmark = pytest.mark.gpu


def _replay_time(call, per_graph=20, reps=20, tries=5):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(per_graph):
                call()
        graph.replay()
        stream.synchronize()
        best = float("inf")
        for _ in range(tries):
            t0 = time.perf_counter()
            for _ in range(reps):
                graph.replay()
            stream.synchronize()
            best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("p", [2.0, 1.7])
@pytest.mark.parametrize("m,most", [(1000, 3.3), (4096, 1.5)])
def test_neighbouring_hits_share_passes(p, m, most):
    n = 16384
    x, z, q = rand_case(7, n, m, 2)
    took = []
    for where in (np.arange(0), np.arange(4) * 100 + 400, np.arange(4) + 400):
        qh = q.copy()
        qh[where] = x[np.arange(len(where)) * 1000 + 17]
        d, qq = points(x, z, qh, "aoas", "f32")
        ws = api.workspace(d, qq, "f32", backward=False)
        out = (torch.empty(m, dtype=torch.float32, device="cuda"), torch.empty(m, dtype=torch.float64, device="cuda"))
        took.append(_replay_time(lambda: api.forward(d, qq, p, "f32", out_z=out[0], out_den=out[1], ws=ws)))
        assert int(torch.isinf(out[1]).sum()) == len(where)
    none, apart, together = took
    assert together - none < most * (apart - none)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dim,p", [(2, 0.4), (2, 2.0), (3, 3.1)])
@pytest.mark.parametrize("n,m", [(16384, 2560), (16384, 2561), (10240, 6553), (10241, 6553)])
def test_both_sides_of_the_limit(prec, dim, p, n, m):
    x, z, q = rand_case(n + m, n, m, dim, prec)
    t = np.float64 if prec == "f64" else np.float32
    q[:6] = x[100:106]
    q[6:12] = (x[200:206] + (1e-7 if prec == "f64" else 2.0 ** -22)).astype(t)
    d, qq = points(x, z, q, "soa", prec)
    Z, D = api.forward(d, qq, p, prec)
    some = np.r_[np.arange(130), np.arange(m - 130, m)]
    ref = oracle_forward_par(x, z, q[some], p)
    assert np.max(scaled_err(Z.cpu().numpy().astype(np.float64)[some], ref)) <= TOL[prec]
    assert np.array_equal(np.isinf(D.cpu().numpy()[some]), ref["H"] > 0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dim,p", [(2, 0.4), (2, 2.0), (3, 3.1)])
@pytest.mark.parametrize("loo", [False, True])
def test_every_mixture_in_a_group(prec, dim, p, loo):
    n = 1029
    x, z, q = rand_case(11, n, n, dim, prec)
    t = np.float64 if prec == "f64" else np.float32
    step = 1e-7 if prec == "f64" else 2.0 ** -22
    # groups of four over {far, hit, near}, a hit or near point 517 away from the query's own index
    kinds = np.array(list(itertools.product(range(3), repeat=4))).ravel()
    for i, kind in enumerate(kinds):
        if kind:
            q[i] = (x[(i + 517) % n] + (step if kind == 2 else 0.0)).astype(t)
    if loo:
        x[: len(kinds)] = q[: len(kinds)]
        q = x.copy()
    d, qq = points(x, z, q, "hybrid", prec)
    Z, D = api.forward(d, qq, p, prec, exclude_self=loo)
    ref = oracle.forward(x, z, q, p, self_index=np.arange(n) if loo else None)
    assert np.max(scaled_err(Z.cpu().numpy().astype(np.float64), ref)) <= TOL[prec]
    assert np.array_equal(np.isinf(D.cpu().numpy()), ref["H"] > 0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dim,p", [(2, 0.5), (2, 1.7), (3, 3.0)])
def test_a_query_alone_has_the_same_bits(prec, dim, p):
    # next to a point: recomputed in FP64, alone by one pass, beside hits and others two to a pass
    n, m = 1024, 1000
    x, z, q = rand_case(13, n, m, dim, prec)
    q[::3] = x[:m:3]
    q[1::5] = (x[1:m:5] + 2.0 ** -22).astype(np.float64 if prec == "f64" else np.float32)
    d, qq = points(x, z, q, "hybrid", prec)
    Z, D = api.forward(d, qq, p, prec)
    for i in range(1, m, 5):
        Zi, Di = api.forward(d, points(x, z, q[i:i + 1], "hybrid", prec)[1], p, prec)
        assert torch.equal(Z[i:i + 1], Zi) and torch.equal(D[i:i + 1], Di), i
