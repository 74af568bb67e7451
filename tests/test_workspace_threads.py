"""Cached workspaces belong to one thread: a call is several launches, so two threads that enqueue
calls on one stream must not share their scratch memory.  (Host tensors stand in for device ones.)"""
import gc
import os
import threading
import weakref

import pytest
import torch

from paper_1402_4986_amd import _lib, api

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libidw.so not built")
CPU = torch.device("cpu")


def take(n, stream=0, backward=False):
    d = api.Points.hybrid(torch.zeros(n, 2), torch.zeros(n))
    return api._workspace(_lib.load(), d.c(), api.Points.hybrid(torch.zeros(n, 2)).c(), CPU, stream, "f32", None,
                          backward, False)


def test_threads_do_not_share_a_workspace():
    both = threading.Barrier(2)
    got, again, dead = {}, {}, {}

    def work(k):
        ws = take(3000 + k)
        both.wait()  # both alive, both on stream 0
        got[k], again[k] = ws.data_ptr(), take(3000 + k).data_ptr()
        dead[k] = weakref.ref(ws)
        both.wait()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got[0] != got[1] and got == again
    gc.collect()
    assert dead[0]() is None and dead[1]() is None  # given back with their threads


def test_a_thread_keeps_one_workspace_per_stream_and_grows_it():
    api._ws_cache.clear()
    try:
        a, b = take(3000), take(3000, stream=5)
        assert a.data_ptr() != b.data_ptr() and take(3000) is a and take(100) is a
        c = take(3000, backward=True)
        assert c.numel() > a.numel() and take(3000) is c and take(3000, stream=5) is b
    finally:
        api._ws_cache.clear()
