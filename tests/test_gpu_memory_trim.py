"""pj_memory_trim gives back the memory that freed indexes leave for later ones, from any thread, and
leaves the indexes in use alone."""
import threading

import numpy as np
import pytest

import oracle as O
import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_trim():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    S = W.cfg2(100_000, seed=3)
    Q = S.subset(np.arange(50))
    exp = O.join_pj(Q, S, 2).pairs
    P.pj_build_index(S, 1, 2).free()                 # the thread's scratch stays, and code is loaded
    P.pj_memory_trim()
    before = _free()
    index = P.pj_build_index(S, 1, 2)
    held = index.info()["device_bytes"]
    index.free()
    assert held > 16 << 20
    P.pj_memory_trim()
    assert _free() == before
    # an index in use, trims from other threads meanwhile
    index = P.pj_build_index(S, 1, 2)
    stop = threading.Event()

    def trim():
        while not stop.is_set():
            P.pj_memory_trim()

    th = threading.Thread(target=trim)
    th.start()
    try:
        for _ in range(5):
            assert np.array_equal(P.pj_query(index, Q, np.full(Q.n, 2)), exp)
            P.pj_build_index(Q, 1, 2).free()
    finally:
        stop.set()
        th.join()
    index.free()
