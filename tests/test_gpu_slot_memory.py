"""A captured serving slot holds what the server's budget counts for it."""
import re

import numpy as np
import pytest

import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


def test_slot_holds_what_is_counted():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    S = W.cfg5_index(5000)
    Q, taus = W.cfg5_batch(np.random.default_rng(1), S, mean=64)
    index = P.pj_build_index(S, 1, 8)
    with pytest.raises(P.PassJoinError) as ei:
        P.Server(index, slots=1, max_batch_queries=256, mem_budget=1)
    counted = int(re.search(r"\((\d+) bytes\)", str(ei.value)).group(1))
    held = 0
    for _ in range(3):                    # the first server also loads code and makes streams
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        with P.Server(index, slots=1, max_batch_queries=256) as srv:
            srv.wait(srv.submit(Q, taus))
            torch.cuda.synchronize()
            held = before - torch.cuda.mem_get_info()[0]
    index.free()
    print("counted", counted, "held", held, flush=True)
    # memory is handed out in steps of 2 MiB: one for the block's end, one for the graph
    assert held <= counted + (4 << 20)
