"""A plan sees every single changed byte: at the ends of the 16 bytes read at a time, in the last ones of
a set whose size is no multiple of them, and with the bytes at any address.  Results equal an ordinary
join's of the same strings."""
import numpy as np
import pytest

import paper_1111_7171_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", [0, 3, 8])
@pytest.mark.parametrize("rest", [0, 1, 7, 8, 9, 15])
def test_one_byte(rest, at):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    print("bytes over 16", rest, "address", at, flush=True)
    words = [b"plan%03d" % (k % 400) for k in range(800)]
    size = sum(map(len, words))
    words.append(b"z" * ((rest - size) % 16 + 16))
    col = W.from_list(words)
    total = len(col.chars)
    assert total % 16 == rest
    buf = torch.zeros(at + total, dtype=torch.uint8, device="cuda")
    chars = buf[at:]
    chars.copy_(torch.from_numpy(col.chars.copy()))
    offs = torch.from_numpy(col.offsets.copy()).cuda()
    plan = P.Plan((chars, offs), 1)

    def run():
        got = plan.run()
        pairs = got.to_numpy()
        got.free()
        return P.pj_last_stats()["replayed"], pairs

    replayed, first = run()
    assert replayed == 1
    for k in [0, 7, 8, 15, 16, total - 17, total - 16, total - 2, total - 1]:
        saved = int(chars[k])
        chars[k] = saved ^ 1
        torch.cuda.synchronize()
        replayed, pairs = run()
        assert replayed == 0, k
        assert np.array_equal(pairs, P.pj_self_join((chars, offs), 1)), k
        chars[k] = saved
        torch.cuda.synchronize()
    replayed, pairs = run()
    assert replayed == 1 and np.array_equal(pairs, first)
    plan.free()
