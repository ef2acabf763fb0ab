"""The counters that inserts and scans make for themselves: each call returns
its own, starting from zero, on the null stream (where they come from a block
cleared together), on another stream and under capture."""

import numpy as np
import pytest

from gpu_util import say, to_dev, vals_dev
from paper_1712_09624_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [False, True], ids=["null_stream", "side_stream"])
def test_counters_are_each_calls_own(side):
    """A 2-bucket table holds 16 of 16 + k keys: call k fails k of them.  More
    calls than a block has words, the counters kept to the end."""
    import torch
    from paper_1712_09624_amd import ckpp
    from paper_1712_09624_amd.ckpp import Table
    calls = ckpp._ZERO_WORDS + 40
    keys, vals = to_dev(W.distinct_five_tuples(24, 5)), vals_dev(W.insertion_values(24))
    t = Table(1, W.HASH_SEED, W.MAX_KICKS, device=0)
    torch.cuda.synchronize()
    s = torch.cuda.Stream() if side else torch.cuda.default_stream()
    got = []
    say(f"{calls} overfull inserts, side stream {side}")
    with torch.cuda.stream(s):
        for c in range(calls):
            t.clear()
            n = 16 + c % 9
            got.append(t.insert(keys[:n], vals[:n])[1])
            if c % 50 == 0:
                got[-1].add_(1000)  # the caller's own tensor: no other call sees this
    torch.cuda.synchronize()
    want = np.array([c % 9 + (1000 if c % 50 == 0 else 0) for c in range(calls)])
    assert np.array_equal(torch.cat(got).cpu().numpy(), want)
    t.close()


def test_counter_under_capture():
    """A captured insert clears its counter at every replay."""
    import torch
    from paper_1712_09624_amd.ckpp import Table
    keys, vals = to_dev(W.distinct_five_tuples(20, 5)), vals_dev(W.insertion_values(20))
    t = Table(1, W.HASH_SEED, W.MAX_KICKS, device=0)
    t.insert(keys, vals)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        t.clear()
        _, nf = t.insert(keys, vals)
    for rep in range(3):
        say(f"captured overfull insert, replay {rep}")
        g.replay()
        torch.cuda.synchronize()
        assert int(nf.item()) == 4
        t.insert(keys[:4], vals[:4])
    t.close()


def test_scan_counters():
    import torch
    from paper_1712_09624_amd.ckpp import Table
    keys, vals = to_dev(W.distinct_five_tuples(600, 6)), vals_dev(W.insertion_values(600))
    exp = to_dev((np.arange(600) % 3 * 100).astype(np.uint16).view(np.int16))
    t = Table(8, W.HASH_SEED, W.MAX_KICKS, device=0, timers=True)
    t.insert_at(keys, vals, exp, 0)
    say("scans")
    gone = [t.expire_scan(now) for now in (50, 50, 150, 250)]
    torch.cuda.synchronize()
    assert [int(x.item()) for x in gone] == [200, 0, 200, 200]
    t.close()


def test_null_stream_call_while_a_side_stream_is_current():
    """A call that names the null stream while a busy side stream is current
    leaves nothing behind that later calls on the null stream count in."""
    import torch
    from paper_1712_09624_amd.ckpp import Table
    keys, vals = to_dev(W.distinct_five_tuples(20, 5)), vals_dev(W.insertion_values(20))
    st = torch.empty(20, dtype=torch.uint8, device="cuda:0")
    t = Table(1, W.HASH_SEED, W.MAX_KICKS, device=0)
    t.insert(keys, vals)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    say("inserts that name the null stream while a side stream is current")
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        first = [t.insert(keys, vals, status=st, stream=s)[1]
                 for s in (0, torch.cuda.default_stream())]
    got = [t.insert(keys, vals)[1] for _ in range(20)]
    torch.cuda.synchronize()
    assert [int(x.item()) for x in got] == [4] * 20
    assert len(first) == 2
    t.close()
