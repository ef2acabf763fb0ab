"""Lookups on a table whose caller set no launch shape, at the edges of the
rule that picks one from the batch size, the mode and the table's size.  The
stored values are the keys' insertion indexes and the inputs say which key
each lookup drew, so the answers are known without another table."""

import numpy as np
import pytest

from gpu_util import say, to_dev, u64, u8, vals_dev
from paper_1712_09624_amd import workload as W

pytestmark = pytest.mark.gpu

# log2 buckets, stored keys, batch sizes on both sides of each line
EDGES = [
    (15, 0.9, [1, 1 << 14, (1 << 14) + 1, 1 << 19, (1 << 19) + 1]),
    (16, 0.9, [(1 << 21), (1 << 21) + 1]),
    (17, 0.9, [1 << 18, (1 << 18) + 1, (1 << 21) + 1]),
    (22, 0.05, [1 << 18, (1 << 18) + 1, (1 << 21) + 65]),
    (24, 0.01, [1 << 17, (1 << 17) + 1, 1 << 18, (1 << 18) + 1]),
]


@pytest.mark.parametrize("timed", [False, True], ids=["untimed", "timed"])
@pytest.mark.parametrize("B,load,sizes", EDGES, ids=[f"B{e[0]}" for e in EDGES])
def test_auto_shape_edges(B, load, sizes, timed):
    from paper_1712_09624_amd.ckpp import DEFAULT_LAUNCH, Table
    n = W.keys_at_load(B, load)
    keys = W.distinct_five_tuples(n, 200 + B)
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0, timers=timed)
    if timed:
        exp = to_dev(np.full(n, 500, np.uint16).view(np.int16))
        t.insert_at(to_dev(keys), vals_dev(W.insertion_values(n)), exp, 0)
    else:
        t.insert(to_dev(keys), vals_dev(W.insertion_values(n)))
    for size in sizes:
        look, neg, idx = W.lookup_mix(keys, size, 0.3, 17 + B)
        want_v = np.where(neg, 0, idx).astype(np.uint64)
        dl = to_dev(look)
        for mode in ("cuckoopp", "both", "optimistic"):
            say(f"auto shape B={B} n={size} mode={mode} timed={timed}")
            f, v = t.lookup_at(dl, 400, mode) if timed else t.lookup(dl, mode)
            assert np.array_equal(u8(f), (~neg).astype(np.uint8)), (size, mode)
            assert np.array_equal(u64(v), want_v), (size, mode)
    assert t.get_lookup_launch() == DEFAULT_LAUNCH
    t.close()
