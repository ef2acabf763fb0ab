"""Plans whose caller set no launch shape, on both sides of the lines that
pick one (lookups, the tables' size, pessimistic tables): the answers are
those of one lookup call per table, whose shape the caller sets."""

import numpy as np
import pytest

from gpu_util import say, to_dev, vals_dev
from paper_1712_09624_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("timed", [False, True], ids=["untimed", "timed"])
# tables, log2 buckets, lookups in all, mode
@pytest.mark.parametrize("nt,B,total,mode", [
    (3, 11, 1 << 18, "cuckoopp"), (3, 11, (1 << 18) + 1, "optimistic"), (3, 11, 300001, "both"),
    (2, 20, (1 << 18) + 130, "cuckoopp"), (1, 20, 1 << 18, "both"), (1, 20, 270000, "both"),
    (1, 19, 270000, "cuckoopp"), (2, 20, 2000001, "cuckoopp")])
def test_own_shape(nt, B, total, mode, timed):
    import torch
    from paper_1712_09624_amd.ckpp import DEFAULT_PLAN_LAUNCH, Plan, Table
    n = min(W.keys_at_load(B, 0.9), 200000)
    counts = [total // nt + (total % nt if i == 0 else 0) for i in range(nt)]
    offsets = np.concatenate([[0], np.cumsum(counts)[:-1]])
    tables, looks = [], []
    for i in range(nt):
        keys = W.distinct_five_tuples(n, 500 + i)
        t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0, timers=timed)
        vals = vals_dev(W.insertion_values(n, 7 * i))
        if timed:
            exp = to_dev((np.arange(n) % 3 * 300).astype(np.uint16).view(np.int16))
            t.insert_at(to_dev(keys), vals, exp, 0)
        else:
            t.insert(to_dev(keys), vals)
        t.set_lookup_launch(8, 1, 64, 0)
        tables.append(t)
        looks.append(to_dev(W.lookup_mix(keys, counts[i], 0.3, 40 + i)[0]))
    plan = Plan(tables, offsets, counts, [mode] * nt)
    assert plan.get_launch() == DEFAULT_PLAN_LAUNCH
    assert plan.info()["nitems"] == sum((c + 63) // 64 for c in counts)
    say(f"plan own shape tables={nt} B={B} lookups={total} mode={mode} timed={timed}")
    f, v = plan.lookup(torch.cat(looks), now=250 if timed else None)
    for i, t in enumerate(tables):
        wf, wv = t.lookup_at(looks[i], 250, mode) if timed else t.lookup(looks[i], mode)
        o, c = int(offsets[i]), counts[i]
        assert bool(wf.any()) and not bool(wf.all())
        assert torch.equal(f[o:o + c], wf) and torch.equal(v[o:o + c], wv)
    plan.close()
    for t in tables:
        t.close()
