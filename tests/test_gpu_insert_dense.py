"""Dense insert batches: enough keys per bucket that the batch is binned by
primary bucket and placed range by range, the rest by the per-key path.  The
dictionary is known from the inputs (values and expiration times are ours),
the statuses are those of the same batch taken key by key, and the image
passes the oracle's invariant checker."""

import numpy as np
import pytest

from gpu_util import say, to_dev, u64, u8, vals_dev
from oracle import oracle as O
from paper_1712_09624_amd import workload as W

pytestmark = pytest.mark.gpu


def insert(t, keys, vals, exp=None, now=0):
    if exp is None:
        return t.insert(to_dev(keys), vals_dev(vals))
    return t.insert_at(to_dev(keys), vals_dev(vals), to_dev(exp.view(np.int16)), now)


# log2 buckets, keys of the first and the second batch as shares of the slots:
# one bin and many, at and below the least keys per bucket (0.25), and more
# keys than the slots, which the per-key path takes
@pytest.mark.parametrize("timed", [False, True], ids=["untimed", "timed"])
@pytest.mark.parametrize("B,first,second", [(9, 1.0, 0.0), (11, 0.25, 0.7), (11, 0.2499, 0.7),
                                            (12, 0.6, 0.35), (15, 0.5, 0.45), (17, 0.3, 0.65),
                                            (11, 1.01, 0.0)])
def test_dense_batches(B, first, second, timed):
    """Two batches; the second also rewrites half of the first's keys."""
    from paper_1712_09624_amd.ckpp import Table
    slots = 8 << B
    n1, n2 = int(first * slots), int(second * slots)
    keys = W.distinct_five_tuples(n1 + n2, 400 + B)
    vals = W.insertion_values(n1 + n2, 3)
    exp = np.full(n1 + n2, 800, np.uint16) if timed else None
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0, timers=timed)
    say(f"dense B={B} n={n1} timed={timed}")
    st, nf = insert(t, keys[:n1], vals[:n1], None if exp is None else exp[:n1])
    st1 = u8(st)
    assert set(np.unique(st1)) <= {O.INSERTED, O.FAILED}
    assert int(nf.item()) == int((st1 == O.FAILED).sum())
    if first <= 0.97:
        assert not st1.any()
    if n2:
        rows = np.r_[W.choose_rows(n1, n1 // 2, 7), np.arange(n1, n1 + n2)]
        rows = rows[np.argsort(W.raw_u64(11, 0, len(rows)))]  # updates and new keys mixed
        v2 = vals[rows] + np.uint64(10**9)
        say(f"dense B={B} second batch n={len(rows)}")
        st, nf = insert(t, keys[rows], v2, None if exp is None else exp[rows])
        assert int(nf.item()) == 0
        assert np.array_equal(u8(st), np.where(rows < n1, O.UPDATED, O.INSERTED).astype(np.uint8))
        vals[rows] = v2
    live = np.r_[st1 == O.INSERTED, np.ones(n2, bool)]
    probe = np.concatenate([keys, W.five_tuples(5000, 9)])
    f, v = t.lookup_at(to_dev(probe), 100) if timed else t.lookup(to_dev(probe))
    assert np.array_equal(u8(f), np.r_[live, np.zeros(5000, bool)].astype(np.uint8))
    assert np.array_equal(u64(v)[: n1 + n2], np.where(live, vals, 0).astype(np.uint64))
    b, k = t.export()
    rc, msg = O.check_image(b, k, B, W.HASH_SEED, timed=timed)
    assert rc == 0, f"invariant {rc}: {msg}"
    s = t.stats()
    assert s["live"] == int(live.sum()) and s["locked"] == 0 and s["retry_exhausted"] == 0
    t.close()


def test_dense_timed_expired_and_wide():
    """On a table with timers a dense batch overwrites expired copies of its
    keys in place (INSERTED), rewrites alive ones (UPDATED), takes expired
    entries' slots, and fails the keys whose values are too wide."""
    from paper_1712_09624_amd.ckpp import Table
    B = 12
    n = W.keys_at_load(B, 0.9)
    keys = W.distinct_five_tuples(2 * n, 430)
    exp = np.where(np.arange(n) % 2 == 0, 50, 900).astype(np.uint16)
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0, timers=True)
    st, _ = insert(t, keys[:n], W.insertion_values(n), exp)
    assert not u8(st).any()
    now = 100  # the even keys have expired
    # a third of the old keys, and new ones for most of the expired slots
    rows = np.r_[np.arange(0, n, 3), np.arange(n, n + int(0.3 * n))]
    vals = W.insertion_values(len(rows), 7000)
    wide = np.arange(len(rows)) % 17 == 0
    vals[wide] += np.uint64(1 << 48)
    say(f"dense timed n={len(rows)} now={now}")
    st, nf = insert(t, keys[rows], vals, np.full(len(rows), 1000, np.uint16), now)
    want = np.where(wide, O.FAILED,
                    np.where((rows < n) & (rows % 2 == 1), O.UPDATED, O.INSERTED))
    assert np.array_equal(u8(st), want.astype(np.uint8))
    assert int(nf.item()) == int(wide.sum())
    f, v = t.lookup_at(to_dev(keys), now)
    want_f = np.r_[np.arange(n) % 2 == 1, np.zeros(n, bool)]
    want_v = np.r_[W.insertion_values(n), np.zeros(n, np.uint64)]
    want_f[rows[~wide]] = True
    want_v[rows[~wide]] = vals[~wide]
    assert np.array_equal(u8(f), want_f.astype(np.uint8))
    assert np.array_equal(u64(v), np.where(want_f, want_v, 0))
    b, k = t.export()
    rc, msg = O.check_image(b, k, B, W.HASH_SEED, timed=True)
    assert rc == 0, f"invariant {rc}: {msg}"
    t.close()


def test_dense_batch_in_a_graph():
    """A dense batch captured and replayed, with deletes between the replays:
    every replay inserts the whole batch again."""
    import torch
    from paper_1712_09624_amd.ckpp import Table
    B = 11
    n = W.keys_at_load(B, 0.8)
    keys, vals = to_dev(W.distinct_five_tuples(n, 440)), vals_dev(W.insertion_values(n))
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0)
    st = torch.empty(n, dtype=torch.uint8, device="cuda:0")
    nf = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    t.insert(keys, vals, status=st, nfailed=nf)  # allocates the table's buffers
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        t.insert(keys, vals, status=st, nfailed=nf)
    for rep in range(3):
        gone = t.delete(keys[rep * 100:])
        assert int(gone.sum()) == n - rep * 100
        st.fill_(9)
        say(f"dense insert replay {rep}")
        g.replay()
        torch.cuda.synchronize()
        want = np.zeros(n, np.uint8)
        want[: rep * 100] = O.UPDATED
        assert np.array_equal(u8(st), want)
        f, v = t.lookup(keys)
        assert bool(f.all()) and torch.equal(v, vals)
    assert int(nf.item()) == 0
    t.close()


@pytest.mark.parametrize("timed", [False, True], ids=["untimed", "timed"])
@pytest.mark.parametrize("B,top", [(11, False), (11, True), (16, True)],
                         ids=["B11_first_bins", "B11_last_bins", "B16_last_bins"])
def test_dense_full_bins(B, top, timed):
    """All primaries in one eighth of the buckets, the first or the last: eight
    times a bin's mean, so that most keys find their bin full.  Then a uniform
    batch with half of those keys again, whose bins start empty."""
    from paper_1712_09624_amd.ckpp import Table
    nb, n = 1 << B, 2 << B
    drawn = W.distinct_five_tuples(9 * n, 460 + B)
    p = O.hash_keys(drawn, W.HASH_SEED) & np.uint64(nb - 1)
    here = (p >= nb - nb // 8) if top else (p < nb // 8)
    keys, fresh = drawn[here][:n], drawn[~here][:n]
    assert len(keys) == len(fresh) == n
    vals = W.insertion_values(2 * n, 5)
    exp = np.full(2 * n, 700, np.uint16) if timed else None
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0, timers=timed)
    say(f"dense full bins B={B} n={n} top={top} timed={timed}")
    st, nf = insert(t, keys, vals[:n], None if exp is None else exp[:n])
    assert not u8(st).any() and int(nf.item()) == 0
    both = np.concatenate([keys, fresh])
    rows = np.r_[W.choose_rows(n, n // 2, 8), np.arange(n, 2 * n)]
    rows = rows[np.argsort(W.raw_u64(12, 0, len(rows)))]
    vals[rows] += np.uint64(10**9)
    say(f"dense uniform B={B} n={len(rows)}")
    st, nf = insert(t, both[rows], vals[rows], None if exp is None else exp[rows])
    assert int(nf.item()) == 0
    assert np.array_equal(u8(st), np.where(rows < n, O.UPDATED, O.INSERTED).astype(np.uint8))
    f, v = t.lookup_at(to_dev(both), 100) if timed else t.lookup(to_dev(both))
    assert u8(f).all() and np.array_equal(u64(v), vals)
    b, k = t.export()
    rc, msg = O.check_image(b, k, B, W.HASH_SEED, timed=timed)
    assert rc == 0, f"invariant {rc}: {msg}"
    s = t.stats()
    assert s["live"] == 2 * n and s["locked"] == 0 and s["retry_exhausted"] == 0
    t.close()


@pytest.mark.parametrize("apart", [1, 7, 64, 4096])
@pytest.mark.parametrize("B,copies", [(11, 2), (13, 3)])
def test_dense_repeated_keys(B, copies, apart):
    """Every key `copies` times in one dense batch, its copies `apart` keys
    from each other: one of them is INSERTED, the others are UPDATED, and the
    table holds one entry with the value of one of them."""
    from paper_1712_09624_amd.ckpp import Table
    n = ((8 << B) // (2 * copies) // apart + 1) * apart
    once = W.distinct_five_tuples(n, 500 + B)
    at = np.repeat(np.arange(n).reshape(-1, apart), copies, axis=0).reshape(-1)
    vals = W.insertion_values(n * copies, 3)
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0)
    say(f"dense repeated B={B} copies={copies} apart={apart} n={n * copies}")
    st, nf = insert(t, once[at], vals)
    st = u8(st)
    assert int(nf.item()) == 0
    assert np.array_equal(np.bincount(at[st == O.INSERTED], minlength=n), np.ones(n, int))
    assert int((st == O.UPDATED).sum()) == n * (copies - 1)
    f, v = t.lookup(to_dev(once))
    assert u8(f).all()
    of_key = vals[np.argsort(at, kind="stable")].reshape(n, copies)
    assert (of_key == u64(v)[:, None]).any(axis=1).all()
    b, k = t.export()
    rc, msg = O.check_image(b, k, B, W.HASH_SEED)
    assert rc == 0, f"invariant {rc}: {msg}"
    assert t.stats()["live"] == n
    t.close()


@pytest.mark.parametrize("B,n", [(19, (2 << 19) - 1), (19, 2 << 19), (20, (1 << 20) - 1),
                                 (20, 1 << 20), (22, 2 << 22), (23, (1 << 23) + 1),
                                 (24, 1 << 24), (24, (3 << 24) + 5)])
def test_dense_large_tables(B, n):
    """The least keys per bucket on each side of 2^20 buckets, and the largest
    bin counts (2^14 bins of 2^8, 2^9 and 2^10 buckets); keys drawn on the
    device."""
    import torch

    from paper_1712_09624_amd.ckpp import Table
    g = torch.Generator(device="cuda").manual_seed(B)
    keys = torch.randint(-(1 << 63), (1 << 63) - 1, (n, 2), dtype=torch.int64, device="cuda",
                         generator=g).view(torch.uint8)
    vals = torch.arange(n, dtype=torch.int64, device="cuda") * 3 + 1
    t = Table(B, W.HASH_SEED, W.MAX_KICKS, device=0)
    say(f"dense large B={B} n={n}")
    st, nf = t.insert(keys, vals)
    assert int(nf.item()) == 0 and not bool(st.any())
    s = t.stats()
    assert s["live"] == n and s["locked"] == 0 and s["retry_exhausted"] == 0
    f, v = t.lookup(keys)
    assert bool(f.all()) and torch.equal(v, vals)
    gone = t.delete(keys)
    assert bool(gone.all())
    s = t.stats()
    assert s["live"] == 0 and s["bloom_pc_sum"] == 0
    t.close()
