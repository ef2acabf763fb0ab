"""What device memory inserts take and keep, without a GPU: the library runs on
a stand-in for the HIP runtime (fake_hip.c) that reports every allocation and
can refuse large ones."""

import os
import subprocess
import sys

import pytest

from paper_1712_09624_amd import ckpp

HERE = os.path.dirname(os.path.abspath(__file__))
KICKS = 500
MB = 10**6

PROGRAM = """
import ctypes, os, sys
ctypes.CDLL(sys.argv[1], mode=os.RTLD_GLOBAL | os.RTLD_NOW)  # before the real runtime
from paper_1712_09624_amd import ckpp
lib = ckpp.load()
libc = ctypes.CDLL(None)
at = 1 << 20                      # an address nobody reads

def largest(n):
    libc.setenv(b"FAKE_HIP_LARGEST", str(n).encode(), 1)

def table(B, kicks):
    h = ctypes.c_void_p()
    assert lib.ckpp_create(ctypes.byref(h), B, 1, kicks, 0, 0) == ckpp.OK
    return h

def insert(h, n, status=at):
    print("insert", flush=True)
    print("rc", lib.ckpp_insert_batch(h, at, at, n, status, None, None), flush=True)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    fake = str(tmp_path_factory.mktemp("hip") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", fake,
                    os.path.join(HERE, "fake_hip.c")], check=True)

    def go(body, created=None):
        """[(allocations of the insert as (call, bytes, granted), its status)];
        the bytes of those after the first insert's end go to `created`."""
        out = subprocess.run([sys.executable, "-c", PROGRAM + body, fake], text=True, check=True,
                             capture_output=True, cwd=os.path.dirname(HERE)).stdout
        inserts = []
        for part in out.split("insert\n")[1:]:
            lines = [x.split() for x in part.splitlines()]
            end = next(i for i, x in enumerate(lines) if x[0] == "rc")
            if created is not None and not inserts:
                created += [int(n) for _, n, _ in lines[end + 1:]]
            inserts.append(([(c, int(n), ok == "ok") for c, n, ok in lines[:end]],
                            int(lines[end][1])))
        return inserts
    return go


@pytest.mark.parametrize("kicks", [0, 1, 100, KICKS, 4096])
@pytest.mark.parametrize("B", [1, 10, 13, 15, 17, 20, 24])
def test_path_scratch_follows_the_table(run, B, kicks):
    """An insert key by key keeps path arrays of an eighth of the table, at
    most 65536, and on small tables at least 1024 and at most 4096."""
    (allocs, rc), = run(f"insert(table({B}, {kicks}), 1000, None)")
    assert rc == ckpp.OK and len(allocs) == 1
    call, held, ok = allocs[0]
    path = 4 * max(4, (kicks + 3) // 4 * 4)
    share = (256 << B) // 8
    assert call == "malloc" and ok and held % path == 0
    assert held // path >= 1024
    assert held <= max(min(share, 65536 * path), 1024 * path,
                       min(4096 * path, (256 << B) * 4 // 3))


@pytest.mark.parametrize("B,bins", [(1, 0), (8, 0), (9, 16), (15, 512), (22, 1 << 14),
                                    (24, 1 << 14), (25, 0)])
def test_bin_counters_follow_the_table(run, B, bins):
    """Beside its buckets a table takes 1 KiB and a word per bin of its dense
    batches (seen by creating it between two inserts)."""
    (_, first), (_, second) = run(f"""
t = table(10, {KICKS})
insert(t, 1000)
u = table({B}, {KICKS})
insert(t, 1000)
""", created := [])
    assert first == second == ckpp.OK
    assert created == [256 << B, 1024 + 4 * bins]


def test_path_scratch_with_little_memory_left(run):
    """The buffer is halved where the device does not grant it; below the least
    it is an error, and the table works once there is memory again."""
    tight, none, again = run(f"""
t = table(20, {KICKS})
largest({10 * MB})
insert(t, 5000)
u = table(10, {KICKS})
largest({MB})
insert(u, 5000, None)
largest({10 * MB})
insert(u, 5000, None)
""")
    assert tight[1] == ckpp.OK
    sizes = [n for _, n, _ in tight[0]]
    assert sizes == sorted(sizes, reverse=True) and len(sizes) > 1
    assert [ok for _, _, ok in tight[0]] == [False] * (len(sizes) - 1) + [True]
    assert none[1] == ckpp.ENOMEM
    assert again[1] == ckpp.OK and again[0][0][2]


def test_bins_of_dense_batches_are_bounded(run):
    """Tables keep the bins of their dense batches up to 1/64 of the device's
    288 GiB in all; beyond it a batch takes them from the pool, or does without
    when it is small, and a destroyed table's share is free again."""
    got = run(f"""
ts = [table(22, {KICKS}) for _ in range(10)]
for t in ts:
    insert(t, 1 << 24)
insert(ts[0], 1 << 24)
s = table(20, {KICKS})
insert(s, 1 << 21)
lib.ckpp_destroy(ts[0])
insert(s, 1 << 21)
""")
    assert all(rc == ckpp.OK for _, rc in got)
    bins = (256 << 22) * 5 // 8
    kept = [a[1:] for a, _ in got[:10]]  # after the path scratch
    room = (288 << 30) // 64 // bins
    assert [c for a in kept for c, n, _ in a if c == "malloc" and n == bins] == ["malloc"] * room
    assert all([c for c, _, _ in a] == ["pool"] and a[0][1] <= bins for a in kept[room:])
    assert got[10][0] == []                                   # its bins were kept
    assert [c for c, _, _ in got[11][0]] == ["malloc"]        # path scratch alone
    assert got[12][0] == [("malloc", (256 << 20) * 5 // 8, True)]
