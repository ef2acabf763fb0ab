"""The wait that closes a critical section: on every way from a read of an
entry's value word (its time, on a table with timers) to the store that drops
the bucket's lock, the compiled code passes the section's full wait.  Without
it the lock's next holder could write the word before the read is performed.
Checked on the gfx950 assembly of the device functions, compiled here."""

import os
import re
import shutil
import subprocess

import pytest

from paper_1712_09624_amd import build

SOURCE = r"""
#include "ckpp_update_dev.h"
namespace ckpp {
__global__ void section(uint8_t *bk, const uint4 *keys, int *out, uint32_t log2b, uint64_t seed,
                        uint32_t now) {
  const uint4 key = keys[threadIdx.x];
  bool pair = false;
  const KeyFields f = key_fields(key_hash(key, seed), log2b);
  out[threadIdx.x] = delete_direct<WITH_TIMES>(bk, key, f, false, now, pair);
}
}  // namespace ckpp
"""

VALUE_LOAD = re.compile(r"global_load_dwordx2 .* sc1")
UNLOCK = re.compile(r"global_store_dword(x2 .* offset:24| .* offset:28) sc1")
FULL_WAIT = "s_waitcnt vmcnt(0) expcnt(0) lgkmcnt(0)"


def instructions(asm):
    """The kernel's instructions, and the index each label stands at."""
    body = asm[re.search(r"^_ZN4ckpp7section\w*:", asm, re.M).end():]
    body = body[:body.index(".Lfunc_end")]
    code, labels = [], {}
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        m = re.fullmatch(r"(\.L\w+):", line)
        if m:
            labels[m.group(1)] = len(code)
        elif line and not line.startswith((".", "//")):
            code.append(re.sub(r"\s+", " ", line))
    return code, labels


def unwaited(code, labels):
    """(value load, unlock) pairs that a way without the full wait connects."""
    bad = []
    for start in [i for i, c in enumerate(code) if VALUE_LOAD.match(c)]:
        seen, todo = set(), [start + 1]
        while todo:
            i = todo.pop()
            while i < len(code) and i not in seen:
                seen.add(i)
                c = code[i]
                if c == FULL_WAIT or c.startswith("s_endpgm"):
                    break
                if UNLOCK.match(c):
                    bad.append((code[start], c))
                    break
                m = re.match(r"s_(c?)branch\w* (\.L\w+)", c)
                if m:
                    todo.append(labels[m.group(2)])
                    if not m.group(1):
                        break
                i += 1
    return bad


@pytest.mark.parametrize("timed", [False, True], ids=["untimed", "timed"])
def test_delete_waits_for_the_time_it_read(tmp_path, timed):
    if not (shutil.which(build.hipcc()) or os.path.exists(build.hipcc())):
        pytest.skip("no hipcc")
    src, out = tmp_path / "section.hip", tmp_path / "section.s"
    src.write_text(SOURCE)
    subprocess.run([build.hipcc(), f"--offload-arch={build.ARCH}", "-O3", "-std=c++17",
                    f"-DWITH_TIMES={'true' if timed else 'false'}", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I", build.INCLUDE, "-I", build.CSRC,
                    "--cuda-device-only", "-S", str(src), "-o", str(out)],
                   check=True, capture_output=True)
    code, labels = instructions(out.read_text())
    assert any(UNLOCK.match(c) for c in code)
    assert any(VALUE_LOAD.match(c) for c in code) == timed
    assert unwaited(code, labels) == []
