"""The construction's search on few rows waits by hand, in front of its barrier, for what its waves have written to LDS, but not for the
reads behind that, whose number it counts on.  A wave's LDS accesses complete in order, so a wait for at most N outstanding covers the writes
where N or more accesses stand behind the last of them; the assembly that the compiler makes of the kernel is read for that here."""
import os
import re
import shutil
import subprocess

import pytest

from __graft_entry__ import CSRC, HIPCC_FLAGS, ROOT


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "construct.s")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    subprocess.run(["hipcc"] + flags + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                                        os.path.join(CSRC, "construct.hip"), "-o", out], check=True, capture_output=True)
    lines = [l.split(";")[0].strip().replace("\t", " ") for l in open(out)]
    at = next(i for i, l in enumerate(lines) if re.match(r"^_ZN5duqpp\S*construct_rows_kernel\S*:", l))
    end = next(i for i in range(at, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return [l for l in lines[at + 1:end] if l]


def uncovered(lines):
    """(Waits in front of a barrier that do not cover every LDS write ahead of them, all waits that leave something outstanding.)"""
    bad, seen = [], 0
    for i, line in enumerate(lines):
        m = re.match(r"s_waitcnt .*lgkmcnt\((\d+)\)", line)
        if not m or int(m[1]) == 0 or lines[i + 1:i + 2] != ["s_barrier"]:
            continue
        seen += 1
        behind = 0                                           # LDS accesses behind the last write, as far as the code is straight
        for l in reversed(lines[:i]):
            if l.startswith("ds_write") or l.endswith(":") or l.startswith(("s_branch", "s_cbranch")):
                break
            behind += l.startswith("ds_read")
        if behind < int(m[1]):
            bad.append((i, behind, line))
    return bad, seen


def test_the_wait_ahead_of_the_barrier_covers_what_was_written(kernel):
    bad, seen = uncovered(kernel)
    assert seen == 1 and not bad, bad


def test_the_reading_notices_a_read_too_few(kernel):
    at = next(i for i, l in enumerate(kernel) if "lgkmcnt(12)" in l)
    reads = [i for i in range(at) if kernel[i].startswith("ds_read")][-5:]
    assert uncovered([l for i, l in enumerate(kernel) if i not in reads])[0]
    assert uncovered(kernel[:at] + ["ds_write_b64 v0, v[0:1]"] + kernel[at:])[0]
