"""The kernels of the tiled product that spread token row tiles evenly hold two bodies, for MT and MT - 1 of them.  Their assembly is
read as that of the others is: no register named between its request and the wait that covers it, and the next K step's tokens
there behind every barrier, in each body."""
import os
import re
import shutil
import subprocess

import pytest

from __graft_entry__ import CSRC, HIPCC_FLAGS, ROOT
from test_gemm_tiled_requests import _touched


def _bodies(lines):
    """The code of the two bodies: the branch ahead of the first barrier that leads farthest, by way of another branch or not."""
    labels = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}

    def end(label):
        i = labels[label]
        while lines[i].endswith(":"):
            i += 1
        while lines[i].startswith("s_mov"):                  # nothing but registers set on the way
            i += 1
        return end(lines[i].split()[-1]) if lines[i].startswith(("s_branch", "s_cbranch_execnz")) else labels[label]

    first = lines.index("s_barrier")
    leads = {i: end(l.split()[-1]) for i, l in enumerate(lines[:first]) if l.startswith("s_cbranch_scc")}
    at = max(leads, key=leads.get)
    return lines[at + 1:leads[at]], lines[leads[at]:]


def _arguments(name):
    return (int(v) for v in re.search(r"ILb[01]ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi\d+E", name).groups())


def _transfers(mt, w):
    return mt * (4 // w) + (mt + w - 1) // w


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "gemm_tiled.s")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    subprocess.run(["hipcc"] + flags + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                                        os.path.join(CSRC, "gemm_tiled.hip"), "-o", out], check=True, capture_output=True)
    kernels, name = {}, None
    for line in open(out):
        m = re.match(r"^(_ZN5duqpp\S*gemm_spread_kernel\S*):", line)
        if m:
            name = m[1]
            kernels[name] = []
            continue
        line = line.split(";")[0].strip().replace("\t", " ")
        if line.startswith(".Lfunc_end"):
            name = None
        elif name and line and (not line.startswith(".") or line.endswith(":")):
            kernels[name].append(line)
    assert len(kernels) == 10
    found = []
    for name, lines in kernels.items():
        mt, nt, d, w = _arguments(name)
        two = sorted(_bodies(lines), key=lambda b: -sum(l.startswith("v_mfma") for l in b))
        for m, body in zip((mt, mt - 1), two):
            # the products of four quarters of D steps, in the loop and behind it
            assert sum(l.startswith("v_mfma") for l in body) == 8 * d * m * nt, (name, m)
            found.append((name, m, _transfers(m, w), _transfers(m, w) + 5 * nt, body))
    return found


def test_no_register_is_touched_while_its_request_is_in_flight(bodies):
    for name, m, transfers, _, body in bodies:
        found, loads = _touched(body, transfers)
        assert loads >= 40 and not found, (name, m, found[:5])


def test_the_reading_notices_waits_that_are_too_short(bodies):
    for name, m, transfers, step, body in bodies:
        later = [re.sub(r"vmcnt\((\d+)\)", lambda k: f"vmcnt({int(k[1]) + 5})", l) for l in body]
        assert _touched(later, transfers)[0], (name, m)
        later = [re.sub(r"vmcnt\((\d+)\)", lambda k: f"vmcnt({int(k[1]) + step})", l) if body[i + 1:i + 2] == ["s_barrier"] else l
                 for i, l in enumerate(body)]
        found = _touched(later, transfers)[0]
        assert found and all(f.startswith("barrier") for f in found), (name, m, found[:5])
