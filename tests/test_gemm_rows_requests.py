"""The product's form for row-major weights brings their codes by transfers into LDS, too: what test_gemm_tiled_requests.py reads in the
assembly of the tiled form holds for it, with four transfers more for a K step and only the scales in registers."""
import os
import re
import shutil
import subprocess

import pytest

from __graft_entry__ import CSRC, HIPCC_FLAGS, ROOT
from test_gemm_tiled_requests import _touched, _transfers_per_step

SHAPES = 7                               # those of 32 channels per wave


def _transfers(name):
    return _transfers_per_step(name) + 4


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "gemm_rows.s")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    subprocess.run(["hipcc"] + flags + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                                        os.path.join(CSRC, "gemm_tiled.hip"), "-o", out], check=True, capture_output=True)
    found, name = {}, None
    for line in open(out):
        m = re.match(r"^(_ZN5duqpp\S*gemm_rows_kernel\S*):", line)
        if m:
            name = m[1]
            found[name] = []
            continue
        line = line.split(";")[0].strip().replace("\t", " ")
        if line.startswith(".Lfunc_end"):
            name = None
        elif name and line and (not line.startswith(".") or line.endswith(":")):
            found[name].append(line)
    return found


def test_no_register_is_touched_while_its_request_is_in_flight(kernels):
    assert len(kernels) == 2 * SHAPES
    for name, lines in kernels.items():
        found, loads = _touched(lines, _transfers(name))
        assert loads >= 4 and not found, (name, found[:5])
        later = [re.sub(r"vmcnt\((\d+)\)", lambda m: f"vmcnt({int(m[1]) + 5})", l) for l in lines]
        assert _touched(later, _transfers(name))[0], name


def test_the_reading_notices_a_barrier_that_is_too_early(kernels):
    for name, lines in kernels.items():
        step = _transfers(name) + 1
        later = [re.sub(r"vmcnt\((\d+)\)", lambda m: f"vmcnt({int(m[1]) + step})", l) if lines[i + 1:i + 2] == ["s_barrier"] else l
                 for i, l in enumerate(lines)]
        found = _touched(later, _transfers(name))[0]
        assert found and all(f.startswith("barrier") for f in found), (name, found[:5])
