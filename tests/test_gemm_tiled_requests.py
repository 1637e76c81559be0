"""The tiled product's requests are left to the compiler where they write registers, and awaited by hand where they write LDS,
which counts on the order it keeps them in.  The assembly it makes of the kernels is read here: between a request and the wait
that covers it no instruction may name one of its registers, and behind every barrier the tokens of the next K step have
arrived.  A load that writes registers from an asm statement would be unknown to the compiler until an asm statement waits for
it, so there is none in any source."""
import os
import re
import shutil
import subprocess

import pytest

from __graft_entry__ import CSRC, HIPCC_FLAGS, ROOT

SHAPES = 11


def _registers(token):
    m = re.match(r"^([va])\[(\d+):(\d+)\]$", token)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"^([va])(\d+)$", token)
    return {(m[1], int(m[2]))} if m else set()


def _touched(lines, per_step):
    """Instructions that name a register in flight or barriers passed too early, and the loads seen, walking the code with every
    loop run three times; per_step: transfers into LDS that one K step takes."""
    labels = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    queue, found, loads, taken, i = [], [], 0, {}, 0
    sent, barriers = 0, 0
    while i < len(lines):
        line, at = lines[i], i
        i += 1
        if line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        words = [w for w in re.split(r"[,\s]+", rest) if w]
        if op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", rest)
            if m:
                queue = queue[max(0, len(queue) - int(m[1])):]        # they complete in the order of their issue
            continue
        if op == "s_barrier":
            barriers += 1
            if sent - sum(not q for q in queue) < min(sent, barriers * per_step):
                found.append(f"barrier {barriers}")
        live = set().union(*queue)
        if any(_registers(w) & live for w in words):
            found.append(line)
        if op.startswith("buffer_load") and words[-1] == "lds":
            queue.append(set())
            sent += 1
        elif op.startswith("global_load"):
            queue.append(_registers(words[0]))
            loads += 1
        elif op.startswith(("global_store", "buffer_", "scratch_", "flat_")):
            assert op.startswith("global_store"), f"not expected in this kernel: {line}"
            queue.append(set())
        if op.startswith(("s_branch", "s_cbranch")) and labels.get(words[0], i) <= at and taken.get(at, 0) < 2:
            taken[at] = taken.get(at, 0) + 1
            i = labels[words[0]]
    return found, loads


def _transfers_per_step(name):
    """LDS-DMA transfers that a wave makes for one K step, from the template arguments in the kernel's name."""
    mt, _, _, w = (int(v) for v in re.search(r"ILb[01]ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi\d+E", name).groups())
    return mt * (4 // w) + (mt + w - 1) // w


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "gemm_tiled.s")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    subprocess.run(["hipcc"] + flags + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                                        os.path.join(CSRC, "gemm_tiled.hip"), "-o", out], check=True, capture_output=True)
    found, name = {}, None
    for line in open(out):
        m = re.match(r"^(_ZN5duqpp\S*gemm_tiled_kernel\S*):", line)
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
        found, loads = _touched(lines, _transfers_per_step(name))
        assert loads >= 40 and not found, (name, found[:5])


def test_the_reading_notices_a_wait_that_is_too_short(kernels):
    for name, lines in kernels.items():
        later = [re.sub(r"vmcnt\((\d+)\)", lambda m: f"vmcnt({int(m[1]) + 5})", l) for l in lines]
        assert _touched(later, _transfers_per_step(name))[0], name


def test_the_reading_notices_a_barrier_that_is_too_early(kernels):
    """The waits ahead of the barriers alone cover a K step less: the registers are still waited for, the tokens are not."""
    for name, lines in kernels.items():
        step = _transfers_per_step(name) + 5 * int(re.search(r"ILb[01]ELi\d+ELi(\d+)E", name)[1])
        later = [re.sub(r"vmcnt\((\d+)\)", lambda m: f"vmcnt({int(m[1]) + step})", l) if lines[i + 1:i + 2] == ["s_barrier"] else l
                 for i, l in enumerate(lines)]
        found = _touched(later, _transfers_per_step(name))[0]
        assert found and all(f.startswith("barrier") for f in found), (name, found[:5])


def test_no_asm_statement_loads_registers_it_does_not_wait_for():
    """The text of an asm statement with a load that writes registers also holds the wait for it."""
    for source in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, source)) as f:
            text = f.read()
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            code = m[1]
            if re.search(r"\b(?:global|buffer|flat|scratch|s|s_buffer)_load_|\bds_read", code) and not re.search(r"_load_lds|\blds\b", code):
                assert "s_waitcnt" in code, (source, code)
