"""The package without its native module, or with one that another torch built: it imports, says so, and every call takes the Python
path."""
import os
import subprocess
import sys

import pytest

import __graft_entry__ as graft
from paper_2604_17789_amd import binding

USE = """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import paper_2604_17789_amd as duqpp
from paper_2604_17789_amd import binding
print([str(w.message) for w in seen if "_calls.so" in str(w.message)])
print(binding._calls is binding._NoCalls, duqpp.version())
import torch
x, b = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(8192, dtype=torch.uint8)
for call in [lambda: duqpp.rotq_gemm_tiled_packed(x, b, b, b, 4), lambda: duqpp.rotq_gemm_tiled(x, b, b, b, 4), lambda: duqpp.rotq_gemm(x, b, b, b),
             lambda: duqpp.rotate_quantize_tiled_packed(x, b), lambda: duqpp.rotate_quantize_tiled(x, b), lambda: duqpp.quantize_weights_tiled(x, b),
             lambda: duqpp.mxfp4_gemm_tiled(b, b, b, b, 4, 4, 64), lambda: duqpp.group_error(x, b)]:
    try:
        call()
        print("accepted")
    except TypeError as e:
        assert "must be a cuda tensor" in str(e)
print("all refused as ever")
"""


def run(first):
    env = dict(os.environ, PYTHONPATH=graft.ROOT)
    return subprocess.run([sys.executable, "-c", first + USE], cwd=graft.ROOT, env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


@pytest.mark.parametrize("first,why", [
    ("import sys; sys.modules['paper_2604_17789_amd._calls'] = None\n", "does not load"),
    ("import sys, types; m = types.ModuleType('c'); m.built_for = 'torch 1.0, Python 3.10'; sys.modules['paper_2604_17789_amd._calls'] = m\n",
     "was built for torch 1.0, Python 3.10"),
    ("import sys, types; sys.modules['paper_2604_17789_amd._calls'] = types.ModuleType('c')\n", "was built for something else"),
])
def test_imports_without_the_native_module(first, why):
    r = run(first)
    assert r.returncode == 0, r.stdout
    assert why in r.stdout and "\nTrue " in r.stdout and "all refused as ever" in r.stdout and "accepted" not in r.stdout


def test_with_it_nothing_is_said():
    r = run("")
    assert r.returncode == 0 and "[]\nFalse " in r.stdout, r.stdout
    assert binding._calls is not binding._NoCalls            # what the tests of the native path run


def test_a_build_without_its_compiler_leaves_no_older_module(tmp_path, capsys):
    out = tmp_path / "_calls.so"
    out.write_bytes(b"older")
    assert graft.build_calls(str(out), compiler="no-such-compiler") is False
    assert not out.exists() and "not built" in capsys.readouterr().out
