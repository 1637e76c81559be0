"""CPU-only checks of the binding's short cuts: they answer as the calls they stand in for, and it works without them."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2604_17789_amd as duqpp


def _by_the_library(rows, K):
    cb, sb = ctypes.c_size_t(0), ctypes.c_size_t(0)
    status = duqpp.lib.duqpp_tiled_bytes(rows, K, ctypes.byref(cb), ctypes.byref(sb))
    return (cb.value, sb.value) if status == 0 else status


@pytest.mark.parametrize("rows,K", [(1, 32), (33, 64), (32, 256), (32, 288), (7, 14368), (1 << 30, 1 << 30), (True, 64),
                                    (np.int64(33), 64), (33, np.int32(64)), (np.int32(1 << 30), np.int32(1 << 30)),
                                    (0, 64), (33, 48), (33, 0), ((1 << 30) + 1, 64), (33, (1 << 30) + 32),
                                    (32.0, 64), (32, 64.0), (np.float32(3), 64), ("1", 64), (None, 64)])
def test_tiled_bytes_is_the_library_s_answer(rows, K):
    """Python integers whatever kind of integer comes in, and what the C call refuses is refused."""
    try:
        want = _by_the_library(rows, K)
    except ctypes.ArgumentError as e:
        want = type(e)
    if isinstance(want, tuple):
        got = duqpp.tiled_bytes(rows, K)
        assert got == want and all(type(v) is int for v in got)
    else:
        with pytest.raises(want if isinstance(want, type) else duqpp.binding.DuqppError):
            duqpp.tiled_bytes(rows, K)


@pytest.mark.parametrize("missing", ["_cuda_getDevice", "_cuda_getCurrentRawStream"])
def test_the_stream_without_torch_s_private_names(missing):
    """The package imports where torch lacks them and asks for the stream the public way."""
    code = f"""
import torch
if hasattr(torch._C, {missing!r}):
    delattr(torch._C, {missing!r})
from paper_2604_17789_amd import binding
torch.cuda.current_stream = lambda: type("Stream", (), {{"cuda_stream": 4711}})
assert binding._stream() == 4711
"""
    subprocess.run([sys.executable, "-c", code], check=True, timeout=300,
                   cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
