"""GPU: duqpp_group_error with a place for the partial sums of its mean gives the bits of the call without one, either side of the
size from which there are partial sums, with an odd number of groups and more workgroups than tokens, and the mean in pinned host memory
is the one in device memory."""
import pytest

import workloads as wl
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

ERR_ALIGN, ERR_WORKSPACE = -3, -5


@pytest.mark.parametrize("T,K,rotated", [(511, 4096, 1), (512, 4096, 1), (513, 4128, 1), (2100, 1024, 0), (70000, 32, 1), (5, 14368 * 32, 0), (10, 64, 1)])
def test_same_bits_with_and_without(T, K, rotated):
    import torch

    import paper_2604_17789_amd as duqpp
    from paper_2604_17789_amd.binding import _stream, lib
    name = f"gpu-gerr-ws-{T}-{K}"
    x = to_dev_bf16(wl.make_activations(name, T, K, (wl.OutlierSpec(1, 50.0),)), torch)
    R = to_dev(wl.make_rotation_blocks(name, K // 32), torch) if rotated else None
    n = lib.duqpp_group_error_workspace_bytes(T, K)
    assert (n > 0) == (T * (K // 32) >= 65536)
    ws = torch.randint(0, 256, (n + 24,), dtype=torch.uint8, device="cuda")
    tail = ws[n + 8:].clone()

    def call(workspace, nbytes, pinned=False):
        err = torch.full((T, K // 32), 9.0, device="cuda")
        mean = torch.full((1,), 9.0, dtype=torch.float64, **(dict(pin_memory=True) if pinned else dict(device="cuda")))
        st = lib.duqpp_group_error_ws(x.data_ptr(), T, K, K, R.data_ptr() if rotated else None, K // 32, err.data_ptr(), mean.data_ptr(),
                                      workspace, nbytes, _stream())
        torch.cuda.synchronize()
        return st, err, mean

    print(f"[group error] workspace T={T} K={K} rotated={rotated}", flush=True)
    want = call(None, 0)
    got = call(ws.data_ptr() + 8, n)                         # aligned to 8 bytes, no more
    assert want[0] == got[0] == 0
    assert torch.equal(want[1], got[1]) and torch.equal(want[2], got[2])
    assert torch.equal(ws[n + 8:], tail)                     # nothing behind the bytes it was told of
    for args in ((None, 0), (ws.data_ptr() + 8, n)):
        assert torch.equal(call(*args, pinned=True)[2], want[2].cpu())
    assert call(ws.data_ptr() + 4, n)[0] == ERR_ALIGN
    if n:
        assert call(ws.data_ptr(), n - 1)[0] == ERR_WORKSPACE
