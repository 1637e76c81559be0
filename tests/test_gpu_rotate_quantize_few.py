"""GPU: the tiled rotate + quantise of few tokens (a wave per block and token tile) gives the bytes of the row-major kernel in their
tiled places: ragged token tiles, groups that the layout pads, strided rows, a shared block, and either side of the numbers of
waves up to which it is taken.  Likewise the kernel beyond them where rows are short."""
import numpy as np
import pytest

import workloads as wl
from helpers import to_dev, untile_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,shared", [(1, 32, 0), (1, 4096, 0), (31, 96, 1), (32, 288, 0), (33, 14336, 0), (65, 8224, 1),
                                        (512, 4096, 0), (513, 4096, 0),          # 2048 and 2176 waves: packed blocks
                                        (1024, 4096, 1), (1025, 4096, 0),        # 4096 and 4224: fp32 blocks
                                        # rows below 2048 channels, where an XCD has token runs: 4 waves per workgroup, 5 and groups that
                                        # the layout pads, 4 and a ring of three tiles for one group
                                        (8200, 1024, 0), (8200, 1120, 1), (70000, 32, 0)])
def test_same_bytes_as_the_row_major_kernel(T, K, shared):
    import torch

    import paper_2604_17789_amd as duqpp
    name = f"gpu-few-{T}-{K}"
    g = torch.Generator(device="cuda").manual_seed(T * 31 + K)
    x = torch.randn((T, K + 16), generator=g, device="cuda").to(torch.bfloat16)[:, :K]
    x[T // 2, :32] = 0                                       # a group without a magnitude
    x[:, K - 1] *= 900
    R = to_dev(wl.make_rotation_blocks(name, 1 if shared else K // 32), torch)
    print(f"[rotate few] T={T} K={K} shared={shared}", flush=True)
    codes, scales = duqpp.rotate_quantize(x, R)
    n = duqpp.tiled_bytes(T, K)
    for blocks, call in ((R, duqpp.rotate_quantize_tiled), (duqpp.pack_rotation(R), duqpp.rotate_quantize_tiled_packed)):
        out = [torch.full((m + 256,), 0xA5, dtype=torch.uint8, device="cuda") for m in n]
        ct, st = call(x, blocks, out=tuple(o[:m] for o, m in zip(out, n)))
        torch.cuda.synchronize()
        c, s, pad_c, pad_s = untile_np(ct.cpu().numpy(), st.cpu().numpy(), T, K)
        np.testing.assert_array_equal(c, codes.cpu().numpy())
        np.testing.assert_array_equal(s, scales.cpu().numpy())
        assert np.all(pad_c == 0) and np.all(pad_s == 127)   # every byte of the padding, too
        assert all(torch.all(o[m:] == 0xA5) for o, m in zip(out, n))


@pytest.mark.parametrize("T,K,N", [(1, 32, 8), (33, 288, 70), (64, 1024, 9000), (512, 4096, 100), (513, 4096, 33),
                                   (1, 32, 32 * 8192), (40, 32, 32 * 8192 + 1), (3, 64, 32 * 32768 + 70)])
def test_beside_the_retiling_of_the_weights(T, K, N):
    """The row-major call, which rotates in the launch that re-tiles its weights: bit for bit the tiled call, either side of 2048
    waves, with a row tile of weights that is mostly padding and with more of them than tokens, and either side of 8192 units of weights
    (workgroups of one wave and of four) and of 32768 (a wave per unit and several units)."""
    import torch

    import paper_2604_17789_amd as duqpp
    g = torch.Generator(device="cuda").manual_seed(T + K + N)
    x = torch.randn((T, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    R = to_dev(wl.make_rotation_blocks(f"gpu-few-row-{K}", K // 32), torch)
    print(f"[rotate few] row-major T={T} K={K} N={N}", flush=True)
    ws = torch.full((duqpp.gemm_workspace_bytes(T, N, K, True),), 0xA5, dtype=torch.uint8, device="cuda")
    y = duqpp.rotq_gemm(x, R, *duqpp.quantize_weights(w, R), workspace=ws)
    wt = duqpp.quantize_weights_tiled(w, R)
    want = duqpp.rotq_gemm_tiled(x, R, *wt, N)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    at = 0                                                   # every byte of both operands, the padding's too
    for part in duqpp.rotate_quantize_tiled(x, R) + wt:
        assert torch.equal(ws[at:at + part.numel()], part)
        at += part.numel()
