"""The row-major fused call prepares both operands in one launch: every byte it leaves in the workspace, at the edges of the
units (32 rows x 8 groups), with a wave per block and token tile and beyond 2048 of these with rings of both depths, four and more
waves per workgroup and both orders of the workgroups, and with more units than waves."""
import numpy as np
import pytest

import workloads as wl
from helpers import tile_np, to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,K,shift", [
    (1, 33, 32, 0),             # one group; a row tile of one row
    (45, 100, 352, 0),          # 11 groups: scale rows that are not whole words
    (64, 64, 1024, 1),          # scales that do not start on a word
    (33, 31, 288, 3),
    (300, 200, 14336, 0),       # 4480 blocks and token tiles: the ring, five waves per workgroup
    (2048, 40, 4096, 0),        # four waves per workgroup
    (4100, 40, 4096, 0),        # the deeper ring
    (2100, 70, 1120, 2),        # rows below 2048 channels
    (1, 12000, 8192, 0),        # a wave per block and token tile, 12000 units in workgroups of four waves
    (513, 65573, 4096, 0),      # the ring, four waves per workgroup, 32800 units: several per wave
])
def test_workspace_of_the_rowmajor_call(T, N, K, shift):
    import torch

    import paper_2604_17789_amd as duqpp
    rng = np.random.default_rng(T + N + K)
    codes = rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8)
    scales = rng.integers(118, 137, size=(N, K // 32)).astype(np.uint8)
    x = to_dev_bf16(wl.make_activations(f"rm-{T}-{K}", T, K, (wl.OutlierSpec(4, 50.0),)), torch)
    R = to_dev(wl.make_rotation_blocks(f"rm-{K}", K // 32), torch)
    bc = to_dev(codes, torch)
    store = torch.zeros(scales.size + shift, dtype=torch.uint8, device="cuda")
    bs = store[shift:].view(N, K // 32)
    bs.copy_(to_dev(scales, torch))
    ws = torch.full((duqpp.gemm_workspace_bytes(T, N, K, True),), 0xA5, dtype=torch.uint8, device="cuda")
    print(f"[row-major call] T={T} N={N} K={K} shift={shift}", flush=True)
    y = duqpp.rotq_gemm(x, R, bc, bs, workspace=ws)
    a = duqpp.rotate_quantize_tiled(x, R)
    ct, st = tile_np(codes, scales)
    want = duqpp.mxfp4_gemm_tiled(*a, to_dev(ct, torch), to_dev(st, torch), T, N, K)
    torch.cuda.synchronize()
    at = 0
    for part in (a[0].cpu().numpy(), a[1].cpu().numpy(), ct, st):       # every part is a multiple of 256 bytes
        np.testing.assert_array_equal(ws[at:at + part.size].cpu().numpy(), part.reshape(-1))
        at += part.size
    assert torch.equal(y, want)
