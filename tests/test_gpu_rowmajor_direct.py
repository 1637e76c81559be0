"""The row-major fused call where the product takes the weights, or their codes, as they are: the bits of the product on tiled weights, in every
kernel that does it, with fewer and more K steps than are in flight; and where it may not, they are re-tiled into the workspace as
before."""
import numpy as np
import pytest

import workloads as wl
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

# half row tiles on the 16-row and the 32-row instruction, whole ones, two token row tiles at once; 9 and 17 K steps (waves with fewer)
AS_THEY_ARE = [(1, 4096, 4096), (16, 4096, 4352), (1, 8192, 2304), (16, 16384, 1024), (17, 4096, 4352), (32, 8192, 2304), (33, 4096, 4096), (64, 4096, 8448),
               (40, 6144, 8192)]
# the seven tiles of 32 channels per wave (the first five, 67 x 20480 x 2048, 97 x 20480 x 2048); one K step, 9 (steps past the end; the scales of
# 8 steps and one), 33; tokens that do not fill their tiles, the most tokens at several widths; two rounds of tiles
CODES_AS_THEY_ARE = [(19, 10240, 2048), (19, 20480, 1024), (34, 8704, 8192), (34, 20480, 1024), (67, 11264, 4096), (67, 20480, 2048), (97, 20480, 2048),
                     (32, 65536, 256), (130, 8192, 2304), (128, 65536, 256), (333, 4096, 8448), (512, 8192, 2048), (512, 4096, 4352), (640, 6144, 4096),
                     (1024, 4096, 4096), (480, 8320, 2304), (320, 14336, 1280), (385, 8320, 4096), (417, 12032, 4352)]
# another token, row or group than that takes; scales that start elsewhere; fewer weights; a second round of tiles with few of them, or against
# fewer channels, or a third of few K steps
RE_TILED = [(513, 8320, 2048, 0), (480, 8320, 2560, 0), (384, 12288, 2560, 0), (288, 14336, 2560, 0), (385, 8320, 4352, 0), (417, 11904, 4352, 0),
            (192, 65536, 256, 0), (129, 65536, 256, 0), (320, 28672, 1280, 0), (1025, 4096, 4096, 0), (641, 6144, 4096, 0), (16, 4128, 4096, 0), (16, 4096, 4128, 0), (16, 4096, 4096, 1),
            (100, 4096, 4096, 4), (16, 3968, 8192, 0), (16, 4096, 3840, 0)]


def weights(torch, T, N, K, shift):
    rng = np.random.default_rng(T + N + K)
    bc = to_dev(rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8), torch)
    scales = rng.integers(118, 137, size=(N, K // 32)).astype(np.uint8)
    bs = torch.zeros(scales.size + shift, dtype=torch.uint8, device="cuda")[shift:].view(N, K // 32)
    bs.copy_(to_dev(scales, torch))
    return bc, bs


def run(torch, T, N, K, shift, codes, scales):
    import paper_2604_17789_amd as duqpp
    print(f"[row-major direct] T={T} N={N} K={K} shift={shift}", flush=True)
    bc, bs = weights(torch, T, N, K, shift)
    x = to_dev_bf16(wl.make_activations(f"rmd-{T}-{K}", T, K, (wl.OutlierSpec(4, 50.0),)), torch)
    R = to_dev(wl.make_rotation_blocks("rmd", 1), torch)
    a, b = duqpp.rotate_quantize_tiled(x, R), duqpp.tile_operand(bc, bs)
    cb, sb = duqpp.tiled_bytes(T, K)
    for code, dtype in ((duqpp.F32, torch.float32), (duqpp.BF16, torch.bfloat16)):
        ws = torch.full((duqpp.gemm_workspace_bytes(T, N, K, True),), 0xA5, dtype=torch.uint8, device="cuda")
        want = duqpp.mxfp4_gemm_tiled(*a, *b, T, N, K, out_dtype=code)
        got = duqpp.rotq_gemm(x, R, bc, bs, out_dtype=code, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        at = cb + sb + b[0].numel()
        assert bool((ws[cb + sb:at] == 0xA5).all()) if codes else torch.equal(ws[cb + sb:at], b[0].reshape(-1))
        assert bool((ws[at:] == 0xA5).all()) if scales else torch.equal(ws[at:at + b[1].numel()], b[1].reshape(-1))
    # into a wider matrix: rows of their own length, nothing beside them
    wide = torch.full((T, N + 9), 3.0, dtype=torch.bfloat16, device="cuda")
    duqpp.rotq_gemm(x, R, bc, bs, out_dtype=duqpp.BF16, out=wide[:, :N], workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :N], want) and bool((wide[:, N:] == 3.0).all())


@pytest.mark.parametrize("T,N,K", AS_THEY_ARE)
def test_weights_as_they_are(T, N, K):
    import torch
    run(torch, T, N, K, 0, True, True)


@pytest.mark.parametrize("T,N,K", CODES_AS_THEY_ARE)
def test_codes_as_they_are(T, N, K):
    import torch
    run(torch, T, N, K, 0, True, False)


@pytest.mark.parametrize("T,N,K,shift", RE_TILED)
def test_weights_that_are_re_tiled(T, N, K, shift):
    import torch
    run(torch, T, N, K, shift, False, False)
