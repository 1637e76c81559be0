"""GPU parity of every tile shape of the tiled MXFP4 GEMM at the sizes where it can go wrong: ragged in tokens and
channels, one K step, and numbers of K steps that leave a remainder against the steps in flight."""
import numpy as np
import pytest

from oracle import linear
from helpers import bf16_dev_to_bits, rel_fro, tile_np, to_dev

pytestmark = pytest.mark.gpu
GEMM_TOL = 1e-5      # fp32 sums of at most 16416 exact products: a relative error of 2^-24 sqrt(16416) at most, here 8e-6
AUTO, DECODE = 0, 1

# smallest shapes for which the library picks each tile (tokens x channels of a workgroup), from one K step of 256 up
TILES = [
    (AUTO, 33, 70, 32),          # 32 x 64, one step
    (DECODE, 128, 1000, 2336),   # 32 x 64, ten steps of which the last is mostly padding
    (AUTO, 33, 8300, 800),       # 32 x 128, four steps
    (AUTO, 33, 8300, 4128),      # 64 x 64, 17 steps
    (DECODE, 77, 14400, 1184),   # 96 x 64, five steps
    (AUTO, 200, 5000, 4128),     # 96 x 64, 17 steps
    (AUTO, 130, 14400, 544),     # 64 x 128, three steps
    (AUTO, 200, 20000, 288),     # 96 x 128, two steps
    (AUTO, 700, 8300, 32),       # 128 x 128, one step
    (AUTO, 1000, 8300, 544),     # 96 x 256, three steps
    (AUTO, 1500, 8300, 288),     # 128 x 256, two steps
    (AUTO, 500, 20000, 8224),    # 192 x 256, 33 steps
    (AUTO, 1500, 8300, 8224),    # 256 x 256 (or 128 x 256 with a result off the 16-byte grid), 33 steps
    (AUTO, 33, 8300, 16416),     # K split over eight waves, two activation row tiles, 65 steps
    (AUTO, 64, 8192, 16416),     # the same without ragged edges
    (AUTO, 65, 8192, 16416),     # one token more: a tile again
]


@pytest.mark.parametrize("kernel,T,N,K", TILES)
def test_tile_against_oracle(kernel, T, N, K):
    """fp32 against the oracle, bf16 the rounding of that fp32 result bit for bit, also into rows that are not on the
    16-byte grid (stored element by element) with nothing written beside them."""
    import torch

    import paper_2604_17789_amd as duqpp
    rng = np.random.default_rng(T * 1000003 + N * 1009 + K)
    ac = rng.integers(0, 256, size=(T, K // 2)).astype(np.uint8)
    bc = rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8)
    asc = rng.integers(118, 137, size=(T, K // 32)).astype(np.uint8)
    bsc = rng.integers(118, 137, size=(N, K // 32)).astype(np.uint8)
    print(f"[gemm tiles] kernel={kernel} T={T} N={N} K={K}", flush=True)
    ops = [to_dev(t, torch) for t in tile_np(ac, asc) + tile_np(bc, bsc)]
    y = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, kernel=kernel)
    y16 = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, out_dtype=duqpp.BF16, kernel=kernel)
    wide = torch.full((T, N + 3), -77.0, dtype=torch.bfloat16, device="cuda:0")
    duqpp.mxfp4_gemm_tiled(*ops, T, N, K, out_dtype=duqpp.BF16, kernel=kernel, out=wide[:, :N])
    torch.cuda.synchronize()
    rows = np.sort(rng.choice(T, min(T, 64), replace=False))
    y32 = y.cpu().numpy()
    assert rel_fro(y32[rows], linear.mxfp4_gemm(ac[rows], asc[rows], bc, bsc)) <= GEMM_TOL
    cols = np.sort(rng.choice(N, min(N, 64), replace=False))
    assert rel_fro(y32[:, cols], linear.mxfp4_gemm(ac, asc, bc[cols], bsc[cols])) <= GEMM_TOL
    want = linear.round_to_bf16_bits(y32)
    np.testing.assert_array_equal(bf16_dev_to_bits(y16), want)
    np.testing.assert_array_equal(bf16_dev_to_bits(wide[:, :N].contiguous()), want)
    assert torch.all(wide[:, N:] == -77.0)
