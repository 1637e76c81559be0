"""GPU parity of every tile of the tiled MXFP4 GEMM, run by its index, at the sizes where it can go wrong: ragged in tokens and
channels, one K step, numbers of K steps that leave a remainder against the steps in flight, result rows on and off the
16-byte grid; and of the shapes at which the library picks each of them, with the tile it says it picks."""
import numpy as np
import pytest

from oracle import linear
from helpers import bf16_dev_to_bits, rel_fro, tile_np, to_dev

pytestmark = pytest.mark.gpu
GEMM_TOL = 1e-5      # fp32 sums of at most 16416 exact products: a relative error of 2^-24 sqrt(16416) at most, here 8e-6
AUTO, DECODE = 0, 1
TILES = [(32, 64), (64, 64), (96, 64), (32, 128), (64, 128), (96, 128), (128, 128), (96, 256), (128, 256), (192, 256), (256, 256)]
SPLIT_K = (0, 0)


def _operands(T, N, K):
    rng = np.random.default_rng(T * 1000003 + N * 1009 + K)
    ac = rng.integers(0, 256, size=(T, K // 2)).astype(np.uint8)
    bc = rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8)
    asc = rng.integers(118, 137, size=(T, K // 32)).astype(np.uint8)
    bsc = rng.integers(118, 137, size=(N, K // 32)).astype(np.uint8)
    return ac, asc, bc, bsc


@pytest.mark.parametrize("K", [32, 544, 2048, 4128])        # 1, 3, 8 and 17 K steps of 256, the odd ones mostly padding at the end
@pytest.mark.parametrize("tile", range(len(TILES)))
def test_every_tile_by_index(tile, K):
    """Two tiles each way, the second a sliver: fp32 against the oracle and bit for bit what the first tile shape gives, bf16 the
    rounding of that fp32 result bit for bit, into rows on and off the 16-byte grid, and nothing written beside the rows."""
    import torch

    import paper_2604_17789_amd as duqpp
    tokens, channels = TILES[tile]
    T, N = tokens + 5, channels + 11
    kernel = duqpp.KERNEL_TILE + tile
    assert duqpp.gemm_tiles() == len(TILES)
    assert duqpp.gemm_tile_for(T, N, K, kernel=kernel) == (tile, tokens, channels)
    ac, asc, bc, bsc = _operands(T, N, K)
    print(f"[gemm tiles] {tokens} x {channels} T={T} N={N} K={K}", flush=True)
    ops = [to_dev(t, torch) for t in tile_np(ac, asc) + tile_np(bc, bsc)]
    y = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, kernel=kernel)
    other = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, kernel=duqpp.KERNEL_TILE)
    wide = [torch.full((T, ld), -77.0, dtype=torch.bfloat16, device="cuda:0") for ld in ((N + 15) // 8 * 8, N + 2)]
    for w in wide:
        duqpp.mxfp4_gemm_tiled(*ops, T, N, K, out_dtype=duqpp.BF16, kernel=kernel, out=w[:, :N])
    torch.cuda.synchronize()
    y32 = y.cpu().numpy()
    assert rel_fro(y32, linear.mxfp4_gemm(ac, asc, bc, bsc)) <= GEMM_TOL
    assert torch.equal(y, other)
    for w in wide:
        np.testing.assert_array_equal(bf16_dev_to_bits(w[:, :N].contiguous()), linear.round_to_bf16_bits(y32))
        assert torch.all(w[:, N:] == -77.0)


# shapes for which the library picks each tile
PICKED = [
    (AUTO, 33, 4200, 32, (32, 64)),          # one step
    (AUTO, 200, 72, 2336, (32, 64)),         # ten steps of which the last is mostly padding
    (AUTO, 33, 8300, 800, (32, 128)),
    (AUTO, 33, 8300, 4128, (64, 64)),
    (DECODE, 77, 14400, 1184, (96, 64)),
    (AUTO, 200, 5000, 4128, (96, 64)),
    (AUTO, 200, 5000, 2336, (64, 128)),
    (AUTO, 130, 14400, 544, (96, 128)),
    (AUTO, 300, 8296, 2336, (128, 128)),
    (AUTO, 700, 8300, 32, (128, 128)),
    (AUTO, 200, 20000, 288, (96, 256)),
    (AUTO, 1000, 8300, 544, (96, 256)),
    (AUTO, 1500, 8300, 288, (128, 256)),
    (AUTO, 500, 20000, 8224, (192, 256)),
    (AUTO, 1500, 8296, 8224, (256, 256)),    # in both directions ragged; 33 steps
    (AUTO, 1500, 8300, 8224, (128, 256)),    # channels that are no multiple of 8
    # K split over eight waves
    (AUTO, 17, 4097, 288, SPLIT_K),          # whole row tiles, one more than there are pairs of CUs
    (AUTO, 33, 70, 32, SPLIT_K),             # half row tiles, a second token row tile of one token, seven waves without a step
    (AUTO, 65, 1000, 2336, SPLIT_K),         # half row tiles, three token row tiles
    (DECODE, 128, 1024, 2336, SPLIT_K),      # four, the last of the round
    (AUTO, 64, 4070, 2336, SPLIT_K),         # whole row tiles, two token row tiles
    (AUTO, 97, 2040, 544, SPLIT_K),          # four
    (AUTO, 33, 4100, 8000, SPLIT_K),         # both token row tiles in a workgroup
    (AUTO, 64, 8192, 16416, SPLIT_K),
    # their edges
    (AUTO, 65, 4096, 544, (32, 64)),
    (DECODE, 65, 2049, 544, (32, 64)),
    (AUTO, 64, 4100, 7904, (32, 64)),
    (AUTO, 64, 8193, 16416, (64, 64)),
    (AUTO, 65, 8192, 16416, (64, 64)),
]


@pytest.mark.parametrize("kernel,T,N,K,picked", PICKED)
def test_tile_against_oracle(kernel, T, N, K, picked):
    """fp32 against the oracle, bf16 the rounding of that fp32 result bit for bit, also into rows that are not on the
    16-byte grid (stored element by element) with nothing written beside them."""
    import torch

    import paper_2604_17789_amd as duqpp
    rng = np.random.default_rng(T + N + K)
    assert duqpp.gemm_tile_for(T, N, K, kernel=kernel)[1:] == picked
    ac, asc, bc, bsc = _operands(T, N, K)
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
