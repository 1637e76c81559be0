"""GPU parity of the tiled product where the token row tiles do not fill its tiles and are spread evenly over them: two and three
tiles of MT and MT - 1 row tiles, the fewest row tiles that spread and the most that do not, ragged channels, several K steps."""
import numpy as np
import pytest

from oracle import linear
from helpers import bf16_dev_to_bits, rel_fro, tile_np, to_dev
from test_gpu_gemm_tiles import GEMM_TOL, TILES, _operands

pytestmark = pytest.mark.gpu


def _row_tiles(mt):
    """Numbers of row tiles: spread over two and three tiles, and one more than a tile's (spread up to MT = 3 only)."""
    return sorted({2 * mt - 1, 3 * mt - 2, mt + 1})


@pytest.mark.parametrize("K", [7936, 7968, 8192, 8480])      # the longest that is not spread, the shortest, and a remainder of steps
@pytest.mark.parametrize("tile", [i for i, (tokens, channels) in enumerate(TILES) if tokens > 96 or channels == 256])
def test_spread_tiles(tile, K):
    """Bit for bit what tiles of one row tile give, those against the oracle; bf16 the rounding of the fp32 result bit for bit, on
    and off the 16-byte grid, and nothing written beside the rows."""
    import torch

    import paper_2604_17789_amd as duqpp
    tokens, channels = TILES[tile]
    for row_tiles in _row_tiles(tokens // 32):
        T, N = 32 * row_tiles - 9, channels + 11
        kernel = duqpp.KERNEL_TILE + tile
        ac, asc, bc, bsc = _operands(T, N, K)
        print(f"[gemm spread] {tokens} x {channels} T={T} N={N} K={K}", flush=True)
        ops = [to_dev(t, torch) for t in tile_np(ac, asc) + tile_np(bc, bsc)]
        whole = torch.full((T + 40, N), -77.0, device="cuda:0")
        y = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, kernel=kernel, out=whole[:T])
        other = duqpp.mxfp4_gemm_tiled(*ops, T, N, K, kernel=duqpp.KERNEL_TILE)
        wide = [torch.full((T, ld), -77.0, dtype=torch.bfloat16, device="cuda:0") for ld in ((N + 15) // 8 * 8, N + 2)]
        for w in wide:
            duqpp.mxfp4_gemm_tiled(*ops, T, N, K, out_dtype=duqpp.BF16, kernel=kernel, out=w[:, :N])
        torch.cuda.synchronize()
        assert torch.equal(y, other) and torch.all(whole[T:] == -77.0)
        y32 = y.cpu().numpy()
        rows = np.sort(np.random.default_rng(T + K).choice(T, 32, replace=False))
        assert rel_fro(y32[rows], linear.mxfp4_gemm(ac[rows], asc[rows], bc, bsc)) <= GEMM_TOL
        for w in wide:
            np.testing.assert_array_equal(bf16_dev_to_bits(w[:, :N].contiguous()), linear.round_to_bf16_bits(y32))
            assert torch.all(w[:, N:] == -77.0)
