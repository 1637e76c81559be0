"""GPU parity of duqpp_group_error where the mean comes from partial sums that use the first ratios' places until it is
formed: sizes either side of the switch, an odd number of groups, one group per token, more token tiles than runs; and either
side of the sizes from which a wave takes two groups and the mean reads ahead."""
import numpy as np
import pytest

import workloads as wl
from oracle import mxfp4, pipeline
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,rotated", [(511, 4096, 1), (512, 4096, 1), (513, 4128, 1), (2100, 1024, 0), (70000, 32, 1), (5, 14368 * 32, 0),
                                         (256, 4096, 1), (257, 4096, 0), (64, 1024, 0), (65, 1024, 1), (10, 32, 0),
                                         (500, 4096, 0), (1030, 4096, 0)])
def test_ratios_and_mean(T, K, rotated):
    """Every ratio within one rounding to fp32 of the oracle's on the device's own rotated values (2e-7), groups of zeros
    marked also among the first ratios, the mean within the fp64 sum's rounding."""
    import torch

    import paper_2604_17789_amd as duqpp
    name = f"gpu-gerr-mean-{T}-{K}"
    xb = wl.make_activations(name, T, K, (wl.OutlierSpec(1, 50.0),))
    xb[:3, :32] = 0
    xb[T - 1, K - 32:] = 0
    x = to_dev_bf16(xb, torch)
    R = to_dev(wl.make_rotation_blocks(name, K // 32), torch) if rotated else None
    print(f"[group error] mean T={T} K={K} rotated={rotated}", flush=True)
    err, mean = duqpp.group_error(x, R)
    err_only, _ = duqpp.group_error(x, R, return_mean=False)
    torch.cuda.synchronize()
    assert torch.equal(err, err_only)
    y = duqpp.rotate_quantize(x, R, return_rotated=True)[2].cpu().numpy() if rotated else wl.bf16_bits_to_f32(xb)
    want = pipeline.per_group_normalised_errors(y, *mxfp4.quantize(y))
    err = err.cpu().numpy()
    ok = want >= 0
    assert not ok[0, 0] and not ok[T - 1, K // 32 - 1]
    np.testing.assert_array_equal(err[~ok], -1.0)
    np.testing.assert_allclose(err[ok], want[ok], rtol=2e-7, atol=1e-12)
    assert abs(mean - float(np.mean(err[ok].astype(np.float64)))) <= 1e-12 * mean
