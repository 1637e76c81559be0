"""GPU: what duqpp_group_error_partials leaves for the mean, either side of the sizes where its workgroups change shape: the ratios are
duqpp_group_error's, the mean of the sums is the ratios' to the rounding of fp64 sums (each of n additions at most 2^-53 of the sum: n = 2^18
ratios give 3e-11), from 65536 ratios on the call's own bits, and nothing is written behind the bytes it asks for."""
import pytest

import workloads as wl
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

ERR_NULL, ERR_ALIGN, ERR_WORKSPACE = -1, -3, -5


@pytest.mark.parametrize("T,K,rotated", [(1, 32, 1), (31, 96, 0), (256, 4096, 1), (257, 4096, 1), (256, 4096, 0), (511, 4096, 1), (512, 4096, 1), (2100, 1024, 0), (33, 128 * 1024, 0)])
def test_mean_of_the_sums(T, K, rotated):
    import torch

    import paper_2604_17789_amd as duqpp
    from paper_2604_17789_amd.binding import _stream, lib
    name = f"gpu-gerr-partials-{T}-{K}"
    x = to_dev_bf16(wl.make_activations(name, T, K, (wl.OutlierSpec(1, 50.0),)), torch)
    x[:, -32:] = 0                                           # groups without a ratio
    R = to_dev(wl.make_rotation_blocks(name, K // 32), torch) if rotated else None
    n = lib.duqpp_group_error_partials_bytes(T, K)
    assert n % 16 == 0 and n > 0
    args = (x.data_ptr(), T, K, K, R.data_ptr() if rotated else None, K // 32)
    want, mean = torch.empty((T, K // 32), device="cuda"), torch.empty(1, dtype=torch.float64, device="cuda")
    assert lib.duqpp_group_error(*args, want.data_ptr(), mean.data_ptr(), _stream()) == 0
    for place in (dict(device="cuda"), dict(pin_memory=True)):
        print(f"[group error] partials T={T} K={K} rotated={rotated} {place}", flush=True)
        err, sums = torch.full((T, K // 32), 9.0, device="cuda"), torch.full((n // 8 + 2,), 9.0, dtype=torch.float64, **place)
        assert lib.duqpp_group_error_partials(*args, err.data_ptr(), sums.data_ptr(), n, _stream()) == 0
        torch.cuda.synchronize()
        sums = sums.cpu()
        got = lib.duqpp_group_error_mean(sums.data_ptr(), n)
        assert torch.equal(err, want) and sums[n // 8:].tolist() == [9.0, 9.0]
        assert sums[1:n // 8:2].sum().item() == (want >= 0).sum().item()
        assert got == mean.item() if T * K // 32 >= 65536 else abs(got - mean.item()) <= 3e-11 * mean.item()
        assert duqpp.group_error(x, R)[1] == got
    assert lib.duqpp_group_error_partials(*args, want.data_ptr(), None, n, _stream()) == ERR_NULL
    assert lib.duqpp_group_error_partials(*args, want.data_ptr(), sums.data_ptr() + 4, n, _stream()) == ERR_ALIGN
    assert lib.duqpp_group_error_partials(*args, want.data_ptr(), sums.data_ptr(), n - 1, _stream()) == ERR_WORKSPACE
