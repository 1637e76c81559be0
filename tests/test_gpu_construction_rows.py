"""GPU parity of the construction's search on the rows that can hold the largest magnitude: which rows are left out, when it leaves the
search to the other kernels, and the result, bit for bit the oracle's in either case."""
import numpy as np
import pytest

import workloads as wl
from oracle import construction
from helpers import to_dev, to_dev_bf16
from test_gpu_construction_forms import AUTO, ONE_32, buffers, call, check

pytestmark = pytest.mark.gpu

def most(T):
    """Rows it takes."""
    return 22 if T <= 992 else 28


def done(torch, o):
    """Whether the search on few rows did the work: the fourth word of the workspace."""
    return bool(o["ws"][24:32].view(torch.int64).item())


def run(torch, duqpp, xf, q, how=AUTO):
    xb = (np.ascontiguousarray(xf, np.float32).view(np.uint32) >> 16).astype(np.uint16)
    o = buffers(torch, xf.shape[0], q.shape[0])
    status = call(torch, duqpp, how, to_dev_bf16(xb, torch), to_dev(q, torch), o)
    assert status == 0
    torch.cuda.synchronize()
    check(o, construction.greedy_rotation(wl.bf16_bits_to_f32(xb), q))
    return done(torch, o)


def activations(name, T, K, large, value=640.0):
    """Small values, and `large` rows with one large value each in the block of channels 32 to 63."""
    xf = wl.bf16_bits_to_f32(wl.make_activations(name, T, K)).copy()
    rng = np.random.default_rng(T + large)
    rows = rng.permutation(T)[:large]
    xf[rows, 32 + rng.integers(0, 32, large)] = value
    return xf


# as many tokens as rows, as many rows as the kernel takes, one more, either side of the tokens where that changes; rows in the first, the
# last and every pass over the norms; 1, 2, 3, 6, 7 rows that count (waves without rows, with one row, more than the four that stay), 14, 15 and
# 28 (two rows a wave or four), 29: too many; no step, one and two
@pytest.mark.parametrize("T,K,large,steps", [(2, 64, 1, 5), (22, 64, 22, 9), (23, 64, 23, 9), (28, 64, 28, 9), (28, 64, 2, 9), (29, 64, 1, 9), (64, 64, 2, 1),
                                             (100, 96, 3, 2), (257, 64, 6, 0), (992, 64, 22, 3), (992, 64, 23, 3), (993, 64, 23, 3),
                                             (2048, 64, 7, 33), (2048, 64, 14, 20), (2049, 64, 15, 20), (2049, 64, 28, 20), (500, 64, 29, 4), (16352, 64, 12, 3)])
def test_rows_that_count(T, K, large, steps):
    import torch

    import paper_2604_17789_amd as duqpp
    print(f"[construct rows] T={T} K={K} large={large} steps={steps}", flush=True)
    q = wl.make_orthogonal_steps("gpu-cons-rows", steps)
    xf = activations("gpu-cons-rows", T, K, large)
    assert run(torch, duqpp, xf, q) == (large <= most(T))
    assert not run(torch, duqpp, xf, q, ONE_32)


def test_rows_of_equal_norm_count():
    """A row a little below N / sqrt(32) may be left out, one above may not; equal magnitudes in several rows: the smallest channel."""
    import torch

    import paper_2604_17789_amd as duqpp
    q = wl.make_orthogonal_steps("gpu-cons-rows-equal", 24)
    xf = np.zeros((300, 64), np.float32)
    xf[7, 40], xf[250, 37], xf[111, 61] = 64.0, -64.0, 64.0
    xf[20:40] = 64.0 / np.sqrt(32.0) / np.sqrt(64.0) * 0.9      # norms of the block 0.9 / sqrt(2) of the bound
    xf[60:79, 33] = 64.0 / np.sqrt(32.0) * 1.02
    assert run(torch, duqpp, xf, q)
    xf[:, 50] = 64.0 / np.sqrt(32.0) * 1.02                     # every row counts
    assert not run(torch, duqpp, xf, q)
    assert not run(torch, duqpp, np.zeros((100, 64), np.float32), q)
    assert run(torch, duqpp, np.zeros((20, 64), np.float32), q)


@pytest.mark.parametrize("spoilt", ["scaled", "nan", "orthogonal to 1e-5"])
def test_draws_that_are_not_orthogonal(spoilt):
    """Rows may only be left out while the steps keep their norms; what the draws are like is measured."""
    import torch

    import paper_2604_17789_amd as duqpp
    steps = 12
    q = wl.make_orthogonal_steps("gpu-cons-rows-draws", steps)
    xf = activations("gpu-cons-rows-draws", 400, 64, 3)
    if spoilt == "scaled":
        q[5] *= 1.5
        assert not run(torch, duqpp, xf, q)
    elif spoilt == "nan":
        q[5, 3, 4] = np.nan
        o = buffers(torch, 400, steps)
        xb = (xf.view(np.uint32) >> 16).astype(np.uint16)
        assert call(torch, duqpp, AUTO, to_dev_bf16(xb, torch), to_dev(q, torch), o) == 0
        torch.cuda.synchronize()
        assert not done(torch, o)
    else:
        q[5, 3] *= 1.0 + 1e-5                                # 31 times 2e-5, times 12 steps: below 0.02
        assert run(torch, duqpp, xf, q)


def test_infinities_go_to_the_other_kernels():
    import torch

    import paper_2604_17789_amd as duqpp
    q = wl.make_orthogonal_steps("gpu-cons-rows-inf", 6)
    for T in (20, 200):
        for value in (np.inf, -np.inf, np.nan):
            xf = activations("gpu-cons-rows-inf", T, 64, 2)
            xf[T // 2, 40] = value
            xb = to_dev_bf16((xf.view(np.uint32) >> 16).astype(np.uint16), torch)
            results = []
            for how in (ONE_32, AUTO):
                o = buffers(torch, T, 6)
                assert call(torch, duqpp, how, xb, to_dev(q, torch), o) == 0
                torch.cuda.synchronize()
                assert not done(torch, o)
                results.append((o["info"].tolist(), o["peaks"].view(torch.int64).tolist(), o["R"].view(torch.int32).tolist()))
            assert results[0] == results[1]


@pytest.mark.parametrize("captured", [True, False])
def test_one_workspace_for_few_rows_and_many(captured):
    """Replays of one graph, and calls with one workspace, whose activations leave few rows, too many, and few again: what the call before left
    in the workspace does not decide which kernel does the work."""
    import torch

    import paper_2604_17789_amd as duqpp
    T, K, steps = 400, 64, 10
    q = wl.make_orthogonal_steps("gpu-cons-rows-reuse", steps)
    inputs = [activations(f"gpu-cons-rows-reuse-{i}", T, K, large) for i, large in enumerate((3, 60, 20, 200, 1))]
    bits = [(xf.view(np.uint32) >> 16).astype(np.uint16) for xf in inputs]
    x, qd, o = to_dev_bf16(bits[0], torch).clone(), to_dev(q, torch), buffers(torch, T, steps)
    duqpp.init()
    if captured:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call(torch, duqpp, AUTO, x, qd, o) == 0
    for i in (0, 1, 2, 3, 4, 1, 1, 0, 0):
        print(f"[construct rows] one workspace, captured={captured}, activations {i}", flush=True)
        x.copy_(to_dev_bf16(bits[i], torch))
        if captured:
            graph.replay()
        else:
            assert call(torch, duqpp, AUTO, x, qd, o) == 0
        torch.cuda.synchronize()
        check(o, construction.greedy_rotation(wl.bf16_bits_to_f32(bits[i]), q))
        assert done(torch, o) == (i in (0, 2, 4))
        torch.ones(1 << 16, device="cuda").sum().item()
