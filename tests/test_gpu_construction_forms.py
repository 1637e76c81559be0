"""GPU parity of the forms of the construction (one launch for all steps with 16 or 32 rows per workgroup, a launch per step, and
one workgroup for everything where the others gave up waiting) at the sizes where their split changes."""
import numpy as np
import pytest

import workloads as wl
from oracle import construction
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

AUTO, ONE_16, ONE_32, STEPS, IMPATIENT = 0, 1, 2, 3, 8
ERR_SHAPE = -2


def call(torch, duqpp, how, x, q, o):
    from paper_2604_17789_amd.binding import _stream, lib
    return lib.duqpp_construct_rotation_on(how, x.data_ptr(), x.shape[0], x.shape[1], x.stride(0), q.data_ptr(), q.shape[0],
                                           o["R"].data_ptr(), o["info"].data_ptr(), o["peaks"].data_ptr(), o["ws"].data_ptr(),
                                           o["ws"].numel(), _stream())


def buffers(torch, T, steps):
    from paper_2604_17789_amd.binding import lib
    n = lib.duqpp_construct_rotation_workspace_bytes(T, steps)      # what was in the workspace must not matter: all kinds of bytes
    return dict(R=torch.full((32, 32), 7.0, device="cuda"), info=torch.full((2,), -1, dtype=torch.int32, device="cuda"),
                peaks=torch.full((steps + 1,), -1.0, dtype=torch.float64, device="cuda"),
                ws=torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda"))


def given_up(torch, o):
    """What the search kernel's workgroups leave in the second word of the workspace: 1 where one of them gave up, and then the launch
    behind them did the work; 0 where it found nothing to do."""
    return int(o["ws"][8:16].view(torch.int64).item())


def check(o, ref):
    """fp64 in the oracle's operation order: block, steps kept, peaks and matrix bit for bit."""
    assert o["info"].tolist() == [ref["block"], ref["steps"]]
    np.testing.assert_array_equal(o["peaks"].cpu().numpy(), ref["peaks"])
    np.testing.assert_array_equal(o["R"].cpu().numpy(), ref["R"])


# 1, 2, 3: the workspace holds what none, two and three workgroups publish; 992 / 993: 64 / 65 workgroups of 16 rows, i.e. one or more
# looks of 64 lanes; 4064 / 4065: 256 workgroups, the most of 16 rows; 8160 / 8161: 256 / 257 workgroups of 32; 16352: the most
CASES = [(1, 64, 3, ()), (2, 64, 3, (ONE_32,)), (3, 64, 4, (ONE_16, ONE_32)), (17, 32, 3, (ONE_16, ONE_32)), (33, 96, 5, (ONE_16, ONE_32)), (992, 64, 3, (ONE_16, ONE_32)),
         (993, 32, 3, (ONE_16,)), (4064, 32, 2, (ONE_16, ONE_32)), (4065, 32, 2, (ONE_32,)), (8160, 32, 2, (ONE_32,)),
         (8161, 32, 3, (ONE_32,)), (16352, 32, 2, (ONE_32,)), (16353, 32, 2, ()), (777, 64, 0, (ONE_16, ONE_32)), (300, 512, 40, (ONE_16, ONE_32))]


@pytest.mark.parametrize("T,K,steps,one", CASES)
def test_every_form_matches_the_oracle(T, K, steps, one):
    import torch

    import paper_2604_17789_amd as duqpp
    name = f"gpu-cons-form-{T}-{K}"
    xb = wl.make_activations(name, T, K, (wl.OutlierSpec(3, 50.0),))
    q = wl.make_orthogonal_steps(name, steps)
    x, qd = to_dev_bf16(xb, torch), to_dev(q, torch)
    ref = construction.greedy_rotation(wl.bf16_bits_to_f32(xb), q)
    for how in (AUTO, STEPS) + one + tuple(f + IMPATIENT for f in one):
        print(f"[construct] T={T} K={K} steps={steps} form={how}", flush=True)
        o = buffers(torch, T, steps)
        assert call(torch, duqpp, how, x, qd, o) == 0
        torch.cuda.synchronize()
        check(o, ref)
        if how in (ONE_16, ONE_32) or how & IMPATIENT:
            assert given_up(torch, o) == (1 if how & IMPATIENT else 0)
    for how in {ONE_16, ONE_32} - set(one) if T > 4064 or T < 3 else ():
        assert call(torch, duqpp, how, x, qd, buffers(torch, T, steps)) == ERR_SHAPE


@pytest.mark.parametrize("how", [ONE_16, ONE_32, ONE_16 + IMPATIENT, STEPS])
@pytest.mark.parametrize("kind", ["zeros", "ties"])
def test_smallest_channel_among_equals(kind, how):
    """All-zero activations, and the same magnitude in several channels and workgroups: the first channel, the first step."""
    import torch

    import paper_2604_17789_amd as duqpp
    T, K, steps = 100, 64, 6
    xf = np.zeros((T, K), np.float32)
    if kind == "ties":
        xf[3, 40], xf[90, 37], xf[50, 37], xf[17, 61] = 2.0, -2.0, 2.0, 2.0
    xb = (xf.view(np.uint32) >> 16).astype(np.uint16)
    q = wl.make_orthogonal_steps("gpu-cons-ties", steps)
    o = buffers(torch, T, steps)
    assert call(torch, duqpp, how, to_dev_bf16(xb, torch), to_dev(q, torch), o) == 0
    torch.cuda.synchronize()
    check(o, construction.greedy_rotation(xf, q))


def test_construction_in_a_graph():
    """Captured once and replayed, with other work and other activations between the replays."""
    import torch

    import paper_2604_17789_amd as duqpp
    T, K, steps = 500, 128, 12
    q = wl.make_orthogonal_steps("gpu-cons-graph", steps)
    inputs = [wl.make_activations(f"gpu-cons-graph-{i}", T, K, (wl.OutlierSpec(2, 20.0 + i),)) for i in range(3)]
    x, qd, o = to_dev_bf16(inputs[0], torch).clone(), to_dev(q, torch), buffers(torch, T, steps)
    duqpp.init()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert call(torch, duqpp, AUTO, x, qd, o) == 0
    for xb in inputs + inputs[:1]:
        x.copy_(to_dev_bf16(xb, torch))
        graph.replay()
        torch.cuda.synchronize()
        check(o, construction.greedy_rotation(wl.bf16_bits_to_f32(xb), q))
        torch.ones(1 << 16, device="cuda").sum().item()
