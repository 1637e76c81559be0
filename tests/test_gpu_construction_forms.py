"""GPU parity of the forms of the construction (one launch for all steps with 16 or 32 rows per workgroup, a launch per step, and
a few workgroups or one for everything where the others gave up waiting) at the sizes where their split changes."""
import numpy as np
import pytest

import workloads as wl
from oracle import construction
from helpers import to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

AUTO, ONE_16, ONE_32, STEPS, IMPATIENT, ALONE, LEAVES = 0, 1, 2, 3, 8, 24, 32
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
    """What the workgroups leave in the second and third word of the workspace: that one of the search kernel's gave up, and then a few
    did the work behind them; that one of these gave up, and then one did it."""
    return o["ws"][8:24].view(torch.int64).tolist()


def check(o, ref):
    """fp64 in the oracle's operation order: block, steps kept, peaks and matrix bit for bit."""
    assert o["info"].tolist() == [ref["block"], ref["steps"]]
    np.testing.assert_array_equal(o["peaks"].cpu().numpy(), ref["peaks"])
    np.testing.assert_array_equal(o["R"].cpu().numpy(), ref["R"])


# 1, 2, 3: the workspace holds what none, two and three workgroups publish; 992 / 993: 64 / 65 workgroups of 16 rows, i.e. one or more
# looks of 64 lanes; 64 / 65: one or two workgroups where those gave up, 300: five, 993: sixteen, 777 without a step: six; 8160 with
# seven steps: 49, two or three waves of each with rows; 4064 / 4065: 256 workgroups, the most of 16 rows; 8160 / 8161: 256 / 257 workgroups of 32; 16352: the most
CASES = [(1, 64, 3, ()), (2, 64, 3, (ONE_32,)), (3, 64, 4, (ONE_16, ONE_32)), (17, 32, 3, (ONE_16, ONE_32)), (33, 96, 5, (ONE_16, ONE_32)), (64, 32, 4, (ONE_16, ONE_32)), (65, 32, 4, (ONE_16, ONE_32)), (992, 64, 3, (ONE_16, ONE_32)),
         (993, 32, 3, (ONE_16,)), (4064, 32, 2, (ONE_16, ONE_32)), (4065, 32, 2, (ONE_32,)), (8160, 32, 7, (ONE_32,)),
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
    few = min(64, -(-T // 64), 31 * (steps + 1) // 5)
    for how in (AUTO, STEPS) + one + tuple(f + hurry for f in one for hurry in (IMPATIENT, ALONE)):
        print(f"[construct] T={T} K={K} steps={steps} form={how}", flush=True)
        o = buffers(torch, T, steps)
        assert call(torch, duqpp, how, x, qd, o) == 0
        torch.cuda.synchronize()
        check(o, ref)
        if how not in (AUTO, STEPS):
            assert given_up(torch, o) == [int(how & ALONE > 0), int(how & ALONE == ALONE and few > 1)]
    for how in {ONE_16, ONE_32} - set(one) if T > 4064 or T < 3 else ():
        assert call(torch, duqpp, how, x, qd, buffers(torch, T, steps)) == ERR_SHAPE


# two, five and 49 workgroups; the first, one in the middle and the last exchange, without a step the only one
@pytest.mark.parametrize("T,steps,at", [(300, 0, 0), (65, 1, 1), (300, 4, 0), (300, 4, 2), (300, 4, 4), (8160, 7, 7)])
def test_the_first_of_the_few_gives_up(T, steps, at):
    """The first workgroup goes on alone behind one exchange that the others complete: those that have seen the last one leave with all
    steps done, the others when their patience ends."""
    import torch

    import paper_2604_17789_amd as duqpp
    K, how = 64, ONE_32 + IMPATIENT + LEAVES * (at + 1)
    name = f"gpu-cons-leaves-{T}-{steps}"
    xb = wl.make_activations(name, T, K, (wl.OutlierSpec(3, 50.0),))
    q = wl.make_orthogonal_steps(name, steps)
    print(f"[construct] T={T} steps={steps} the first gives up at {at}", flush=True)
    o = buffers(torch, T, steps)
    assert call(torch, duqpp, how, to_dev_bf16(xb, torch), to_dev(q, torch), o) == 0
    torch.cuda.synchronize()
    check(o, construction.greedy_rotation(wl.bf16_bits_to_f32(xb), q))
    assert given_up(torch, o) == [1, 1]


@pytest.mark.parametrize("how", [ONE_16, ONE_32, ONE_16 + IMPATIENT, ONE_16 + ALONE, STEPS])
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


def test_infinities_and_nan_are_the_same_in_every_form():
    """What no oracle states: the bits of peaks and matrix of all forms agree where the state holds infinities and NaN."""
    import torch

    import paper_2604_17789_amd as duqpp
    T, K, steps = 200, 64, 6
    q = to_dev(wl.make_orthogonal_steps("gpu-cons-inf", steps), torch)
    for value, at in ((np.inf, (7, 33)), (-np.inf, (150, 40)), (np.nan, (99, 5))):
        xf = wl.bf16_bits_to_f32(wl.make_activations("gpu-cons-inf", T, K, (wl.OutlierSpec(2, 20.0),))).copy()
        xf[at] = value
        x = to_dev_bf16((xf.view(np.uint32) >> 16).astype(np.uint16), torch)
        results = []
        for how in (STEPS, ONE_16, ONE_32, ONE_32 + IMPATIENT, ONE_16 + ALONE):
            o = buffers(torch, T, steps)
            assert call(torch, duqpp, how, x, q, o) == 0
            torch.cuda.synchronize()
            results.append((o["info"].tolist(), o["peaks"].view(torch.int64).tolist(), o["R"].view(torch.int32).tolist()))
        assert all(r == results[0] for r in results)


@pytest.mark.parametrize("T,streams", [(16352, 2), (8160, 3), (2048, 4)])
def test_calls_on_several_streams_at_once(T, streams):
    """Workgroups that wait for each other, on a device that cannot hold all of them at once: every call ends, with the result that it
    has by itself, whether it got on or gave up."""
    import torch

    import paper_2604_17789_amd as duqpp
    K, steps = 64, 24
    q = wl.make_orthogonal_steps("gpu-cons-streams", steps)
    qd, sides = to_dev(q, torch), [torch.cuda.Stream() for _ in range(streams)]
    xs = [to_dev_bf16(wl.make_activations(f"gpu-cons-streams-{T}-{i}", T, K, (wl.OutlierSpec(2, 20.0 + i),)), torch) for i in range(streams)]
    alone, both = [buffers(torch, T, steps) for _ in xs], [buffers(torch, T, steps) for _ in xs]
    for x, o in zip(xs, alone):
        assert call(torch, duqpp, STEPS, x, qd, o) == 0
    torch.cuda.synchronize()
    torch.cuda._sleep(2000000)                               # all of them wait for this, so that they start together
    for side in sides:
        side.wait_stream(torch.cuda.current_stream())
    for side, x, o in zip(sides, xs, both):
        with torch.cuda.stream(side):
            assert call(torch, duqpp, AUTO, x, qd, o) == 0
    torch.cuda.synchronize()
    print(f"[construct] T={T} streams={streams} given up {[given_up(torch, o) for o in both]}", flush=True)
    for a, o in zip(alone, both):
        assert all(torch.equal(a[k], o[k]) for k in ("R", "info", "peaks"))


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
