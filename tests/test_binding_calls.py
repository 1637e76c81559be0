"""The binding's native module: what it does not take goes on to the Python path, which refuses and accepts as it does without the
module, and what it takes gives the same bits, objects and errors as that path."""
import pytest
import torch

import paper_2604_17789_amd as duqpp
from paper_2604_17789_amd import binding

T, K, N = 48, 512, 96


class Never:
    """In the place of the native module: the Python path for everything."""
    linear = rows = product = error = staticmethod(lambda *a: None)


@pytest.mark.parametrize("fn", ["linear", "rows", "product", "error"])
def test_anything_else_is_left_to_the_python_path(fn):
    f = getattr(binding._calls, fn)
    x, b = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(8192, dtype=torch.uint8)
    for args in [(), (1,), (None,) * 9, (0, x, None, None), (x, None), (0, x, b, b, b, 4, 0, None, None),
                 (b, b, b, b, 4, 4, 64, 0, None), (1 << 80, x, b, None), ("0", "x"), (b,) * 40]:
        assert f(*args) is None


def test_errors_without_a_gpu_are_the_python_path_s(monkeypatch):
    x, b = torch.zeros(4, 64, dtype=torch.bfloat16), torch.zeros(8192, dtype=torch.uint8)
    calls = [lambda: duqpp.rotq_gemm_tiled_packed(x, b, b, b, 4), lambda: duqpp.rotq_gemm_tiled(3, b, b, b, 4), lambda: duqpp.rotq_gemm(x, b, b, b),
             lambda: duqpp.rotate_quantize_tiled_packed(x, b), lambda: duqpp.quantize_weights_tiled(x, b),
             lambda: duqpp.mxfp4_gemm_tiled(b, b, b, b, 4, 4, 64), lambda: duqpp.group_error(x, b)]

    def seen():
        out = []
        for c in calls:
            with pytest.raises(Exception) as e:
                c()
            out.append((type(e.value), str(e.value)))
        return out

    native = seen()
    monkeypatch.setattr(binding, "_calls", Never)
    assert native == seen()


@pytest.fixture(scope="module")
def data():
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((T, K + 64), generator=g, device="cuda").to(torch.bfloat16)[:, :K]
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    R = torch.linalg.qr(torch.randn((K // 32, 32, 32), generator=g, device="cuda"))[0].contiguous()
    return x, w, R, duqpp.pack_rotation(R)


def both_ways(monkeypatch, f, native=True):
    """f's results on the native path and on the Python path; native: that the former was taken."""
    taken = []

    class Watched:
        pass

    for n in ("linear", "rows", "product", "error"):
        setattr(Watched, n, staticmethod(lambda *a, n=n: (lambda r: (taken.append(r is not None), r)[1])(getattr(real, n)(*a))))
    real = binding._calls
    monkeypatch.setattr(binding, "_calls", Watched)
    a = f()
    monkeypatch.setattr(binding, "_calls", Never)
    b = f()
    monkeypatch.setattr(binding, "_calls", real)
    assert taken and all(t == native for t in taken)
    return a, b


def same(a, b):
    if isinstance(a, (tuple, list)):
        return type(a) is type(b) and len(a) == len(b) and all(same(p, q) for p, q in zip(a, b))
    if isinstance(a, torch.Tensor):
        return a.dtype == b.dtype and a.device == b.device and a.stride() == b.stride() and torch.equal(a, b)
    return type(a) is type(b) and a == b


@pytest.mark.gpu
@pytest.mark.parametrize("out_dtype", [duqpp.F32, duqpp.BF16])
def test_same_results(monkeypatch, data, out_dtype):
    x, w, R, Rp = data
    wr, wt = duqpp.quantize_weights(w, R), duqpp.quantize_weights_tiled(w, R)
    at = duqpp.rotate_quantize_tiled(x, R)
    t = torch.float32 if out_dtype == duqpp.F32 else torch.bfloat16
    ws = torch.empty(sum(duqpp.tiled_bytes(T, K)), dtype=torch.uint8, device="cuda")

    def wide():                                              # a result with a row stride of its own
        return torch.zeros((T, N + 8), dtype=t, device="cuda")[:, :N]

    for f in [lambda: duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N, out_dtype), lambda: duqpp.rotq_gemm_tiled(x, R, *wt, N, out_dtype=out_dtype, workspace=ws),
              lambda: duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N, out_dtype=out_dtype, out=wide(), workspace=ws), lambda: duqpp.rotq_gemm(x, R, *wr, out_dtype),
              lambda: duqpp.rotq_gemm(x, R[:1].contiguous(), *wr, out_dtype=out_dtype, out=wide()), lambda: duqpp.mxfp4_gemm_tiled(*at, *wt, T, N, K, out_dtype),
              lambda: duqpp.mxfp4_gemm_tiled(*at, *wt, T, N, K, out_dtype=out_dtype, out=wide()), lambda: duqpp.rotate_quantize_tiled(x, R),
              lambda: duqpp.rotate_quantize_tiled_packed(x, Rp), lambda: duqpp.quantize_weights_tiled(w, R, out=tuple(torch.zeros_like(v) for v in wt)),
              lambda: duqpp.group_error(x, R), lambda: duqpp.group_error(x), lambda: duqpp.group_error(x.repeat(100, 1), R)]:
        a, b = both_ways(monkeypatch, f)
        torch.cuda.synchronize()
        assert same(a, b)


@pytest.mark.gpu
def test_same_objects_streams_and_errors(monkeypatch, data):
    x, w, R, Rp = data
    wt = duqpp.quantize_weights_tiled(w, R)
    y = torch.empty((T, N), device="cuda")
    a, b = both_ways(monkeypatch, lambda: duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N, out=y))
    assert a is y and b is y
    c = tuple(torch.empty_like(v) for v in wt)
    a, b = both_ways(monkeypatch, lambda: duqpp.quantize_weights_tiled(w, R, out=c))
    assert type(a) is type(b) and a[0] is c[0] is b[0] and a[1] is c[1] is b[1]

    # on a stream of the caller's, behind work that it has queued there
    want = duqpp.rotq_gemm_tiled_packed(x * 2, Rp, *wt, N)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        late = x.clone()
        torch.cuda._sleep(2000000)
        late.mul_(2)
        got = duqpp.rotq_gemm_tiled_packed(late, Rp, *wt, N)
        err, mean = duqpp.group_error(late, R)
    side.synchronize()
    assert torch.equal(got, want) and mean == duqpp.group_error(x * 2, R)[1]

    # the library's own refusals
    small, odd = torch.empty(256, dtype=torch.uint8, device="cuda"), torch.empty(1 << 20, dtype=torch.uint8, device="cuda")[16:]
    for f in [lambda: duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N, workspace=small), lambda: duqpp.rotq_gemm_tiled(x, R, *wt, N, workspace=odd),
              lambda: duqpp.rotate_quantize_tiled(x[:, 1:][:, :K - 32].contiguous()[:, :32 * 3], R[:3].contiguous()[:2].contiguous())]:
        seen = []
        for path in (binding._calls, Never):
            monkeypatch.setattr(binding, "_calls", path)
            with pytest.raises(duqpp.DuqppError) as e:
                f()
            seen.append((e.value.status, str(e.value)))
        monkeypatch.undo()
        assert seen[0] == seen[1]


@pytest.mark.gpu
def test_modes_and_subclasses_take_the_python_path(monkeypatch, data):
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    x, w, R, Rp = data
    wt = duqpp.quantize_weights_tiled(w, R)

    class Sub(torch.Tensor):
        pass

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    plain = duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N)
    for mode in (Function, Dispatch):
        def f():
            with mode():
                return duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N)
        a, b = both_ways(monkeypatch, f, native=False)
        assert torch.equal(a, plain) and torch.equal(b, plain)
    a, b = both_ways(monkeypatch, lambda: duqpp.rotq_gemm_tiled_packed(x.as_subclass(Sub), Rp, *wt, N), native=False)
    assert torch.equal(a, plain) and type(a) is type(b)
    p = torch.nn.Parameter(Rp, requires_grad=False)          # what a module's weights are
    a, b = both_ways(monkeypatch, lambda: duqpp.rotq_gemm_tiled_packed(x, p, *wt, N))
    assert torch.equal(a, plain) and torch.equal(b, plain)


@pytest.mark.gpu
def test_function_transforms_end_as_on_the_python_path(monkeypatch, data):
    """Under vmap, grad and functionalization tensors have no memory to pass on; a tensor from outside still has, with the result's not."""
    x, w, R, Rp = data
    wt = duqpp.quantize_weights_tiled(w, R)
    calls = [lambda v: duqpp.rotq_gemm_tiled_packed(v, Rp, *wt, N), lambda v: duqpp.rotate_quantize_tiled(v, R)[0], lambda v: duqpp.group_error(v, R)[0],
             lambda v: duqpp.rotq_gemm_tiled_packed(x, Rp, *wt, N) + v.sum(), lambda v: duqpp.group_error(x, R)[0].sum() + v.sum()]
    transforms = [lambda f: torch.func.vmap(f)(x.expand(2, T, K)), lambda f: torch.func.grad(lambda v: f(v).sum().float())(x),
                  lambda f: torch.func.functionalize(f)(x), lambda f: torch.func.jvp(f, (x,), (x,))]

    def ends(f):
        try:
            r = f()
            return r if isinstance(r, torch.Tensor) else [v for v in r]
        except Exception as e:
            return type(e), str(e).split("\n")[0]

    for transform in transforms:
        for call in calls:
            native = ends(lambda: transform(call))
            with monkeypatch.context() as m:
                m.setattr(binding, "_calls", Never)
                python = ends(lambda: transform(call))
            assert type(native) is type(python), (native, python)
            assert native == python if isinstance(native, tuple) else same(native, python)


@pytest.mark.gpu
def test_two_threads_on_two_streams(data):
    """Each thread its own stream, tensors and results, with the interpreter let go during the launches."""
    import threading
    x, w, R, Rp = data
    wt, wr = duqpp.quantize_weights_tiled(w, R), duqpp.quantize_weights(w, R)
    inputs = [x * (i + 1) for i in range(4)]
    want = [(duqpp.rotq_gemm_tiled_packed(v, Rp, *wt, N), duqpp.rotq_gemm(v, R, *wr), duqpp.group_error(v, R)) for v in inputs]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        try:
            side = torch.cuda.Stream()
            with torch.cuda.stream(side):
                for _ in range(50):
                    y, z, e = duqpp.rotq_gemm_tiled_packed(inputs[i], Rp, *wt, N), duqpp.rotq_gemm(inputs[i], R, *wr), duqpp.group_error(inputs[i], R)
                    side.synchronize()
                    if not (torch.equal(y, want[i][0]) and torch.equal(z, want[i][1]) and same(e, want[i][2])):
                        wrong.append(i)
        except BaseException as e:
            wrong.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.gpu
def test_captured_once_and_replayed(data):
    """Calls through the native path in a graph, results and workspaces from the graph's pool: every replay, between other work, gives what
    eager calls do."""
    x, w, R, Rp = data
    wt, wr = duqpp.quantize_weights_tiled(w, R), duqpp.quantize_weights(w, R)
    held = x.clone(memory_format=torch.contiguous_format)

    def f():
        a = duqpp.rotate_quantize_tiled_packed(held, Rp)
        return (duqpp.rotq_gemm_tiled_packed(held, Rp, *wt, N, duqpp.BF16), duqpp.rotq_gemm(held, R, *wr), duqpp.mxfp4_gemm_tiled(*a, *wt, T, N, K),
                duqpp.group_error(held, R, return_mean=False)[0], *a)

    f()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = f()
    for i in range(4):
        held.copy_(x * (i + 1))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, f()))
        torch.ones(1 << 16, device="cuda").sum().item()


@pytest.mark.gpu
def test_compiled_callers(data):
    """A function that dynamo traces: it breaks its graph at the call, as it did at the Python path's, and the result is the eager one."""
    x, w, R, Rp = data
    wt = duqpp.quantize_weights_tiled(w, R)

    def f(v):
        return duqpp.rotq_gemm_tiled_packed(v * 2, Rp, *wt, N) + 1

    want = f(x)
    torch._dynamo.reset()
    got = torch.compile(f, backend="eager")(x)
    assert torch.equal(got, want)
