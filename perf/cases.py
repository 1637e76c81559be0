"""Performance cases of the DuQuant++ path: the calls a program makes when it prepares, serves or analyses a model.

Kinds of case
  linear    one linear layer online, Y = Q(X R) Q(R^T W): eager calls on weights kept in the tiled layout
  layer     the seven linears of a LLaMA-3-8B decoder layer, one after the other, each with its own rotation blocks:
            eager calls, or one HIP graph that holds them (how a decode loop is served)
  rowmajor  one linear whose weights are kept in the row-major interchange layout
  weights   the offline transform of one weight matrix (rotate, quantise, tiled layout)
  error     the per-group quantisation error of a batch of activations
  construct the greedy construction of the shared rotation block from calibration activations

Inputs follow the synthetic recipe of the repository's workloads: X normal with outlier channels and a few massive
values, W normal with a small deviation, R orthogonal per block of 32 channels.
"""
import numpy as np
import torch

import paper_2604_17789_amd as duqpp

BLOCK = 32
# K, N of the linears of LLaMA-3-8B and of the LLaMA-3-70B down, gate/up and square projections
LAYER = {"q": (4096, 4096), "k": (4096, 1024), "v": (4096, 1024), "o": (4096, 4096),
         "gate": (4096, 14336), "up": (4096, 14336), "down": (14336, 4096)}
SHAPES = [(4096, 4096), (4096, 1024), (4096, 14336), (14336, 4096), (8192, 8192), (8192, 28672), (28672, 8192)]
MOST_MACS = 4096 * 28672 * 8192          # what one drawn linear may cost: the 70B down projection at 4096 tokens


def listed():
    return [
        # decoding one sequence: every linear of a layer for one token, launched as one graph
        dict(name="decode_layer_T1", kind="layer", T=1, graph=True, out="bf16", blocks="own"),
        # decoding a batch of 16 sequences with eager calls: latency of the calls themselves counts
        dict(name="decode_layer_T16", kind="layer", T=16, graph=False, out="bf16", blocks="own"),
        # 64 tokens through q_proj, fp32 rotation blocks and fp32 result (the parity reference's shape)
        dict(name="qproj_T64", kind="linear", T=64, K=4096, N=4096, out="f32", entry="fp32", blocks="own", pad=0),
        # a chunk of prompt tokens of no round number through gate/up, one block shared by all groups
        dict(name="chunk_gateup_T333", kind="linear", T=333, K=4096, N=14336, out="bf16", entry="packed", blocks="shared", pad=0),
        # the same through down, with a long reduction axis
        dict(name="chunk_down_T777", kind="linear", T=777, K=14336, N=4096, out="bf16", entry="packed", blocks="own", pad=0),
        # prefill of 2048 tokens through down: the benchmark's headline workload
        dict(name="prefill_down_T2048", kind="linear", T=2048, K=14336, N=4096, out="bf16", entry="packed", blocks="own", pad=0),
        # prefill of 8192 tokens through every linear of a layer: the largest
        dict(name="prefill_layer_T8192", kind="layer", T=8192, graph=False, out="bf16", blocks="own"),
        # the 70B down projection with rotate+quantise and product as separate calls, fp32 result
        dict(name="prefill_70b_down_T4096", kind="linear", T=4096, K=28672, N=8192, out="f32", entry="separate", blocks="own", pad=0),
        # weights as they are exchanged and stored: row-major codes and scales
        dict(name="rowmajor_qproj_T512", kind="rowmajor", T=512, K=4096, N=4096, out="f32", blocks="own"),
        # preparing a model: rotate and quantise a gate/up weight matrix
        dict(name="weights_gateup", kind="weights", N=14336, K=4096, blocks="own"),
        # looking at a model: quantisation error of 2048 tokens' activations per group, and its mean
        dict(name="error_T2048", kind="error", T=2048, K=4096, blocks="own"),
        # calibrating a model: 128 greedy steps on 2048 tokens' activations
        dict(name="construct_T2048", kind="construct", T=2048, K=4096, steps=128),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _shape(rng):
    """K, N of a linear: mostly a model's, else a generic pair (K a multiple of 32, N a multiple of 8 or anything)."""
    if rng.random() < 0.6:
        return rng.choice(SHAPES)
    return BLOCK * _log_uniform(rng, 16, 448), _log_uniform(rng, 64, 1792) * 8 - rng.choice((0, 0, 0, 3))


def draw(rng):
    kind = rng.choices(("linear", "layer", "rowmajor", "weights", "error", "construct"), (10, 2, 2, 2, 1, 1))[0]
    blocks = rng.choice(("own", "own", "shared"))
    out = rng.choice(("bf16", "bf16", "f32"))
    if kind == "linear":
        K, N = _shape(rng)
        T = _log_uniform(rng, 1, max(1, min(8192, MOST_MACS // (K * N))))
        return dict(kind=kind, T=T, K=K, N=N, out=out, entry=rng.choice(("packed", "packed", "fp32", "separate")), blocks=blocks,
                    pad=rng.choice((0, 0, 0, 64)))
    if kind == "layer":
        graph = rng.random() < 0.5
        return dict(kind=kind, T=_log_uniform(rng, 1, 64 if graph else 6000), graph=graph, out=out, blocks=blocks)
    if kind == "rowmajor":
        K, N = _shape(rng)
        return dict(kind=kind, T=_log_uniform(rng, 1, max(1, min(4096, MOST_MACS // (K * N)))), K=K, N=N, out=out, blocks=blocks)
    if kind == "weights":
        K, N = _shape(rng)
        return dict(kind=kind, N=N, K=K, blocks=blocks)
    if kind == "error":
        return dict(kind=kind, T=_log_uniform(rng, 64, 8192), K=BLOCK * _log_uniform(rng, 16, 448), blocks=blocks)
    return dict(kind=kind, T=_log_uniform(rng, 64, 8192), K=BLOCK * _log_uniform(rng, 16, 448), steps=_log_uniform(rng, 16, 192))


# ---- inputs ----------------------------------------------------------------------------------------------------------

def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + what) % (1 << 62))


def _orthogonal(seed, what, count, n, dtype):
    rng = np.random.default_rng([int(seed), what])
    q, r = np.linalg.qr(rng.standard_normal((count, n, n)))
    q = q * np.where(np.diagonal(r, axis1=1, axis2=2) < 0, -1.0, 1.0)[:, None, :]
    return torch.from_numpy(np.ascontiguousarray(q.astype(dtype))).cuda()


def _rotation(seed, what, K, blocks):
    return _orthogonal(seed, what, 1 if blocks == "shared" else K // BLOCK, BLOCK, np.float32)


def _activations(seed, what, T, K, pad=0):
    g = _gen(seed, what)
    x = torch.empty((T, K + pad), dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 2048):
        x[t:t + 2048] = torch.randn((min(2048, T - t), K + pad), generator=g, device="cuda")
    x = x[:, :K]
    x[:, torch.randperm(K, generator=g, device="cuda")[:8]] *= 50.0
    x[torch.randint(0, T, (8,), generator=g, device="cuda"), torch.randint(0, K, (8,), generator=g, device="cuda")] = 900.0
    return x


def _weights(seed, what, N, K):
    g = _gen(seed, what)
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    for n in range(0, N, 2048):
        w[n:n + 2048] = torch.randn((min(2048, N - n), K), generator=g, device="cuda") * 0.02
    return w


def _dtype(out):
    return (duqpp.F32, torch.float32) if out == "f32" else (duqpp.BF16, torch.bfloat16)


def _workspace(T, K):
    codes, scales = duqpp.tiled_bytes(T, K)
    return torch.empty(((codes + 255) // 256 + (scales + 255) // 256) * 256, dtype=torch.uint8, device="cuda")


def _layer_calls(s):
    return [duqpp.rotq_gemm_tiled_packed(x, rp, bc, bs, N, out_dtype=s["out_dtype"], out=y, workspace=ws)
            for x, rp, bc, bs, N, y, ws in s["linears"]]


def prepare(case, seed):
    kind, K, T = case["kind"], case.get("K"), case.get("T")
    duqpp.init()
    if kind == "layer":
        code, torch_type = _dtype(case["out"])
        s = dict(kind=kind, out_dtype=code, linears=[], graph=None)
        for i, (K, N) in enumerate(LAYER.values()):
            R = _rotation(seed, 3 * i, K, case["blocks"])
            bc, bs = duqpp.quantize_weights_tiled(_weights(seed, 3 * i + 1, N, K), R)
            s["linears"].append((_activations(seed, 3 * i + 2, T, K), duqpp.pack_rotation(R), bc, bs, N,
                                 torch.empty((T, N), dtype=torch_type, device="cuda"), _workspace(T, K)))
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _layer_calls(s)
            torch.cuda.current_stream().wait_stream(side)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                _layer_calls(s)
        return s
    if kind == "construct":
        return dict(kind=kind, x=_activations(seed, 1, T, K), q=_orthogonal(seed, 2, case["steps"], BLOCK - 1, np.float64))
    R = _rotation(seed, 0, K, case["blocks"])
    if kind == "error":
        return dict(kind=kind, x=_activations(seed, 1, T, K), R=R)
    if kind == "weights":
        codes, scales = duqpp.tiled_bytes(case["N"], K)
        return dict(kind=kind, w=_weights(seed, 1, case["N"], K), R=R,
                    kept=(torch.empty(codes, dtype=torch.uint8, device="cuda"), torch.empty(scales, dtype=torch.uint8, device="cuda")))
    w = _weights(seed, 1, case["N"], K)
    s = dict(kind=kind, x=_activations(seed, 2, T, K, case.get("pad", 0)), R=R, T=T, K=K, N=case["N"], out_dtype=_dtype(case["out"])[0])
    if kind == "rowmajor":
        s["b"] = duqpp.quantize_weights(w, R)
        s["workspace"] = torch.empty(duqpp.gemm_workspace_bytes(T, case["N"], K, True), dtype=torch.uint8, device="cuda")
        return s
    s["entry"], s["b"], s["workspace"] = case["entry"], duqpp.quantize_weights_tiled(w, R), _workspace(T, K)
    if s["entry"] != "fp32":
        s["Rp"] = duqpp.pack_rotation(R)
    if s["entry"] == "separate":
        codes, scales = duqpp.tiled_bytes(T, K)
        s["a"] = (torch.empty(codes, dtype=torch.uint8, device="cuda"), torch.empty(scales, dtype=torch.uint8, device="cuda"))
    return s


def run(s):
    kind = s["kind"]
    if kind == "layer":
        if s["graph"] is None:
            return _layer_calls(s)
        s["graph"].replay()
        return [y for _, _, _, _, _, y, _ in s["linears"]]
    if kind == "construct":
        return duqpp.construct_rotation(s["x"], s["q"], return_peaks=True)
    if kind == "error":
        return duqpp.group_error(s["x"], s["R"])
    if kind == "weights":
        return duqpp.quantize_weights_tiled(s["w"], s["R"], out=s["kept"])
    if kind == "rowmajor":
        return duqpp.rotq_gemm(s["x"], s["R"], *s["b"], out_dtype=s["out_dtype"], workspace=s["workspace"])
    if s["entry"] == "packed":
        return duqpp.rotq_gemm_tiled_packed(s["x"], s["Rp"], *s["b"], s["N"], out_dtype=s["out_dtype"], workspace=s["workspace"])
    if s["entry"] == "fp32":
        return duqpp.rotq_gemm_tiled(s["x"], s["R"], *s["b"], s["N"], out_dtype=s["out_dtype"], workspace=s["workspace"])
    a = duqpp.rotate_quantize_tiled_packed(s["x"], s["Rp"], out=s["a"])
    y = duqpp.mxfp4_gemm_tiled(*a, *s["b"], s["T"], s["N"], s["K"], out_dtype=s["out_dtype"])
    return a + (y,)


# ---- what a pass cannot do without, and how far two correct implementations may be apart ----------------------------

MX = 0.5 + 1.0 / BLOCK                   # bytes of one MXFP4 value: half a byte of code, 1/32 byte of scale


def _linear_work(T, K, N, case):
    packed = case.get("entry", "packed") in ("packed", "separate") and case["kind"] != "rowmajor"
    blocks = 1 if case["blocks"] == "shared" else K // BLOCK
    out = 4 if case["out"] == "f32" else 2
    extra = T * K * MX if case.get("entry") == "separate" else 0       # the codes are an output of their own
    return (2.0 * T * K + blocks * (6144 if packed else 4096) + N * K * MX + T * N * out + extra,
            2.0 * T * N * K + 2.0 * T * K * BLOCK)


def work(case):
    kind, T, K = case["kind"], case.get("T"), case.get("K")
    blocks = 1 if case.get("blocks") == "shared" else (K or 0) // BLOCK
    if kind == "layer":
        parts = [_linear_work(T, K, N, case) for K, N in LAYER.values()]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if kind in ("linear", "rowmajor"):
        by, fl = _linear_work(T, K, case["N"], case)
        return {"bytes": by, "flops": fl}
    if kind == "weights":
        N = case["N"]
        return {"bytes": 2.0 * N * K + blocks * 4096 + N * K * MX, "flops": 2.0 * N * K * BLOCK}
    if kind == "error":
        return {"bytes": 2.0 * T * K + blocks * 4096 + T * (K // BLOCK) * 4, "flops": 2.0 * T * K * BLOCK}
    n = case["steps"]
    return {"bytes": 2.0 * T * K + n * 31 * 31 * 8 + 4096 + 8 * (n + 1),
            "flops": n * (2.0 * T * BLOCK * BLOCK + 4.0 * BLOCK ** 3)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("weights", "construct"):
        return "exact"                   # bytes; fp64 in a stated order
    if kind == "error":
        return {"rel": 4e-7, "max": 4e-6}    # fp32 ratios of fp64 sums
    # The codes are bytes and the same for any correct implementation of the rotation used here; the products are exact,
    # so only the order of the fp32 sums is free (against fp64 sums: no difference seen at K = 4096 to 28672).  A bf16
    # result may land on the neighbouring value (2^-7) where the sum falls near a tie.
    if case["out"] == "f32":
        return {"rel": 2e-6, "max": 2e-4}
    return {"rel": 4e-4, "max": 1.6e-2}
