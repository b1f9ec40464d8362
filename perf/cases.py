"""Performance cases: what a program that uses this library has it do, with real sizes and through the
public entry points of the binding and the layer chain.

    listed()  the cases;  draw(rng)  one more case of the same ranges
    prepare(case, seed)  weights, plans and inputs on the GPU;  run(state)  one pass, outputs whole
    work(case)  bytes and operations of a pass;  tolerance(case);  exact(case, seed)  the outputs in 64 bits

Weights are N(0, 0.02^2) latents packed by the library; activations are N(0, 1) with one channel in a
hundred twenty times as large (the outliers a per-token quantiser meets), squared behind a ReLU where
they feed a down projection.  The 2B-style layer is the one of chain.SHAPES.
"""
import math

import torch

from paper_2504_12285_amd import binding as bl
from paper_2504_12285_amd import chain

DEV = "cuda"
HIDDEN, FFN = 2560, 6912          # the 2B-style layer: qkv 3840, o 2560, gate+up 13824, down 2560
LAYERS_2B = 30


def listed():
    return [
        # the smallest call: one token through one projection, called eagerly (time to the answer)
        {"name": "decode_one", "kind": "decode", "M": 1, "N": 2560, "K": 2560, "layout": 1},
        # a server's decode step written call by call: sixteen sequences, quantise + product for each projection
        {"name": "batch_calls_m16", "kind": "calls", "M": 16, "hidden": HIDDEN, "ffn": FFN, "layout": 1},
        # the latency of one generated token: thirty dependent layers with RMS normalisation, one HIP graph
        {"name": "token_chain_m1", "kind": "token", "M": 1, "layers": LAYERS_2B, "norm": True, "layout": 1},
        # the weight stream of a whole 2B-style stack at one token (the library's headline workload)
        {"name": "stream_m1", "kind": "stream", "M": 1, "layers": LAYERS_2B, "hidden": HIDDEN, "ffn": FFN, "layout": 1},
        # the same stack in the smaller footprint, five weights per byte
        {"name": "stream_five_m1", "kind": "stream", "M": 1, "layers": LAYERS_2B, "hidden": HIDDEN, "ffn": FFN, "layout": 2},
        # batched decode of the stack: a few sequences, and as many as the batched form takes
        {"name": "stream_m8", "kind": "stream", "M": 8, "layers": LAYERS_2B, "hidden": HIDDEN, "ffn": FFN, "layout": 1},
        {"name": "stream_m64", "kind": "stream", "M": 64, "layers": LAYERS_2B, "hidden": HIDDEN, "ffn": FFN, "layout": 1},
        # prompt processing: the four projections of a layer at 2048 tokens (quantise + product)
        {"name": "prefill_m2048", "kind": "prefill", "M": 2048, "hidden": HIDDEN, "ffn": FFN, "layout": 1},
        # sizes that divide by nothing: a short prompt, a matrix with ragged rows and columns
        {"name": "prefill_ragged", "kind": "gemm", "M": 777, "N": 5003, "K": 2999, "layout": 1},
        # weights in the plain bit order of a checkpoint, a prompt of a thousand tokens
        {"name": "prefill_rowmajor", "kind": "gemm", "M": 1000, "N": 3840, "K": 2560, "layout": 0},
        # a long prompt through whole layers: fused residual / gate epilogues and one-pass quantisers
        {"name": "prefill_chain_m4096", "kind": "prompt", "M": 4096, "layers": 2, "norm": False, "layout": 1},
        # loading a model: ternarize and pack the widest matrix of the layer
        {"name": "pack_gate_up", "kind": "pack", "N": 13824, "K": 2560, "layout": 1, "source": "fp32"},
    ]


def _log(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    kind = rng.choice(["decode", "calls", "token", "stream", "stream", "prefill", "gemm", "gemm", "prompt", "pack"])
    if kind == "decode":
        M, K = _log(rng, 1, 16), _log(rng, 256, 8192, 64)
        while M * (K + 16) > 96 * 1024:
            M -= 1
        return {"kind": kind, "M": M, "N": _log(rng, 256, 14000), "K": K, "layout": rng.choice([0, 1, 1])}
    if kind in ("calls", "prefill"):
        M = _log(rng, 1, 64) if kind == "calls" else _log(rng, 65, 3000)
        hidden = _log(rng, 640, 2560, rng.choice([1, 64, 128]))
        return {"kind": kind, "M": M, "hidden": hidden, "ffn": _log(rng, 2 * hidden, int(2.7 * hidden), rng.choice([1, 64, 128])),
                "layout": rng.choice([0, 1, 1])}
    if kind == "token":
        return {"kind": kind, "M": _log(rng, 1, 8), "layers": rng.randint(2, 15), "norm": rng.random() < 0.5, "layout": 1}
    if kind == "stream":
        M = rng.choice([1, 1, _log(rng, 2, 64)])
        hidden = _log(rng, 640, 4096, 64)
        ffn = _log(rng, 2 * hidden, 3 * hidden, 64)
        most = int(500e6 / (sum(n * k for _, n, k in _layer(hidden, ffn)) / 4))
        return {"kind": kind, "M": M, "layers": max(1, min(_log(rng, 1, 60), most)), "hidden": hidden, "ffn": ffn,
                "layout": rng.choice([0, 1, 2]) if M == 1 else 1}
    if kind == "gemm":
        M = _log(rng, 65, 4096)
        return {"kind": kind, "M": M, "N": _log(rng, 300, 14000), "K": _log(rng, 300, 7000, rng.choice([1, 64, 128])),
                "layout": rng.choice([0, 1])}
    if kind == "prompt":
        return {"kind": kind, "M": _log(rng, 65, 4096), "layers": rng.choice([1, 2]), "norm": rng.random() < 0.5, "layout": 1}
    step = rng.choice([1, 64])
    layout = rng.choice([0, 1, 1, 2, 3])
    return {"kind": kind, "N": _log(rng, 300, 3000 if layout == 3 else 14000, step), "K": _log(rng, 300, 7000, step),
            "layout": layout, "source": rng.choice(["fp32", "fp32", "int8"])}


# ---- sizes -------------------------------------------------------------------------------------

def _layer(hidden, ffn):
    """(name, N, K) of the four projections; a fused qkv with a quarter of the heads for k and for v."""
    return [("qkv", hidden + 2 * (hidden // 4), hidden), ("o", hidden, hidden), ("gate_up", 2 * ffn, hidden), ("down", hidden, ffn)]


def _products(case):
    """(name, M, N, K) of every product of a pass."""
    kind = case["kind"]
    if kind in ("decode", "gemm"):
        return [("o", case["M"], case["N"], case["K"])]
    if kind in ("token", "prompt"):
        return [(n, case["M"], N, K) for _ in range(case["layers"]) for n, (N, K) in chain.SHAPES.items()]
    return [(n, case["M"], N, K) for _ in range(case.get("layers", 1)) for n, N, K in _layer(case["hidden"], case["ffn"])]


# ---- inputs ------------------------------------------------------------------------------------

def _rng(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _latent(g, N, K):
    return torch.randn((N, K), generator=g, device=DEV) * 0.02


def _activations(g, M, K, name):
    x = torch.randn((M, K), generator=g, device=DEV)
    outliers = torch.randperm(K, generator=g, device=DEV)[: max(1, round(0.01 * K))]
    x[:, outliers] *= 20.0
    x = x.to(torch.bfloat16)
    return torch.relu(x).square() if name == "down" else x


def _gains(g, case):
    if not case["norm"]:
        return None
    return {n: 1.0 + 0.1 * torch.randn(K, generator=g, device=DEV) for n, (N, K) in chain.SHAPES.items()}


def _chain_inputs(g, case):
    """Latent weights and gains, layer by layer, in one order for prepare and exact."""
    for _ in range(case["layers"]):
        yield {n: _latent(g, N, K) for n, (N, K) in chain.SHAPES.items()}, _gains(g, case)


def _pack_source(g, case):
    W = _latent(g, case["N"], case["K"])
    if case["source"] == "fp32":
        return W, None
    return (W / 0.016).round().clamp(-1, 1).to(torch.int8), torch.full((1,), 0.016, device=DEV)


def prepare(case, seed):
    g, kind, layout = _rng(seed), case["kind"], case.get("layout")
    st = {"kind": kind, "case": dict(case)}
    if kind == "pack":
        st["W"], st["beta"] = _pack_source(g, case)
    elif kind in ("token", "prompt"):
        st["x"] = torch.randn((case["M"], HIDDEN), generator=g, device=DEV)
        weights, gains = [], []
        for W, G in _chain_inputs(g, case):
            weights.append({n: bl.bl_pack_ternary(w, layout) for n, w in W.items()})
            gains.append(G)
        st["weights"], st["gains"] = weights, gains if case["norm"] else None
        if kind == "token":
            _capture_token(st, case)
    elif kind == "stream":
        _build_stream(st, g, case)
    else:
        st["products"] = []
        for name, M, N, K in _products(case):
            packed, beta = bl.bl_pack_ternary(_latent(g, N, K), layout)
            st["products"].append((packed, beta, _activations(g, M, K, name), N, K))
    return st


def _capture_token(st, case):
    """One token through all layers, recorded into a HIP graph as a decode loop does."""
    B = chain.ChainBuffers(case["M"], torch.device(DEV))
    spare = torch.empty_like(B.x_next)

    def token():
        x, nxt, other = st["x"], B.x_next, spare
        for i, w in enumerate(st["weights"]):
            B.x_next = nxt
            x = chain.layer_decode(w, case["layout"], x, B, None, None if st["gains"] is None else st["gains"][i])
            nxt, other = other, nxt
        return x

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        token()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st["out"] = token()
    st["graph"], st["keep"] = graph, (B, spare)


def _build_stream(st, g, case):
    M, layout = case["M"], case["layout"]
    products = _products(case)
    y = torch.empty(sum(M * N for _, M, N, _ in products), dtype=torch.float32, device=DEV)
    items, at = [], 0
    for name, M, N, K in products:
        packed, beta = bl.bl_pack_ternary(_latent(g, N, K), layout)
        X = _activations(g, M, K, name)
        item = {"packed": packed, "beta": beta, "N": N, "K": K, "y": y[at:at + M * N]}
        if M == 1:
            item["X"] = X
        else:
            item["q"], item["scale"], item["rowsum"] = bl.bl_quant_act_int8(X)
        items.append(item)
        at += M * N
    st["stack"], st["y"] = bl.Stack(items, layout, M, torch.device(DEV)), y


# ---- one pass ----------------------------------------------------------------------------------

def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "stream":
        st["stack"].run()
        return st["y"]
    if kind == "token":
        st["graph"].replay()
        return st["out"]
    if kind == "prompt":
        return chain.run_chain(st["weights"], case["layout"], st["x"], "prefill", layer_gains=st["gains"])
    if kind == "pack":
        return bl.bl_pack_ternary(st["W"], case["layout"], st["beta"])
    layout, out = case["layout"], []
    for packed, beta, X, N, K in st["products"]:
        if kind == "decode":
            out.append(bl.bl_bitlinear_decode(packed, beta, layout, X, N)[1])
        else:
            q, scale, rowsum = bl.bl_quant_act_int8(X)
            product = bl.bl_gemv_w158a8 if kind == "calls" else bl.bl_gemm_w158a8
            out.append(product(packed, beta, layout, q, scale, rowsum, N, want_acc=False, K=K)[1])
    return out


# ---- what a pass cannot do without ---------------------------------------------------------------

def work(case):
    """Packed weights once, each input once (bf16, or int8 where the path takes int8), each output once."""
    if case["kind"] == "pack":
        N, K = case["N"], case["K"]
        return {"bytes": N * K * (4 if case["source"] == "fp32" else 1) + bl.bl_packed_bytes(N, K, case["layout"]) + 4,
                "flops": 2 * N * K}
    products = _products(case)
    flops = sum(2 * M * N * K for _, M, N, K in products)
    weights = sum(bl.bl_packed_bytes(N, K, case["layout"]) for _, M, N, K in products)
    if case["kind"] in ("token", "prompt"):
        gains = 4 * sum(K for _, M, N, K in products) if case["norm"] else 0
        return {"bytes": weights + gains + 2 * 4 * case["M"] * HIDDEN, "flops": flops}
    per_input = 1 if case["kind"] == "stream" and case["M"] > 1 else 2
    return {"bytes": weights + sum(per_input * M * K + 4 * M * N for _, M, N, K in products), "flops": flops}


def tolerance(case):
    """The header fixes every floating-point step (one IEEE rounding each, exact integer sums), so every
    correct implementation gives the same bits."""
    return "exact"


# ---- the same in 64 bits, plain torch --------------------------------------------------------------

def _ternary64(W):
    W = W.double()
    beta = W.abs().mean()
    return (W / (beta + 1e-5)).round().clamp_(-1, 1), beta


def _quant64(x):
    g = x.abs().amax(dim=1, keepdim=True).clamp(min=1e-5)
    return (x * (127.0 / g)).round().clamp(-127, 127), g / 127.0


def _linear64(x, W, scale=None):
    """x: the bf16 values in 64 bits."""
    Wt, beta = _ternary64(W)
    q, s = _quant64(x)
    return (q @ Wt.t()) * (beta * (s if scale is None else scale))


def _chain64(case, x, layers):
    unit = None if case["norm"] else 1.0 / 127.0

    def bit(t, W, G, name):
        if G is not None:
            t = t / torch.sqrt(t.square().mean(dim=1, keepdim=True) + 1e-5) * G[name].double()
        return _linear64(t.to(torch.float32).to(torch.bfloat16).double(), W[name], unit)

    x, M = x.double(), case["M"]
    nq, nkv, hd = chain.N_Q, chain.N_KV, chain.HEAD_DIM
    for W, G in layers:
        qkv = bit(x, W, G, "qkv")
        v = qkv[:, (nq + nkv) * hd:].reshape(M, nkv, 1, hd).expand(M, nkv, nq // nkv, hd).reshape(M, nq * hd)
        h1 = x + bit(v, W, G, "o")
        gu = bit(h1, W, G, "gate_up")
        f = torch.relu(gu[:, :FFN]).square() * gu[:, FFN:]
        x = h1 + bit(f, W, G, "down")
    return x


def exact(case, seed):
    g, kind = _rng(seed), case["kind"]
    if kind == "pack":
        W, beta = _pack_source(g, case)
        return None, (W.double().abs().mean().reshape(1) if beta is None else beta.double())
    if kind in ("token", "prompt"):
        x = torch.randn((case["M"], HIDDEN), generator=g, device=DEV)
        return _chain64(case, x, _chain_inputs(g, case))
    out = []
    for name, M, N, K in _products(case):
        W = _latent(g, N, K)
        out.append(_linear64(_activations(g, M, K, name).double(), W))
    return torch.cat([o.reshape(-1) for o in out]) if kind == "stream" else out
