"""What the library is timed on: the work of an RL step that goes through its public entry points.

Four kinds of work, each over the range of sizes that it has in use:

``layer``  the linears of decoder layers as rollout and log-prob passes call them: RMSNorm -> FP8,
           q/k/v; row quantizer, o; RMSNorm -> FP8, gate/up, SiLU*up -> FP8, down.  Attention is not
           part of the library: its output is an input here.  `batch` counts token rows: 1 to 256
           for decode, up to a few thousand (ragged) for a log-prob or prefill pass.  `fused`: q/k/v
           and gate/up are one matrix each, as serving engines lay them out.  `graph`: the calls are
           captured once and replayed, as a decode loop does; otherwise they are made one by one.
``linear`` one linear layer's training step: weight quantization with the transposed copy, row
           quantization of X, FProp, row + column quantization of dY, DGrad, column quantization
           of the FP8-saved X, WGrad.
``mlp``    forward and backward of an MLP block on FP8-saved activations (mlp_block).
``sync``   weight synchronisation after an optimizer step (weight_sync.WeightStore).

Sizes are those of the 8B- and 32B-class layers of jet_inputs.py and of the small configuration of
the parity tests (256 x 1024 x 1024); values follow the recipes of jet_inputs.py, drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

import paper_2601_14243_amd as jet
from paper_2601_14243_amd import mlp_block
from paper_2601_14243_amd.weight_sync import WeightStore, shard_shape

HIDDEN_8B, KV_8B, INTER_8B = 4096, 1024, 14336
HIDDEN_32B, KV_32B, INTER_32B = 5120, 1024, 27648
EPS = 1e-6
MOST_FLOPS = 18.0 * 16384 * HIDDEN_8B * INTER_8B      # the largest listed case: the MLP block at 16384 tokens
MOST_BYTES = 2.0e9


def _layer(name, batch, sizes, layers, fused, graph):
    hidden, kv, inter = sizes
    return dict(name=name, kind="layer", batch=batch, hidden=hidden, kv=kv, inter=inter, layers=layers,
                fused=fused, graph=graph)


def listed():
    s8, s32 = (HIDDEN_8B, KV_8B, INTER_8B), (HIDDEN_32B, KV_32B, INTER_32B)
    return [
        # the last long answer of a rollout batch: one row, a captured decode loop, weights from HBM
        _layer("decode_b1_8b", 1, s8, 4, True, True),
        # a small batch in an engine that does not capture graphs and keeps the matrices apart
        _layer("decode_b8_8b_eager", 8, s8, 1, False, False),
        # the usual decode batches: moderate, the largest one of the 8B-class runs, and a ragged one between
        _layer("decode_b32_8b", 32, s8, 4, False, True),
        _layer("decode_b77_8b", 77, s8, 4, True, True),
        _layer("decode_b128_8b", 128, s8, 4, True, True),
        # the same of the 32B class
        _layer("decode_b64_32b", 64, s32, 2, True, True),
        _layer("decode_b256_32b", 256, s32, 2, True, True),
        # log-probs of one answer: a ragged number of tokens through the training forward
        _layer("logprob_1000_8b", 1000, s8, 1, False, False),
        # training step of a small linear: seven short launches
        dict(name="linear_256_1k", kind="linear", tokens=256, out=1024, inp=1024),
        # training step of the narrow k/v projection over a micro-batch
        dict(name="linear_16k_kv_8b", kind="linear", tokens=16384, out=KV_8B, inp=HIDDEN_8B),
        # the bulk of a training step: the MLP block over a micro-batch
        dict(name="mlp_16k_8b", kind="mlp", tokens=16384, hidden=HIDDEN_8B, inter=INTER_8B),
        # every weight re-quantized after the update
        dict(name="sync_8b", kind="sync", hidden=HIDDEN_8B, kv=KV_8B, inter=INTER_8B, layers=2, tp=1,
             transposed=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_128(rng, lo, hi):
    return 128 * max(1, _log_int(rng, lo // 128, hi // 128))


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


def _draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "layer", "linear", "mlp", "sync"))
    sizes = rng.choice(((HIDDEN_8B, KV_8B, INTER_8B), (HIDDEN_32B, KV_32B, INTER_32B),
                        (_log_128(rng, 1024, 8192), rng.choice((512, 1024)), _log_128(rng, 3072, 28672))))
    hidden, kv, inter = sizes
    if kind == "layer":
        big = rng.random() < 0.25
        batch = _log_int(rng, 257, 4096) if big else _log_int(rng, 1, 256)
        per_layer = 2 * hidden * hidden + 2 * kv * hidden + 3 * inter * hidden
        layers = 1 if big else max(1, min(4, int(900e6 / per_layer)))
        return {k: v for k, v in _layer("", batch, sizes, layers, rng.random() < 0.5,
                                        not big and rng.random() < 0.75).items() if k != "name"}
    if kind == "linear":
        return dict(kind="linear", tokens=_log_128(rng, 128, 16384), out=_log_128(rng, 512, 14336),
                    inp=_log_128(rng, 512, 14336))
    if kind == "mlp":
        return dict(kind="mlp", tokens=_log_128(rng, 512, 16384), hidden=hidden, inter=inter)
    tp = rng.choice((1, 2)) if inter in (INTER_8B, INTER_32B) else 1
    return dict(kind="sync", hidden=hidden, kv=kv, inter=inter, layers=rng.choice((1, 2)), tp=tp,
                transposed=rng.random() < 0.5)


# ------------------------------------------------------------------ inputs --

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _activations(g, M, K):
    """N(0,1) with one channel in a hundred 50 times as large."""
    x = torch.randn((M, K), generator=g, device="cuda")
    x[:, torch.randperm(K, generator=g, device="cuda")[:-(-K // 100)]] *= 50.0
    return x.to(torch.bfloat16)


def _weights(g, N, K):
    return (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)


def _grads(g, M, N):
    """N(0,1e-3) with 0.5 % of the entries heavy-tailed (Student-t with 3 degrees of freedom)."""
    dy = torch.randn((M, N), generator=g, device="cuda")
    heavy = torch.rand((M, N), generator=g, device="cuda") < 0.005
    n = int(heavy.sum())
    chi = torch.randn((3, n), generator=g, device="cuda").square().sum(0) / 3.0
    dy[heavy] = torch.randn(n, generator=g, device="cuda") / chi.sqrt()
    dy *= 1e-3
    return dy.to(torch.bfloat16)


def _gamma(g, K):
    return (1.0 + 0.1 * torch.randn((K,), generator=g, device="cuda")).to(torch.bfloat16)


def _matrices(c):
    H, kv, I = c["hidden"], c["kv"], c["inter"]
    return (("q_proj", H, H), ("k_proj", kv, H), ("v_proj", kv, H), ("o_proj", H, H),
            ("gate_proj", I, H), ("up_proj", I, H), ("down_proj", H, I))


def prepare(case, seed):
    g = _gen(seed)
    c = dict(case)
    if c["kind"] == "layer":
        H, kv, I, M = c["hidden"], c["kv"], c["inter"], c["batch"]
        layers = []
        for _ in range(c["layers"]):
            q = lambda N, K: jet.quant_weight(_weights(g, N, K))
            w = (dict(qkv=q(H + 2 * kv, H), o=q(H, H), gu=q(2 * I, H), down=q(H, I)) if c["fused"] else
                 dict(q=q(H, H), k=q(kv, H), v=q(kv, H), o=q(H, H), gate=q(I, H), up=q(I, H), down=q(H, I)))
            layers.append(dict(w=w, x1=_activations(g, M, H), attn=_activations(g, M, H), x2=_activations(g, M, H),
                               g1=_gamma(g, H), g2=_gamma(g, H)))
        state = dict(case=c, layers=layers)
        if c["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _layers(state)
            torch.cuda.current_stream().wait_stream(side)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                state["out"] = _layers(state)
            state["graph"] = graph
        return state
    if c["kind"] == "linear":
        M, N, K = c["tokens"], c["out"], c["inp"]
        return dict(case=c, x=_activations(g, M, K), w=_weights(g, N, K), dy=_grads(g, M, N))
    if c["kind"] == "mlp":
        M, H, I = c["tokens"], c["hidden"], c["inter"]
        return dict(case=c, x=_activations(g, M, H), dy=_grads(g, M, H),
                    w=mlp_block.MlpWeights(_weights(g, 2 * I, H), _weights(g, H, I)))
    shapes = [(n, *shard_shape(n, N, K, c["tp"])) for n, N, K in _matrices(c)]
    return dict(case=c, store=WeightStore(_matrices(c), c["layers"], transposed=c["transposed"], tp=c["tp"]),
                masters=[{n: _weights(g, N, K) for n, N, K in shapes} for _ in range(c["layers"])])


# -------------------------------------------------------------------- runs --

def _layers(state):
    fused, out = state["case"]["fused"], []
    for L in state["layers"]:
        w = L["w"]
        n = jet.rmsnorm_quant(L["x1"], L["g1"], EPS)
        for name in (("qkv",) if fused else ("q", "k", "v")):
            out.append(jet.fp8_linear_fwd(n["q_row"], n["s_row"], *w[name]))
        a = jet.quant_act(L["attn"])
        out.append(jet.fp8_linear_fwd(a["q_row"], a["s_row"], *w["o"]))
        n = jet.rmsnorm_quant(L["x2"], L["g2"], EPS)
        if fused:
            gu = jet.fp8_linear_fwd(n["q_row"], n["s_row"], *w["gu"])
            I = gu.shape[1] // 2
            h = jet.silu_mul_quant(gu[:, :I], gu[:, I:])
            out.append(gu)
        else:
            gate = jet.fp8_linear_fwd(n["q_row"], n["s_row"], *w["gate"])
            up = jet.fp8_linear_fwd(n["q_row"], n["s_row"], *w["up"])
            h = jet.silu_mul_quant(gate, up)
            out += [gate, up]
        out.append(jet.fp8_linear_fwd(h["q_row"], h["s_row"], *w["down"]))
    return out


def run(state):
    kind = state["case"]["kind"]
    if kind == "layer":
        if "graph" not in state:
            return _layers(state)
        state["graph"].replay()
        return state["out"]
    if kind == "linear":
        qw, sw, qwT, swT = jet.quant_weight(state["w"], transposed=True)
        qx = jet.quant_act(state["x"])
        y = jet.fp8_linear_fwd(qx["q_row"], qx["s_row"], qw, sw)
        qdy = jet.quant_act(state["dy"], row=True, col=True)
        dx = jet.fp8_linear_dgrad(qdy["q_row"], qdy["s_row"], qwT, swT)
        qxT = jet.quant_act(qx["q_row"], qx["s_row"], row=False, col=True)
        dw = jet.fp8_linear_wgrad(qdy["q_colT"], qdy["s_colT"], qxT["q_colT"], qxT["s_colT"])
        return dict(y=y, dx=dx, dw=dw, qw=qw, sw=sw, qwT=qwT, swT=swT)
    if kind == "mlp":
        y, saved = mlp_block.forward(state["x"], state["w"])
        b = mlp_block.backward(saved, state["dy"], state["w"])
        return dict(y=y, dx=b["dx"], dw_gu=b["dw_gu"], dw_d=b["dw_d"])
    state["store"].sync(state["masters"])
    return state["store"].layers


# ------------------------------------------------------------- what it takes --

def work(case):
    c = case
    fp8 = lambda N, K: N * K + 4 * (N // 128) * (K // 128)
    if c["kind"] == "layer":
        H, kv, I, M = c["hidden"], c["kv"], c["inter"], c["batch"]
        weights = sum(fp8(N, K) for _, N, K in _matrices(c))
        rows = 3 * H + (H + 2 * kv) + H + 2 * I + H        # x1, attn, x2 in; q/k/v, o, gate/up, down out
        return {"bytes": c["layers"] * (weights + 2 * M * rows + 4 * H),
                "flops": c["layers"] * 2.0 * M * sum(N * K for _, N, K in _matrices(c))}
    if c["kind"] == "linear":
        M, N, K = c["tokens"], c["out"], c["inp"]
        return {"bytes": 2 * (N * K + M * K + M * N) + 2 * (M * N + M * K + N * K) + 2 * fp8(N, K),
                "flops": 6.0 * M * N * K}
    if c["kind"] == "mlp":
        M, H, I = c["tokens"], c["hidden"], c["inter"]
        return {"bytes": 2 * (fp8(2 * I, H) + fp8(H, I)) + 2 * M * 4 * H + 2 * 3 * H * I, "flops": 18.0 * M * H * I}
    total = 0
    for n, N, K in _matrices(c):
        n_, k_ = shard_shape(n, N, K, c["tp"])
        total += 2 * n_ * k_ + (2 if c["transposed"] else 1) * fp8(n_, k_)
    return {"bytes": c["layers"] * total, "flops": 0.0}


def tolerance(case):
    """Four times what the path differs by from itself with its GEMMs in binary64: codes and scales have
    one right value; a bf16 output of one GEMM differs in 1-3 % of its roundings (rel 4e-4, max 8e-3);
    behind a second GEMM the codes of its bf16 input flip with them (rel 3.4e-3, max 0.044), and small
    gradients of a whole block cancel (rel 4.1e-3, max 0.53)."""
    if case["kind"] == "sync":
        return "exact"
    if case["kind"] == "linear":
        return {"rel": 1.7e-3, "max": 0.032, "differ": 0.0}
    return {"rel": 1.6e-2, "max": 0.18 if case["kind"] == "layer" else 0.99, "differ": 0.0}
