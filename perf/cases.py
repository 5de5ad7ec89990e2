"""The work that a user of the quantized linear layer has it do: which passes are timed, their inputs, what they
cannot do without and how far a correct result may be off.

Four kinds of pass, all through the public calls of `paper_2206_01861_amd.binding`:

* ``block``   the linears of transformer blocks, in the order a block runs them: LayerNorm + quantization, QKV,
  quantization of the attention context, output projection, LayerNorm + quantization, first feed-forward linear,
  GeLU + quantization, second feed-forward linear.  Attention and the residual additions are not part of the framework,
  so each block's hidden state and attention context are inputs.  ``a16`` keeps the QKV input in FP16 (W8A16),
  ``ffn_bits`` 4 holds the feed-forward weights as packed INT4.
* ``ffn``     the feed-forward pair alone; ``fused`` takes GeLU and the quantizer into the first linear.
* ``linear``  one linear behind its LayerNorm; ``requant`` also wants its output quantized for the linear that follows.
* ``weights`` the group-wise quantization of a block's weights, which is done when a model is loaded.

Up to 128 tokens a pass is launch-bound unless its launches are captured, so a serving program captures a decode step
in a HIP graph once and replays it; larger passes are issued call by call.  Decode passes run over enough blocks that
their weights exceed the 256 MB cache, as in a model, where every step reads all weights from memory.
"""
import math

import torch

from paper_2206_01861_amd import binding as zq

GRAPH_TOKENS = 128          # a pass of up to this many tokens is captured and replayed
DECODE_BYTES = 300e6        # weights that a decode pass reads, at least (up to MAX_LAYERS blocks)
MAX_LAYERS = 8
EPS = 1e-5


def _case(kind, hidden, ffn, tokens, layers=1, ffn_bits=8, a16=False, fused=False, requant=False, tanh=True, name=None):
    c = {"kind": kind, "hidden": hidden, "ffn": ffn, "tokens": tokens, "layers": layers, "ffn_bits": ffn_bits,
         "a16": a16, "fused": fused, "requant": requant, "tanh": tanh}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a BERT-base sized linear for one sentence: the smallest call, launches and latency
        _case("linear", 768, 768, 128, tanh=False, name="linear_768_128"),
        # the feed-forward pair of a BERT-large sized model, batch 32 x 128 tokens: the benchmark's workload
        _case("ffn", 1024, 4096, 4096, tanh=False, name="ffn_1024_4096"),
        # the same pair for a batch without padding (any token count), GeLU and quantizer inside the first linear
        _case("ffn", 1024, 4096, 1237, fused=True, tanh=False, name="ffn_fused_1024_1237"),
        # generation with a 1.3B sized model: one request, and a batch of requests
        _case("block", 2048, 8192, 1, layers=6, name="decode_2048_1"),
        _case("block", 2048, 8192, 27, layers=6, name="decode_2048_27"),
        # prompt of the same model
        _case("block", 2048, 8192, 2048, name="prefill_2048_2048"),
        # generation with a 6B sized model whose feed-forward weights are INT4, batch 16
        _case("block", 4096, 16384, 16, layers=2, ffn_bits=4, name="decode_w4_4096_16"),
        # the same model, a step that mixes requests in generation with a piece of a prompt
        _case("block", 4096, 16384, 333, ffn_bits=4, name="mixed_w4_4096_333"),
        # generation with a 20B sized model whose QKV input stays FP16, batch 64, and a batch of prompts
        _case("block", 6144, 24576, 64, a16=True, name="decode_a16_6144_64"),
        _case("block", 6144, 24576, 16384, a16=True, name="prefill_a16_6144_16384"),
        # a width that is no multiple of 256, a small batch
        _case("block", 1600, 6400, 5, layers=8, name="decode_1600_5"),
        # loading the 6B sized model: one block's weights, INT8 attention and INT4 feed-forward
        _case("weights", 4096, 16384, 1, ffn_bits=4, name="weights_w4_4096"),
    ]


def draw(rng):
    kind = rng.choices(["block", "ffn", "linear", "weights"], [12, 4, 2, 2])[0]
    step = rng.choice([32, 64, 128, 128, 256, 256])
    hidden = max(768, round(math.exp(rng.uniform(math.log(768), math.log(6144))) / step) * step)
    ffn = hidden * 4 if rng.random() < 0.75 else round(hidden * rng.uniform(2.5, 3.8) / step) * step
    tokens = max(1, round(math.exp(rng.uniform(0, math.log(16384)))))
    if tokens > 8 and rng.random() < 0.4:
        tokens = tokens // 8 * 8
    layers = 1
    if kind == "block" and tokens <= GRAPH_TOKENS:
        layers = max(1, min(MAX_LAYERS, math.ceil(DECODE_BYTES / (4 * hidden * hidden + 2 * hidden * ffn))))
    fused = kind == "ffn" and rng.random() < 0.5
    requant = kind == "linear" and rng.random() < 0.5
    a16 = kind == "block" and rng.random() < 0.25
    return _case(kind, hidden, ffn, tokens, layers, ffn_bits=rng.choice([8, 8, 4]), a16=a16, fused=fused,
                 requant=requant, tanh=rng.random() < 0.5)


def _linears(case):
    """(name, output width, input width, bits) of the linears of one block of the case."""
    h, f, b = case["hidden"], case["ffn"], case["ffn_bits"]
    if case["kind"] == "linear":
        return [("fc", h, h, 8)]
    ffn = [("fc1", f, h, b), ("fc2", h, f, b)]
    if case["kind"] == "ffn":
        return ffn
    return [("qkv", 3 * h, h, 8), ("proj", h, h, 8)] + ffn


def _groups(n):
    """Weight groups of a linear: at most 128, each a multiple of 16 rows."""
    return max(g for g in range(1, 129) if (n // 16) % g == 0)


# ---- inputs: the structure of zq_inputs.py (token ranges that differ several-fold, a few outlier channels, weight
# ---- rows whose magnitudes differ by a factor of ten), drawn on the GPU

def _weight(gen, n, k):
    w = torch.randn((n, k), generator=gen, device="cuda", dtype=torch.float16) * 0.02
    rows = torch.rand((n, 1), generator=gen, device="cuda") * math.log(10.0) + math.log(0.3)
    return w.mul_(rows.exp().half())


def _hidden_state(gen, m, k):
    x = torch.randn((m, k), generator=gen, device="cuda")
    x *= (torch.rand((m, 1), generator=gen, device="cuda") * math.log(4.0) + math.log(0.5)).exp()
    x[:, torch.randperm(k, generator=gen, device="cuda")[: max(1, k // 200)]] *= 8.0
    return x.half()


def _vector(gen, n, mean, std):
    return (mean + std * torch.randn(n, generator=gen, device="cuda")).half()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    h, m = case["hidden"], case["tokens"]
    s = {"case": case}
    if case["kind"] == "weights":
        s["weights"] = [(_weight(gen, n, k), _groups(n), bits) for _, n, k, bits in _linears(case)]
        return s
    s["layers"], need = [], 0
    for _ in range(case["layers"]):
        layer = {}
        for name, n, k, bits in _linears(case):
            wq, sw = zq.zq_quantize_weight_groupwise(_weight(gen, n, k), _groups(n), bits)
            layer[name] = (wq, sw, _vector(gen, n, 0.0, 0.01))
            need = max(need, zq.gemm_quant_workspace_bytes(m, n, k, bits))
            if name == "qkv" and case["a16"]:
                need = max(need, zq.gemm_w8a16_workspace_bytes(m, n, k))
        for norm in ("ln1", "ln2"):
            layer[norm] = (_vector(gen, h, 1.0, 0.1), _vector(gen, h, 0.0, 0.1))
        layer["x"] = _hidden_state(gen, m, h)
        if case["kind"] == "block":
            layer["context"] = _hidden_state(gen, m, h)
        s["layers"].append(layer)
    s["ws"] = zq.new_workspace(need)
    if m <= GRAPH_TOKENS and case["kind"] == "block":
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _forward(s)                                  # loads the kernels before the capture
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            s["out"] = _forward(s)
    return s


def _gemm(xq, s_tok, weight, ws, requant=False):
    wq, sw, bias = weight
    call = zq.zq_gemm_i8_dequant if wq.dtype == torch.int8 else zq.zq_gemm_w4a8_dequant
    return call(xq, s_tok, wq, sw, bias, requant=requant, workspace=ws)


def _ffn(s, layer, x):
    case, ws = s["case"], s["ws"]
    xq, st, _ = zq.zq_layernorm_quant_tokenwise(x, *layer["ln2"], EPS)
    wq, sw, bias = layer["fc1"]
    if case["fused"]:
        inside = zq.gemm_quantizes_in_kernel(x.shape[0], wq.shape[0], x.shape[1], case["ffn_bits"], ws.numel())
        _, gq, gs = zq.zq_gemm_gelu_quant_tokenwise(xq, st, wq, sw, bias, approx_tanh=case["tanh"], workspace=ws,
                                                    keep_g=not inside)
    else:
        f = _gemm(xq, st, layer["fc1"], ws)[0]
        gq, gs, _ = zq.zq_gelu_quant_tokenwise(f, None, approx_tanh=case["tanh"])
    return _gemm(gq, gs, layer["fc2"], ws)[0]


def _forward(s):
    case, ws, out = s["case"], s["ws"], []
    if case["kind"] == "linear":
        layer = s["layers"][0]
        x = layer["x"]
        xq, st, _ = zq.zq_layernorm_quant_tokenwise(x, *layer["ln1"], EPS)
        y, _, yq, ys = _gemm(xq, st, layer["fc"], ws, requant=case["requant"])
        return [y, yq, ys] if case["requant"] else [y]
    for layer in s["layers"]:
        x = layer["x"]
        if case["kind"] == "block":
            if case["a16"]:
                _, _, xn = zq.zq_layernorm_quant_tokenwise(x, *layer["ln1"], EPS, y_dtype=torch.float16)
                out.append(zq.zq_gemm_w8a16_dequant(xn, *layer["qkv"], workspace=ws))
            else:
                xq, st, _ = zq.zq_layernorm_quant_tokenwise(x, *layer["ln1"], EPS)
                out.append(_gemm(xq, st, layer["qkv"], ws)[0])
            cq, cs = zq.zq_quantize_tokenwise(layer["context"])
            x = _gemm(cq, cs, layer["proj"], ws)[0]
            out.append(x)
        out.append(_ffn(s, layer, x))
    return out


def run(state):
    if "weights" in state:
        return [zq.zq_quantize_weight_groupwise(w, g, bits) for w, g, bits in state["weights"]]
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return _forward(state)


def work(case):
    """Weights and inputs read once, the pass's outputs written once, and the products of the linears."""
    m, h, linears = case["tokens"], case["hidden"], _linears(case)
    if case["kind"] == "weights":
        return {"bytes": sum(n * k * (2 + bits / 8) + 4 * _groups(n) for _, n, k, bits in linears), "flops": 0}
    weights = sum(n * k * bits / 8 + 4 * _groups(n) + 2 * n for _, n, k, bits in linears)
    norms = 4 * h * (2 if case["kind"] == "block" else 1)
    # FP16: the hidden state and the output; in a block also the context, QKV and the projection
    per_layer = 2 * m * h * (7 if case["kind"] == "block" else 2)
    if case["requant"]:
        per_layer += m * h + 4 * m
    flops = sum(2.0 * m * n * k for _, n, k, _ in linears)
    return {"bytes": case["layers"] * (weights + norms + per_layer), "flops": case["layers"] * flops}


def tolerance(case):
    """Weight codes, scales and nibbles are defined bit for bit.  Elsewhere a rounding of the LayerNorm, of GeLU or of
    an FP16 result that falls the other way moves single INT8 codes by one step, and a whole token's when it falls on
    the token's largest value.  Against the same pass in 64 bits: up to 5.5e-3 in a block (one value by up to 0.23 of the
    root mean square; few tokens show it most) and 3e-4 in a pair or a single linear (0.06)."""
    if case["kind"] == "weights":
        return "exact"
    t = {"rel": 2e-2, "max": 0.9} if case["kind"] == "block" else {"rel": 2e-3, "max": 0.25}
    if case["requant"]:
        t["differ"] = 0.01
    return t
