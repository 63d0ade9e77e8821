"""Performance cases of the W4A4 / W1.58A4 linear layers.

The work that a program built on this package has it do: the linears of the
DiT, FLUX-12B and 8B diffusion-LLM blocks it is made for, at image, text and
decoding-block token counts, on both engines, in every weight format, and the
packing of a layer's weights when a model is loaded.

A case's "kind" says which calls a pass makes:

  linear   one layer on a bf16 input: quantise, GEMM, epilogue;
  chain    several layers back to back, each on an input of its own (the MLP
           of a block: up, then down);
  block    the four linears of a diffusion-LLM block: its three inputs are
           quantised (gate and up share one), then four GEMMs;
  pack     a layer's bf16 weight to the operand the engine keeps.

"engine" is "f6" (6-bit matrix cores) or "int8"; "format" is "w4a4" (one scale
per token and output channel), "w158a4" (ternary weights), "g64" or "g128"
(group-wise scales).  Activations are heavy-tailed with a few outlier
channels, or GELU outputs for the inputs of down projections, as in
paper_2609_33601_amd/workloads.py, but drawn on the GPU.
"""

import math

import torch

from paper_2609_33601_amd import jq

DEV = "cuda"

# name, kind and shape of each case.  "shapes" is a text of M x K x N triples,
# a "b" behind a triple giving the layer a bias and a "g" a GELU input.
LISTED = [
    # the smallest layer of the repository's tests and of smoke(): a call that is all latency
    dict(name="tiny_64x256", kind="linear", engine="f6", format="w4a4", shapes="64x256x256b"),
    # one block of 64 tokens through an 8B diffusion LLM: the decoding step of block diffusion
    dict(name="dllm_block_64", kind="block", engine="f6", format="w4a4", shapes="64x4096x12288"),
    # a short, odd number of tokens with the paper's group128 quantisation, as its ELF/dLLM runs use it
    dict(name="dllm_mlp_g128_33", kind="chain", engine="f6", format="g128", shapes="33x4096x12288,33x12288x4096g"),
    # FLUX's text stream (512 tokens) through its MLP
    dict(name="flux_text_mlp", kind="chain", engine="f6", format="w4a4", shapes="512x3072x12288b,512x12288x3072g"),
    # few tokens on the packed-int4 engine, which keeps 4 bits a weight
    dict(name="int8_few_tokens", kind="linear", engine="int8", format="w4a4", shapes="77x4096x12288"),
    # FLUX-12B MLP, the headline: up for one image, down for two
    dict(name="flux_mlp", kind="chain", engine="f6", format="w4a4", shapes="4608x3072x12288b,9216x12288x3072g"),
    # a prefill or full-sequence denoising step of the 8B diffusion LLM
    dict(name="dllm_block_4096", kind="block", engine="f6", format="w4a4", shapes="4096x4096x12288"),
    # fused QKV of an image whose side is no multiple of anything, odd token count
    dict(name="qkv_ragged", kind="linear", engine="f6", format="w4a4", shapes="2747x3072x9216b"),
    # the DiT fused QKV on the packed-int4 engine
    dict(name="int8_qkv", kind="linear", engine="int8", format="w4a4", shapes="4608x3072x9216b"),
    # ternary weights in their 2-bit form, MLP-down of one image
    dict(name="ternary_down", kind="linear", engine="int8", format="w158a4", shapes="4608x12288x3072g"),
    # FLUX-12B MLP with the paper's group64 quantisation
    dict(name="flux_mlp_g64", kind="chain", engine="f6", format="g64", shapes="4608x3072x12288b,4608x12288x3072g"),
    # loading a model: a gate projection's weight, packed and re-encoded for the 6-bit engine
    dict(name="pack_gate", kind="pack", engine="f6", format="w4a4", shapes="1x4096x12288"),
]

# Time of an operation on each path relative to the 6-bit engine's per-token
# layer, used only to keep the drawn cases below the largest listed one.
COST = {("f6", "w4a4"): 1.0, ("f6", "w158a4"): 1.0, ("f6", "g64"): 3.2, ("f6", "g128"): 2.4,
        ("int8", "w4a4"): 1.6, ("int8", "w158a4"): 1.7, ("int8", "g64"): 4.6, ("int8", "g128"): 3.6}


def _layers(case):
    """(M, K, N, has bias, GELU input) of each layer that a pass runs."""
    out = []
    for t in case["shapes"].split(","):
        bias, gelu = "b" in t, "g" in t
        M, K, N = (int(v) for v in t.rstrip("bg").split("x"))
        out.append((M, K, N, bias, gelu))
    if case["kind"] == "block":
        M, D, F = out[0][:3]
        # gate, up, o, down
        out = [(M, D, F, False, False), (M, D, F, False, False), (M, D, D, False, False), (M, F, D, False, True)]
    return out


def listed():
    return [dict(c) for c in LISTED]


def draw(rng):
    """Another layer of the ranges: 1 to 9216 tokens, K and N from 256 to 12288, any engine and format; or a weight to pack."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    engine = rng.choice(["f6", "f6", "f6", "int8", "int8"])
    fmt = rng.choice(["w4a4", "w4a4", "w4a4", "w158a4", "g64", "g128"])
    kind = "pack" if rng.random() < 0.08 else "linear"
    step = 128 if fmt == "g128" else 64
    K = min(12288, max(256, log(256, 12288) // step * step))
    N = log(256, 12288)
    if rng.random() < 0.5:
        N = max(256, N // 64 * 64)  # hidden sizes of models mostly are multiples of 64
    M = 1 if kind == "pack" else log(1, 9216)
    M = max(1, min(M, int(8.0e11 / (2.0 * K * N * COST[engine, fmt]))))
    return dict(kind=kind, engine=engine, format=fmt,
                shapes="%dx%dx%d%s%s" % (M, K, N, rng.choice(["", "b"]), rng.choice(["", "g"])))


def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + k)
    return g


def _activations(M, K, gelu, g):
    x = torch.randn((M, K), generator=g, device=DEV)
    if gelu:
        x = torch.nn.functional.gelu(x)
    else:  # Student-t with 3 degrees of freedom, unit variance
        c = torch.zeros((M, K), device=DEV)
        for _ in range(3):
            c += torch.randn((M, K), generator=g, device=DEV).square_()
        x = x / c.sqrt_()
    cols = torch.randperm(K, generator=g, device=DEV)[: max(1, round(0.005 * K))]
    x[:, cols] *= 30.0
    return x.to(torch.bfloat16)


def _inputs(case, seed):
    """Per layer: input (None: the previous layer's), weight and bias in bf16."""
    out = []
    for i, (M, K, N, bias, gelu) in enumerate(_layers(case)):
        g = _gen(seed, i)
        x = None if case["kind"] == "pack" or (case["kind"] == "block" and i == 1) else _activations(M, K, gelu, g)
        w = (torch.randn((N, K), generator=g, device=DEV) * 0.02).to(torch.bfloat16)
        b = (torch.randn((N,), generator=g, device=DEV) * 0.01).to(torch.bfloat16) if bias else None
        out.append((x, w, b))
    return out


def _group(case):
    return {"g64": 64, "g128": 128}.get(case["format"], 0)


def _pack(case, w, out=(None, None, None)):
    """The weight operand of the case's engine and format, and its scales."""
    G = _group(case)
    packed, scale, wf6 = out
    if case["format"] == "w158a4":
        q, s = jq.jq_pack_weight_ternary(w, packed, scale)
    elif G:
        q, s = jq.jq_pack_weight_int4_group(w, G, packed, scale)
    else:
        q, s = jq.jq_pack_weight_int4(w, packed, scale)
    if case["engine"] == "f6":
        q2 = (jq.jq_ternary_to_f6_weight if case["format"] == "w158a4" else jq.jq_int4_to_f6_weight)(q, wf6)
        return q, s, q2
    return q, s, None


def prepare(case, seed):
    """Inputs, the packed weights, and the output and workspace that a serving program keeps for each layer."""
    layers, data, G = _layers(case), _inputs(case, seed), _group(case)
    if case["kind"] == "pack":
        w = data[0][1]
        return {"case": case, "w": w, "out": [None if t is None else torch.empty_like(t) for t in _pack(case, w)]}
    ls = []
    for (M, K, N, _, _), (x, w, b) in zip(layers, data):
        q, s, wf6 = _pack(case, w)
        if case["engine"] == "f6":
            ws = jq.jq_w4a4g_f6_workspace_bytes(M, K, G) if G else jq.jq_w4a4_f6_workspace_bytes(M, K)
            q = wf6
        else:
            ws = jq.jq_w4a4g_workspace_bytes(M, K, G) if G else jq.jq_w4a4_workspace_bytes(M, K)
        ls.append({"x": x, "w": q, "ws": s, "b": b, "K": K,
                   "y": torch.empty((M, N), dtype=torch.bfloat16, device=DEV),
                   "work": torch.empty((ws,), dtype=torch.uint8, device=DEV)})
    st = {"case": case, "layers": ls, "G": G}
    if case["kind"] == "block":
        st["xs"] = [ls[0]["x"], ls[2]["x"], ls[3]["x"]]
        st["q"] = [torch.empty((jq.jq_f6_operand_bytes(*x.shape),), dtype=torch.uint8, device=DEV) for x in st["xs"]]
        st["s"] = [torch.empty((x.shape[0],), dtype=torch.float32, device=DEV) for x in st["xs"]]
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "pack":
        return [t for t in _pack(case, state["w"], state["out"]) if t is not None]
    if case["kind"] == "block":
        jq.jq_quantize_act_f6_batch(state["xs"], state["q"], state["s"])
        for l, i in zip(state["layers"], (0, 0, 1, 2)):
            jq.jq_w4a4_f6_gemm(state["q"][i], state["s"][i], l["K"], l["w"], l["ws"], l["b"], l["y"])
        return [l["y"] for l in state["layers"]]
    G, f6, tern = state["G"], case["engine"] == "f6", case["format"] == "w158a4"
    for l in state["layers"]:
        if G:
            f = jq.jq_w4a4g_f6_linear if f6 else jq.jq_w4a4g_linear
            f(l["x"], l["w"], l["ws"], G, l["b"], l["y"], l["work"])
        else:
            f = jq.jq_w4a4_f6_linear if f6 else jq.jq_w158a4_linear if tern else jq.jq_w4a4_linear
            f(l["x"], l["w"], l["ws"], l["b"], l["y"], l["work"])
    return [l["y"] for l in state["layers"]]


def work(case):
    """Each input read once (weights at the 4 or 2 bits they carry) and each output written once; the products' operations."""
    nbytes = flops = 0.0
    G = _group(case)
    wb = 0.25 if case["format"] == "w158a4" else 0.5
    for i, (M, K, N, bias, _) in enumerate(_layers(case)):
        scales = 4.0 * N * (K / G if G else 1)
        if case["kind"] == "pack":
            f6 = jq.jq_f6_operand_bytes(N, K) if case["engine"] == "f6" else 0
            return {"bytes": 2.0 * N * K + wb * N * K + scales + f6, "flops": 2.0 * N * K}
        x = 0.0 if case["kind"] == "block" and i == 1 else 2.0 * M * K
        nbytes += x + wb * N * K + scales + 2.0 * M * N + (2.0 * N if bias else 0.0)
        flops += 2.0 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """The layer's every rounding is defined (codes, scales, exact integer products, the fp32 steps of the
    epilogue and of the group sum, each rounded on its own), so another correct implementation gives the same bits."""
    return "exact"


def _codes(x, G):
    """Codes and scales (fp64 tensors, a scale per row or per group spread over its columns)."""
    R, K = x.shape
    v = x.double().reshape(R, K // G if G else 1, -1)
    s = (v.abs().amax(2, keepdim=True) / 7.0).float().double()
    t = torch.where(s > 0, v / torch.where(s > 0, s, torch.ones_like(s)), torch.zeros_like(v)).float()
    return t.round().clamp_(-8, 7).double().reshape(R, K), s.expand_as(v).reshape(R, K), s.reshape(R, -1)


def _ternary(w):
    g = (w.double().abs().sum(1, keepdim=True) / w.shape[1]).float().double()
    t = torch.where(g > 0, w.double() / torch.where(g > 0, g, torch.ones_like(g)), torch.zeros_like(w.double()))
    return t.float().round().clamp_(-1, 1).double(), g.expand_as(w), g


def exact(case, seed):
    layers, data, G = _layers(case), _inputs(case, seed), _group(case)
    quant_w = _ternary if case["format"] == "w158a4" else (lambda w: _codes(w, G))
    if case["kind"] == "pack":
        _, _, s = quant_w(data[0][1])
        s = s if G else s.reshape(-1)
        return [None, s] + ([None] if case["engine"] == "f6" else [])  # packed bytes have no 64-bit value
    out, last = [], None
    for x, w, b in data:
        if x is None:
            x = last
        last = x
        qx, sx, _ = _codes(x, G)
        qw, sw, _ = quant_w(w)
        y = (qx * sx) @ (qw * sw).t().contiguous()
        out.append(y if b is None else y + b.double())
    return out
