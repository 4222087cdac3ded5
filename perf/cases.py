"""The work that a program has this framework do, as cases that can be timed: one linear call, the projections of decoder
blocks (decode steps and prefill chunks), the feed-forward block of a mixture-of-experts model, and the conversion of a
block's weights when a model is loaded.

A case is a dict of plain values.  `prepare` makes what a program keeps (weights in the kernel layout, workspaces, output
tensors, for decode steps the captured graph) and the inputs of one pass; `run` is one pass through the public entry
points.  Activations are N(0,1) with 1 % of the channels twenty times larger, weights N(0, 0.02), group size 128,
normalised scales, amplifier 2^10: what the benchmark and the tests of this repository use.

Kinds of case
  linear  one linear call on fp16 token rows: m x k times n x k.
  block   the projections of `layers` decoder blocks on m token rows, as a block calls them: RMSNorm folded into the
          quantiser, qkv GEMM on the codes; o_proj as a linear call on fp16 (the attention itself is not this
          framework's); RMSNorm folded into the quantiser, gate_up GEMM, SiLU * up folded into the quantiser (or, "fused",
          the gate_up GEMM with SiLU * up as its epilogue and the quantiser behind it), down GEMM.  "down_bits" 8 is the
          recipe with fine-grained W8A8 down projections.  "scales" float is the float-scale form of the same layer.
          "graph": a decode step as a serving loop keeps it, captured once and replayed.
  moe     the feed-forward block of a mixture of experts: token rows sorted by expert, quantised, grouped GEMM on the
          stacked w1 | w3, SiLU * up folded into the quantiser, grouped GEMM on w2.
  load    a checkpoint's fp16 projections to int4 codes and integer scales, and on to the kernel layout.
"""
import math

import torch

import paper_2405_14597_amd as P

GROUP = 128
ALPHA_LOG2 = 10
EPS = 1e-5


def listed():
    def block(name, m, hidden, qkv, inter, layers=1, graph=False, fused=False, down_bits=4, scales="int"):
        return {"name": name, "kind": "block", "m": m, "hidden": hidden, "qkv": qkv, "inter": inter, "layers": layers,
                "graph": graph, "fused": fused, "down_bits": down_bits, "scales": scales}
    return [
        # the smallest call: one token through one square projection, not captured, so the launch path counts
        {"name": "linear_m1", "kind": "linear", "m": 1, "k": 4096, "n": 4096, "scales": "int"},
        # an odd number of rows and a ragged output width (a vocabulary or adapter slice), between decode and prefill
        {"name": "linear_ragged", "kind": "linear", "m": 93, "k": 4224, "n": 5003, "scales": "int"},
        # decode steps of a 7B model at batch 1, 16 and 64: two blocks, so that the weights come from memory and not from
        # cache (three times 214 MB against a cache of 256 MB)
        block("decode_7b_m1", 1, 4096, 12288, 11008, layers=2, graph=True),
        block("decode_7b_m16", 16, 4096, 12288, 11008, layers=2, graph=True),
        block("decode_7b_m64", 64, 4096, 12288, 11008, layers=2, graph=True),
        # a decode step of one 70B block at batch 32
        block("decode_70b_m32", 32, 8192, 10240, 28672, graph=True),
        # a chunk of a prompt, as a chunked-prefill scheduler feeds it: an odd row count, the recipe with W8A8 down
        block("chunk_8b_m300", 300, 4096, 6144, 14336, down_bits=8),
        # whole prompts: 70B at 2048 tokens, 8B at 4096 tokens with the fused gate_up epilogue
        block("prefill_70b_m2048", 2048, 8192, 10240, 28672),
        block("prefill_8b_m4096", 4096, 4096, 6144, 14336, fused=True),
        # a mixture of eight experts, top-2: 512 tokens of a prompt, and a decode step of 16 tokens
        {"name": "moe_t512", "kind": "moe", "tokens": 512, "experts": 8, "topk": 2, "hidden": 4096, "inter": 14336, "graph": False},
        {"name": "moe_t16", "kind": "moe", "tokens": 16, "experts": 8, "topk": 2, "hidden": 4096, "inter": 14336, "graph": True},
        # loading one block of an 8B model
        {"name": "load_8b", "kind": "load", "hidden": 4096, "qkv": 6144, "inter": 14336, "down_bits": 4},
    ]


def draw(rng):
    """One more case of the same ranges.  Sizes that a layer has are multiples of 128 along K (the kernels' contract);
    row counts and the output widths of a plain linear are any whole numbers."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(("linear", "block", "moe", "load"), (0.3, 0.45, 0.17, 0.08))[0]
    if kind == "linear":
        return {"kind": kind, "m": log_int(1, 4096), "k": 128 * log_int(8, 112), "n": log_int(1000, 28672),
                "scales": rng.choice(("int", "int", "int", "float"))}
    if kind == "block":
        hidden = 128 * rng.randint(16, 64)
        inter = 128 * int(round(hidden * rng.uniform(2.5, 3.5) / 128))
        qkv = hidden + 2 * 128 * rng.choice((4, 8, hidden // 256, hidden // 128))
        decode = rng.random() < 0.6
        m = log_int(1, 64) if decode else log_int(65, 2048)
        return {"kind": kind, "m": m, "hidden": hidden, "qkv": qkv, "inter": inter,
                "layers": 1 if not decode else max(1, min(4, round(2 * 4096 ** 2 / hidden ** 2))), "graph": decode,
                "fused": rng.random() < 0.3, "down_bits": rng.choice((4, 4, 4, 8)),
                "scales": rng.choice(("int", "int", "int", "float"))}
    if kind == "moe":
        decode = rng.random() < 0.5
        return {"kind": kind, "tokens": log_int(1, 64) if decode else log_int(65, 1024), "experts": rng.choice((4, 8, 16)),
                "topk": rng.choice((1, 2, 2, 3)), "hidden": 128 * rng.randint(16, 32), "inter": 128 * rng.randint(24, 112),
                "graph": decode}
    return {"kind": kind, "hidden": 128 * rng.randint(16, 48), "qkv": 128 * rng.randint(16, 96), "inter": 128 * rng.randint(32, 128),
            "down_bits": rng.choice((4, 4, 8))}


# ---- inputs and what a program keeps
class _Maker:
    def __init__(self, seed):
        self.dev = torch.device("cuda:0")
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(seed)

    def activations(self, m, k):
        x = torch.randn((m, k), generator=self.gen, device=self.dev)
        x[:, torch.randperm(k, generator=self.gen, device=self.dev)[: k // 100]] *= 20.0
        return x.half()

    def weights(self, n, k):
        return torch.randn((n, k), generator=self.gen, device=self.dev, dtype=torch.float16).mul_(0.02)

    def gamma(self, k):
        return torch.rand((k,), generator=self.gen, device=self.dev).add_(0.5).half()

    def zeros(self, nbytes):
        return torch.zeros((max(nbytes, 256),), dtype=torch.uint8, device=self.dev)

    def half(self, *shape):
        return torch.zeros(shape, dtype=torch.float16, device=self.dev)

    def int8(self, *shape):
        return torch.zeros(shape, dtype=torch.int8, device=self.dev)

    def float(self, *shape):
        return torch.zeros(shape, dtype=torch.float32, device=self.dev)


def _quantised(mk, n, k):
    return P.is_quantize_weights_int4_group(mk.weights(n, k), GROUP, ALPHA_LOG2, P.IS_SCALE_NORM)


def _projection(mk, n, k, scales):
    q = _quantised(mk, n, k)
    if scales == "float":
        return P.is_prepack_w4(q.qweight, q.scale_f32, GROUP), None
    return P.is_prepack_w4(q.qweight, q.scale_i32, GROUP), q.chan_scale


def _linear(x, proj, out, ws):
    packed, chan = proj
    if packed.float_scales:
        P.is_linear_w4a8_floatscale_prepacked(x, packed, out=out, workspace=ws)
    else:
        P.is_linear_w4a8_intscale_prepacked(x, packed, chan, ALPHA_LOG2, out=out, workspace=ws)


def _gemm(xq, sa, proj, out, ws):
    packed, chan = proj
    if packed.float_scales:
        P.is_gemm_w4a8_floatscale_prepacked(xq, sa, packed, out=out, workspace=ws)
    else:
        P.is_gemm_w4a8_intscale_prepacked(xq, sa, packed, chan, ALPHA_LOG2, out=out, workspace=ws)


def _prepare_linear(c, mk):
    m, n, k = c["m"], c["n"], c["k"]
    return {"x": mk.activations(m, k), "proj": _projection(mk, n, k, c["scales"]), "out": mk.half(m, n),
            "ws": mk.zeros(P.is_linear_prepacked_workspace_bytes(m, n, k, GROUP))}


def _run_linear(s):
    _linear(s["x"], s["proj"], s["out"], s["ws"])
    return s["out"]


def _prepare_block(c, mk):
    m, h, qkv, inter = c["m"], c["hidden"], c["qkv"], c["inter"]
    layers = []
    for _ in range(c["layers"]):
        one = {"x1": mk.activations(m, h), "x2": mk.activations(m, h), "attn": mk.activations(m, h),
               "g1": mk.gamma(h), "g2": mk.gamma(h),
               "qkv": _projection(mk, qkv, h, c["scales"]), "o": _projection(mk, h, h, c["scales"])}
        if c["fused"]:
            q = _quantised(mk, 2 * inter, h)
            one["gate_up"] = P.is_prepack_w4_gate_up(q.qweight, q.scale_f32 if c["scales"] == "float" else q.scale_i32,
                                                     None if c["scales"] == "float" else q.chan_scale, GROUP)
        else:
            one["gate_up"] = _projection(mk, 2 * inter, h, c["scales"])
        if c["down_bits"] == 8:
            one["down"] = P.is_quantize_weights_int8_group(mk.weights(h, inter), GROUP, ALPHA_LOG2, P.IS_SCALE_NORM)
        else:
            one["down"] = _projection(mk, h, inter, c["scales"])
        one["out_qkv"], one["out_o"], one["out_down"] = mk.half(m, qkv), mk.half(m, h), mk.half(m, h)
        layers.append(one)
    down_ws = (P.is_gemm_w8a8_workspace_bytes if c["down_bits"] == 8 else P.is_gemm_prepacked_workspace_bytes)(m, h, inter, GROUP)
    gu_ws = (P.is_gemm_gate_up_silu_prepacked_workspace_bytes(m, inter, h, GROUP) if c["fused"]
             else P.is_gemm_prepacked_workspace_bytes(m, 2 * inter, h, GROUP))
    return {"layers": layers, "fused": c["fused"], "xq": mk.int8(m, h), "sa": mk.float(m), "hq": mk.int8(m, inter),
            "hs": mk.float(m), "gu": mk.half(m, inter if c["fused"] else 2 * inter),
            "ws_qkv": mk.zeros(P.is_gemm_prepacked_workspace_bytes(m, qkv, h, GROUP)),
            "ws_o": mk.zeros(P.is_linear_prepacked_workspace_bytes(m, h, h, GROUP)),
            "ws_gu": mk.zeros(gu_ws), "ws_down": mk.zeros(down_ws)}


def _run_block(s):
    xq, sa, hq, hs, gu = s["xq"], s["sa"], s["hq"], s["hs"], s["gu"]
    for one in s["layers"]:
        P.is_rmsnorm_quantize_act_int8_token(one["x1"], one["g1"], EPS, xq=xq, a_scale=sa)
        _gemm(xq, sa, one["qkv"], one["out_qkv"], s["ws_qkv"])
        _linear(one["attn"], one["o"], one["out_o"], s["ws_o"])
        P.is_rmsnorm_quantize_act_int8_token(one["x2"], one["g2"], EPS, xq=xq, a_scale=sa)
        if s["fused"]:
            if one["gate_up"].packed.float_scales:
                P.is_gemm_w4a8_floatscale_gate_up_silu_prepacked(xq, sa, one["gate_up"], out=gu, workspace=s["ws_gu"])
            else:
                P.is_gemm_w4a8_intscale_gate_up_silu_prepacked(xq, sa, one["gate_up"], ALPHA_LOG2, out=gu, workspace=s["ws_gu"])
            P.is_quantize_act_int8_token(gu, xq=hq, a_scale=hs)
        else:
            _gemm(xq, sa, one["gate_up"], gu, s["ws_gu"])
            P.is_silu_mul_quantize_act_int8_token(gu, xq=hq, a_scale=hs)
        down = one["down"]
        if isinstance(down, P.QuantizedWeights):
            P.is_gemm_w8a8_intscale(hq, hs, down.qweight, down.scale_i32, down.chan_scale, GROUP, ALPHA_LOG2,
                                    out=one["out_down"], workspace=s["ws_down"])
        else:
            _gemm(hq, hs, down, one["out_down"], s["ws_down"])
    return [[one["out_qkv"], one["out_o"], one["out_down"]] for one in s["layers"]]


def _experts(mk, e, n, k):
    q = [_quantised(mk, n, k) for _ in range(e)]
    packed = P.is_prepack_w4_experts(torch.stack([x.qweight for x in q]), torch.stack([x.scale_i32 for x in q]), GROUP)
    return packed, torch.stack([x.chan_scale for x in q])


def _prepare_moe(c, mk):
    t, e, h, inter = c["tokens"], c["experts"], c["hidden"], c["inter"]
    k = min(c["topk"], e)
    # uniform router: k distinct experts per token, the rows sorted by expert
    choice = torch.rand((t, e), generator=mk.gen, device=mk.dev).argsort(dim=1)[:, :k].reshape(-1)
    order = choice.argsort(stable=True)
    rows = mk.activations(t, h)[order // k].contiguous()
    offsets = torch.zeros((e + 1,), dtype=torch.int32, device=mk.dev)
    offsets[1:] = torch.bincount(choice, minlength=e).cumsum(0)
    m = t * k
    return {"rows": rows, "offsets": offsets, "w13": _experts(mk, e, 2 * inter, h), "w2": _experts(mk, e, h, inter),
            "xq": mk.int8(m, h), "sa": mk.float(m), "gu": mk.half(m, 2 * inter), "hq": mk.int8(m, inter), "hs": mk.float(m),
            "out": mk.half(m, h),
            "ws13": mk.zeros(P.is_gemm_grouped_prepacked_workspace_bytes(e, m, 2 * inter, h, GROUP)),
            "ws2": mk.zeros(P.is_gemm_grouped_prepacked_workspace_bytes(e, m, h, inter, GROUP))}


def _run_moe(s):
    P.is_quantize_act_int8_token(s["rows"], xq=s["xq"], a_scale=s["sa"])
    P.is_gemm_w4a8_intscale_grouped_prepacked(s["xq"], s["sa"], s["w13"][0], s["w13"][1], s["offsets"], ALPHA_LOG2,
                                              out=s["gu"], workspace=s["ws13"])
    P.is_silu_mul_quantize_act_int8_token(s["gu"], xq=s["hq"], a_scale=s["hs"])
    P.is_gemm_w4a8_intscale_grouped_prepacked(s["hq"], s["hs"], s["w2"][0], s["w2"][1], s["offsets"], ALPHA_LOG2,
                                              out=s["out"], workspace=s["ws2"])
    return s["out"]


def _load_shapes(c):
    h, qkv, inter = c["hidden"], c["qkv"], c["inter"]
    return {"qkv": (qkv, h), "o": (h, h), "gate_up": (2 * inter, h), "down": (h, inter)}


def _prepare_load(c, mk):
    return {"w": {name: mk.weights(*shape) for name, shape in _load_shapes(c).items()}, "down_bits": c["down_bits"]}


def _run_load(s):
    got = {}
    for name, w in s["w"].items():
        if name == "down" and s["down_bits"] == 8:
            q = P.is_quantize_weights_int8_group(w, GROUP, ALPHA_LOG2, P.IS_SCALE_NORM)
            got[name] = [q.qweight, q.scale_f32, q.scale_i32, q.chan_scale]
        else:
            q = P.is_quantize_weights_int4_group(w, GROUP, ALPHA_LOG2, P.IS_SCALE_NORM)
            packed = P.is_prepack_w4(q.qweight, q.scale_i32, GROUP)
            # (of the scales' 256-byte header the first 16 bytes are defined)
            got[name] = [q.qweight, q.scale_f32, q.scale_i32, q.chan_scale, packed.wpack, packed.spack[:16], packed.spack[256:]]
    return got


_PREPARE = {"linear": _prepare_linear, "block": _prepare_block, "moe": _prepare_moe, "load": _prepare_load}
_RUN = {"linear": _run_linear, "block": _run_block, "moe": _run_moe, "load": _run_load}


def prepare(case, seed):
    state = _PREPARE[case["kind"]](case, _Maker(seed))
    state["pass"] = _RUN[case["kind"]]
    state["graph"] = None
    if case.get("graph"):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            state["pass"](state)  # once before the capture, as every program does
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            state["outputs"] = state["pass"](state)
        state["graph"] = graph
    return state


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return state["outputs"]
    return state["pass"](state)


# ---- what a pass cannot do without
def _w4_bytes(n, k):
    return n * k // 2 + 4 * n * (k // GROUP) + 4 * n


def _w8_bytes(n, k):
    return n * k + 4 * n * (k // GROUP) + 4 * n


def work(case):
    c = case
    if c["kind"] == "linear":
        m, n, k = c["m"], c["n"], c["k"]
        return {"bytes": _w4_bytes(n, k) + 2 * m * k + 2 * m * n, "flops": 2 * m * n * k}
    if c["kind"] == "block":
        m, h, qkv, inter = c["m"], c["hidden"], c["qkv"], c["inter"]
        weights = _w4_bytes(qkv, h) + _w4_bytes(h, h) + _w4_bytes(2 * inter, h)
        weights += _w8_bytes(h, inter) if c["down_bits"] == 8 else _w4_bytes(h, inter)
        acts = 2 * m * (3 * h) + 2 * m * (qkv + 2 * h)  # the three inputs, and the outputs of qkv, o_proj and down
        flops = 2 * m * h * (qkv + h + 3 * inter)
        return {"bytes": c["layers"] * (weights + acts), "flops": c["layers"] * flops}
    if c["kind"] == "moe":
        h, inter, e = c["hidden"], c["inter"], c["experts"]
        k = min(c["topk"], e)
        m = c["tokens"] * k
        hit = e * (1.0 - (1.0 - k / e) ** c["tokens"])  # experts that some token is sent to, on average
        weights = hit * (_w4_bytes(2 * inter, h) + _w4_bytes(h, inter))
        return {"bytes": weights + 4 * m * h, "flops": 2 * m * h * 3 * inter}
    total = 0
    for name, (n, k) in _load_shapes(c).items():
        if name == "down" and c["down_bits"] == 8:
            total += 2 * n * k + n * k + 8 * n * (k // GROUP) + 4 * n
        else:
            # fp16 in; codes, both kinds of scales and channel scales out; the kernel layout of codes and scales out
            total += 2 * n * k + (n * k // 2 + 8 * n * (k // GROUP) + 4 * n) + (n * k // 2 + 4 * n * (k // GROUP))
    return {"bytes": total, "flops": 0}


def tolerance(case):
    """Four times what a pass differs by from the same path in 64 bits (the fp16 tensors between the calls kept): one fp16
    rounding of every output, and a code that a tie turns over here and there, which the second GEMM of a block carries on."""
    if case["kind"] == "load":
        return "exact"
    if case["kind"] == "linear":
        return {"rel": 1e-3, "max": 5e-2}  # seen: 2.4e-4, 1.2e-2
    return {"rel": 3.3e-3, "max": 2e-1}  # seen: 8.3e-4, 5.2e-2
