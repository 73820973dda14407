"""Performance cases of the W4A16 GEMM library: what a serving program has it do.

Each case is one pass through the Python entry points (``w4a16_gemm``,
``gemm_fused``, ``grouped_gemm``, ``grouped_gemm_fused``):

* ``linear``  one quantized linear layer;
* ``layer``   the four quantized linears of a Llama decoder layer in their
  order: QKV projection, output projection, gate+up projection, down
  projection.  With ``gated`` (decode batches of up to 32 rows, where the
  automatic choice always offers it) the gated SiLU is in the gate+up
  projection's epilogue and the down projection reads its result; otherwise
  the program applies the activation itself and the four GEMMs have inputs of
  their own;
* ``moe``     the expert feed-forward of a Mixtral layer: the grouped
  gate+up GEMM over the routed rows (gathered in the kernel, gated SiLU in the
  epilogue), then the grouped down GEMM on its result.

A case with ``graph`` replays a HIP graph of these calls, which is how a
decode loop runs them (the launches of one token are shorter than their host
cost); the others are plain calls.  The automatic kernel choice is used
throughout: no tune table is loaded.

Weights are drawn in packed form: every bit pattern is a valid packing, so
uniform random words are uniform random 4-bit weights and zero points.  Scales
are uniform in [0.002, 0.02], activations standard normal, both binary16.
"""
from __future__ import annotations

import math

import torch

import paper_2402_10076_amd as Q

# hidden size, QKV columns, feed-forward size
LLAMA_7B = {"d": 4096, "qkv": 12288, "f": 11008}
LLAMA_13B = {"d": 5120, "qkv": 15360, "f": 13824}
LLAMA_70B = {"d": 8192, "qkv": 10240, "f": 28672}
MIXTRAL = {"d": 4096, "f": 14336, "experts": 8}


def _layer(name, size, m, layers=1, graph=False, bias=False):
    return dict(size, name=name, kind="layer", m=m, layers=layers, graph=graph, bias=bias, gated=m <= 32)


def _moe(name, size, tokens, graph=False):
    return dict(size, name=name, kind="moe", tokens=tokens, graph=graph)


def listed():
    return [
        # the smallest call: one small linear, where the latency of the call counts
        {"name": "linear_512_m16", "kind": "linear", "k": 512, "n": 512, "m": 16, "graph": False},
        # one user's token through two decoder layers, as the decode graph replays it
        _layer("decode_7b_m1", LLAMA_7B, 1, layers=2, graph=True),
        # the same for a 70B model's layer, called without a graph
        _layer("decode_70b_m1", LLAMA_70B, 1),
        # a batch of 16 sequences decoding
        _layer("decode_13b_m16", LLAMA_13B, 16, layers=2, graph=True),
        # a batch of 64 sequences decoding
        _layer("decode_7b_m64", LLAMA_7B, 64, layers=2, graph=True),
        # a large batch of a large model, or a short prompt
        _layer("batch_70b_m128", LLAMA_70B, 128),
        # a prefill chunk
        _layer("prefill_7b_m256", LLAMA_7B, 256),
        # a prompt of no round length, with biases
        _layer("prefill_13b_m333_bias", LLAMA_13B, 333, bias=True),
        # prefill of a large model
        _layer("prefill_70b_m1024", LLAMA_70B, 1024),
        # a long prompt in one piece
        _layer("prefill_7b_m2048", LLAMA_7B, 2048),
        # mixture of experts: a decode batch (a few rows an expert) ...
        _moe("moe_decode_t20", MIXTRAL, 20, graph=True),
        # ... and a prefill chunk (about 128 rows an expert)
        _moe("moe_prefill_t512", MIXTRAL, 512),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step) * step))


def draw(rng):
    most = max(_flops(c) for c in listed())
    while True:
        kind = rng.choice(["linear", "layer", "layer", "layer", "moe"])
        if kind == "linear":
            c = {"kind": kind, "k": _log_int(rng, 512, 8192, 128), "n": _log_int(rng, 512, 28672, 16),
                 "m": _log_int(rng, 1, 2048), "graph": False}
        elif kind == "layer":
            d = _log_int(rng, 2048, 8192, 128)
            m = _log_int(rng, 1, 2048)
            c = {"kind": kind, "d": d, "qkv": _log_int(rng, d + 256, 3 * d, 16),
                 "f": _log_int(rng, 2 * d, 7 * d // 2, 128), "m": m, "layers": 1,
                 # decode batches run as graphs, prompts do not
                 "graph": m <= 64, "bias": rng.random() < 0.3, "gated": m <= 32}
        else:
            d = _log_int(rng, 2048, 4096, 128)
            tokens = _log_int(rng, 4, 1024)
            c = {"kind": kind, "d": d, "f": _log_int(rng, 2 * d, 7 * d // 2, 128),
                 "experts": rng.choice([4, 8, 16]), "tokens": tokens, "graph": tokens <= 64}
        if _flops(c) <= most:
            return c


def _gemms(case):
    """(rows, K, N, output columns, weight matrices read, rows of the input) of each GEMM of a pass."""
    if case["kind"] == "linear":
        return [(case["m"], case["k"], case["n"], case["n"], 1, case["m"])]
    if case["kind"] == "layer":
        m, d, f = case["m"], case["d"], case["f"]
        one = [(m, d, case["qkv"], case["qkv"], 1, m), (m, d, d, d, 1, m),
               (m, d, 2 * f, f if case["gated"] else 2 * f, 1, m), (m, f, d, d, 1, m)]
        return one * case["layers"]
    r, e = 2 * case["tokens"], min(case["experts"], 2 * case["tokens"])
    return [(r, case["d"], 2 * case["f"], case["f"], e, case["tokens"]), (r, case["f"], case["d"], case["d"], e, r)]


def _flops(case):
    return sum(2 * m * k * n for m, k, n, _, _, _ in _gemms(case))


def work(case):
    # packed weights 4 bits, scales 16 and zero points 4 bits per 128 channels of a column
    nbytes = sum(w * (k * n // 2 + k * n // 64 + k * n // 256) + 2 * rows * k + 2 * m * out
                 for m, k, n, out, w, rows in _gemms(case))
    return {"bytes": nbytes, "flops": _flops(case)}


def tolerance(case):
    # One rounding of each weight and one of each result to binary16 (2^-11
    # relative each), with sums in binary32.
    return {"rel": 1.5e-3, "max": 1e-2}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(g, k, n, matrices=1):
    wb, zb, sb = Q.packed_sizes(k, n)

    def words(nbytes):
        return torch.randint(-2 ** 31, 2 ** 31, (matrices * nbytes // 4,), generator=g, device="cuda",
                             dtype=torch.int32)

    packed = words(wb)
    zeros = words(zb)
    scales = torch.empty(matrices * sb // 2, device="cuda").uniform_(0.002, 0.02, generator=g)
    return packed, scales.to(torch.float16).view(torch.int16), zeros


def _normal(g, *shape, scale=1.0):
    return (torch.randn(*shape, generator=g, device="cuda") * scale).to(torch.float16)


def _inputs(case, seed):
    g = _gen(seed)
    if case["kind"] == "linear":
        return {"x": _normal(g, case["m"], case["k"]), "w": _weights(g, case["k"], case["n"])}
    if case["kind"] == "layer":
        m, d, f, qkv = case["m"], case["d"], case["f"], case["qkv"]
        out = []
        for _ in range(case["layers"]):
            out.append({
                "xq": _normal(g, m, d), "xo": _normal(g, m, d), "xm": _normal(g, m, d),
                "wq": _weights(g, d, qkv), "wo": _weights(g, d, d),
                "wgu": _weights(g, d, 2 * f), "wd": _weights(g, f, d),
                "xd": None if case["gated"] else _normal(g, m, f),
                "bq": _normal(g, qkv) if case["bias"] else None, "bo": _normal(g, d) if case["bias"] else None,
                "bgu": _normal(g, 2 * f, scale=0.5) if case["bias"] else None,
                "bd": _normal(g, d) if case["bias"] else None})
        return {"layers": out}
    d, f, e, tokens = case["d"], case["f"], case["experts"], case["tokens"]
    # each token goes to two different experts; rows sorted by expert
    expert = torch.rand(tokens, e, generator=g, device="cuda").topk(2, dim=1).indices.reshape(-1)
    order = torch.argsort(expert, stable=True)
    count = torch.bincount(expert, minlength=e)
    offsets = torch.zeros(e + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = count.cumsum(0).to(torch.int32)
    return {"x": _normal(g, tokens, d), "rows": (order // 2).to(torch.int32), "offsets": offsets,
            "w13": _weights(g, d, 2 * f, e), "w2": _weights(g, f, d, e)}


def _calls(case, s, out=None):
    """The pass: its outputs, in new tensors or in those of ``out``."""
    it = iter(out) if out is not None else None

    def y():
        return next(it) if it is not None else None

    if case["kind"] == "linear":
        return [Q.w4a16_gemm(s["x"], *s["w"], case["n"], y=y())]
    if case["kind"] == "layer":
        d, f, qkv = case["d"], case["f"], case["qkv"]
        got = []

        def linear(x, w, n, bias):
            if bias is None:
                got.append(Q.w4a16_gemm(x, *w, n, y=y()))
            else:
                got.append(Q.gemm_fused(x, *w, n, bias=bias, y=y()))

        for t in s["layers"]:
            linear(t["xq"], t["wq"], qkv, t["bq"])
            linear(t["xo"], t["wo"], d, t["bo"])
            if case["gated"]:
                got.append(Q.gemm_fused(t["xm"], *t["wgu"], 2 * f, bias=t["bgu"], activation=Q.ACT_SILU_GATE, y=y()))
            else:
                linear(t["xm"], t["wgu"], 2 * f, t["bgu"])
            linear(got[-1] if case["gated"] else t["xd"], t["wd"], d, t["bd"])
        return got
    h = Q.grouped_gemm_fused(s["x"], s["offsets"], *s["w13"], 2 * case["f"], rows=s["rows"],
                             activation=Q.ACT_SILU_GATE, y=y())
    return [h, Q.grouped_gemm(h, s["offsets"], *s["w2"], case["d"], y=y())]


_capture_stream = None


def prepare(case, seed):
    global _capture_stream
    s = _inputs(case, seed)
    s["case"] = case
    if not case["graph"]:
        return s
    # the library's workspace belongs to the stream it was first needed on:
    # warm the capture stream up with the same calls, then capture them
    if _capture_stream is None:
        _capture_stream = torch.cuda.Stream()
    st = _capture_stream
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        s["out"] = _calls(case, s)
    torch.cuda.current_stream().wait_stream(st)
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"], stream=st):
        _calls(case, s, s["out"])
    return s


def run(state):
    case = state["case"]
    if case["graph"]:
        state["graph"].replay()
        return state["out"]
    return _calls(case, state)


# ---------------------------------------------------------------------------
# the same results in binary64
# ---------------------------------------------------------------------------

def _dequantized(w, k, n, index=0):
    """[K][N] binary64 weights (q - z) * s of one packed matrix.

    A unit of 16 columns x 128 channels (units ordered column tile, then
    channel group) is 64 lanes x 4 words: lane 16 g + c, word j holds channels
    32 j + 8 g .. + 7 of column c, even channels in nibbles 0..3 and odd ones
    in 4..7; scales are 16 values a unit, zero points 16 nibbles a unit."""
    packed, scales, zeros = w
    nt, kg = n // 16, k // 128
    p = packed.view(-1, nt, kg, 4, 16, 4)[index]
    shifts = torch.tensor([0, 16, 4, 20, 8, 24, 12, 28], device=p.device, dtype=torch.int32)
    q = ((p.unsqueeze(-1) >> shifts) & 15).to(torch.int8)             # nt, kg, g, c, j, e
    q = q.permute(1, 4, 2, 5, 0, 3).reshape(kg, 128, n)
    zs = torch.arange(0, 32, 4, device=p.device, dtype=torch.int32)
    z = ((zeros.view(-1, nt, kg, 2, 1)[index] >> zs) & 15).to(torch.int8).reshape(nt, kg, 16)
    z = z.permute(1, 0, 2).reshape(kg, 1, n)
    s = scales.view(torch.float16).view(-1, nt, kg, 16)[index].permute(1, 0, 2).reshape(kg, 1, n)
    return ((q - z).double() * s.double()).reshape(k, n)


def _exact_linear(x, w, k, n, bias=None, index=0):
    y = x.double() @ _dequantized(w, k, n, index)
    return y if bias is None else y + bias.double()


def _exact_gated(h, f):
    h = h.reshape(h.shape[0], f // 16, 2, 16)
    return (torch.nn.functional.silu(h[:, :, 0]) * h[:, :, 1]).reshape(h.shape[0], f)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "linear":
        return [_exact_linear(s["x"], s["w"], case["k"], case["n"])]
    if case["kind"] == "layer":
        d, f, qkv = case["d"], case["f"], case["qkv"]
        got = []
        for t in s["layers"]:
            got.append(_exact_linear(t["xq"], t["wq"], d, qkv, t["bq"]))
            got.append(_exact_linear(t["xo"], t["wo"], d, d, t["bo"]))
            h = _exact_linear(t["xm"], t["wgu"], d, 2 * f, t["bgu"])
            h = _exact_gated(h, f) if case["gated"] else h
            got += [h, _exact_linear(h if case["gated"] else t["xd"], t["wd"], f, d, t["bd"])]
        return got
    d, f = case["d"], case["f"]
    rows, at = s["rows"].long(), s["offsets"].tolist()
    hs, ys = [], []
    for e in range(case["experts"]):
        x = s["x"][rows[at[e]:at[e + 1]]]
        hs.append(_exact_gated(_exact_linear(x, s["w13"], d, 2 * f, index=e), f))
        ys.append(_exact_linear(hs[-1], s["w2"], f, d, index=e))
    return [torch.cat(hs), torch.cat(ys)]
