"""The work a user of this package has it do, as cases that can be timed.

Four kinds, all through the package's public entry points:

* ``op``: ``gtr_gla_fwd``, the chunkwise GLA operator on a token grid, with the
  options it is used with (the four scan directions, gate logits and the output
  gate fused in, initial and final state, float32);
* ``swiglu``: ``gtr_spatial_swiglu``, the block's channel mixer;
* ``block``: ``block.forward``, one GTR block;
* ``backbone``: a chain of blocks with weights of their own, the scan direction
  cycling from block to block.

Grids are images at patch stride 16 (640 x 640 pixels are 40 x 40 tokens, 1280 x
1280 are 80 x 80, 800 x 1328 are 50 x 83) and the operator's 256, 1.6K and 16.4K
tokens. Values follow ``paper_2609_26590_amd/workloads.py``. A case with
``graph`` is one that a program captures once in a HIP graph and replays (an
engine that serves one image at a time); the others are ordinary eager calls
into preallocated outputs (batches, or a single call).
"""
import math

import torch

import paper_2609_26590_amd as gtr
from paper_2609_26590_amd import block
from paper_2609_26590_amd.workloads import BLOCK_SIZES, GATE_RANK, SCANS

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
TAU, NORM_EPS, LN_EPS = 16.0, 1e-5, 1e-6


def op(name, B, heads, H, W, dk, dv, dtype, odtype, scans, fused=False, state=False, graph=True):
    case = {"kind": "op", "B": B, "heads": heads, "H": H, "W": W, "dk": dk, "dv": dv, "dtype": dtype, "odtype": odtype,
            "scans": scans, "fused": fused, "state": state, "graph": graph}
    return dict(case, name=name) if name else case


def swiglu(name, B, H, W, d, hidden, dtype, graph=False):
    case = {"kind": "swiglu", "B": B, "H": H, "W": W, "d": d, "hidden": hidden, "dtype": dtype, "graph": graph}
    return dict(case, name=name) if name else case


def blocks(name, model, depth, B, H, W, dtype, first, graph):
    case = {"kind": "block" if depth == 1 else "backbone", "model": model, "depth": depth, "B": B, "H": H, "W": W,
            "dtype": dtype, "first": first, "graph": graph}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: the paper's operator shape at 256 tokens, called eagerly (latency of one call)
        op("op_256_eager", 1, 6, 16, 16, 32, 64, "f16", "f16", "row", graph=False),
        # the operator at one 640 x 640 image as a block calls it: gate logits and output gate fused in
        op("op_640_fused", 1, 6, 40, 40, 64, 64, "f16", "f16", "col", fused=True),
        # the four scan directions of one image, bf16 inputs and float32 outputs
        op("op_640_directions", 1, 12, 40, 40, 64, 64, "bf16", "f32", "row,col,row_rev,col_rev"),
        # high resolution: one 1280 x 1280 image
        op("op_1280", 1, 6, 80, 80, 64, 64, "f16", "f16", "row"),
        # a batch of 8 images, states carried in and out (a sequence continued from call to call)
        op("op_batch8_state", 8, 12, 40, 40, 64, 64, "bf16", "f32", "row", state=True, graph=False),
        # long sequences: the paper's operator shape at 16.4K tokens, 4 images
        op("op_16k_batch4", 4, 6, 128, 128, 32, 64, "f16", "f16", "col_rev", graph=False),
        # float32, the precision for checking and for exporting a model: 2 images
        op("op_f32_batch2", 2, 12, 40, 40, 64, 64, "f32", "f32", "row", graph=False),
        # the channel mixer at the GTR-X width on a batch of 8 images
        swiglu("swiglu_x_batch8", 8, 40, 40, 384, 2304, "f16"),
        # one block of the small model, one image (an engine's unit of work)
        blocks("block_s_640", "gtr_s", 1, 1, 40, 40, "f16", "row", True),
        # one block of the large model on a batch of 8 images in bf16
        blocks("block_l_batch8", "gtr_l", 1, 8, 40, 40, "bf16", "col", False),
        # one block of the large model at 800 x 1328 pixels, 2 images: a grid that no tile divides
        blocks("block_l_ragged", "gtr_l", 1, 2, 50, 83, "f16", "row_rev", True),
        # a whole model's chain of blocks on one image, served from a graph
        blocks("backbone_l_640", "gtr_l", 12, 1, 40, 40, "f16", "row", True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _grid(rng, lo, hi):
    """H x W of lo to hi tokens, sides up to 2 : 1, odd sizes among them."""
    tokens, ratio = _log(rng, lo, hi), _log(rng, 0.5, 2.0)
    H = max(1, round(math.sqrt(tokens * ratio)))
    return H, max(1, min(round(tokens / H), int(hi) // H))


def draw(rng):
    kind = rng.choice(("op", "op", "op", "swiglu", "block", "block", "backbone"))
    dtype = rng.choice(("f16", "bf16"))
    if kind == "op":
        if rng.random() < 0.2:
            dtype = "f32"
        dk, dv = rng.choice(((64, 64), (64, 64), (32, 64), (32, 32)))
        H, W = _grid(rng, 256, 16384)
        # batch x heads x tokens up to the listed batches (float32: up to its listed case)
        most = (38400 if dtype == "f32" else 153600) / (H * W)
        heads = rng.choice([h for h in (2, 3, 6, 12) if h <= max(2, most)])
        B = max(1, min(8, int(_log(rng, 1, max(1.0, most / heads)))))
        fused = rng.random() < 0.4
        odtype = dtype if rng.random() < 0.7 else "f32"
        scans = ",".join(SCANS) if B * heads * H * W <= 19200 and rng.random() < 0.3 else rng.choice(SCANS)
        state = not fused and rng.random() < 0.4  # the gated operator is a block's, which carries no state
        return op(None, B, heads, H, W, dk, dv, dtype, odtype, scans, fused, state,
                  graph=B * heads * H * W <= 76800 and rng.random() < 0.7)
    if kind == "swiglu":
        H, W = _grid(rng, 256, 6400)
        d, hidden = rng.choice(((192, 768), (384, 1536), (384, 2304)))
        B = int(_log(rng, 1, max(1.0, min(8.99, 12800 / (H * W)))))
        return swiglu(None, B, H, W, d, hidden, dtype, graph=B * H * W <= 3200)
    model = rng.choice(sorted(BLOCK_SIZES))
    if kind == "block":
        H, W = _grid(rng, 256, 6400)
        B = int(_log(rng, 1, max(1.0, min(8.99, 12800 / (H * W)))))
        return blocks(None, model, 1, B, H, W, dtype, rng.choice(SCANS), graph=B * H * W <= 8300)
    H, W = _grid(rng, 256, 1600)
    return blocks(None, model, rng.choice((4, 6, 8, 12)), 1, H, W, "f16", rng.choice(SCANS), True)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _draws(seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    return lambda *shape, std=1.0, mu=0.0: torch.randn(shape, generator=gen, device="cuda") * std + mu


def _op_inputs(case, seed):
    n, dt = _draws(seed), DTYPES[case["dtype"]]
    B, h, L, dk, dv = case["B"], case["heads"], case["H"] * case["W"], case["dk"], case["dv"]
    x = {"q": n(B, h, L, dk, std=dk ** -0.5).to(dt), "k": n(B, h, L, dk, std=dk ** -0.5).to(dt),
         "v": n(B, h, L, dv).to(dt), "s0": n(B, h, dk, dv, std=0.1) if case["state"] else None}
    if case["fused"]:  # gate logits, the output gate before its SiLU, the RMSNorm weight
        x["g"] = n(B, h, L, dk, std=0.5, mu=2.0).to(dt)
        x["z"] = n(B, h, L, dv).to(dt)
        x["w"] = n(dv, std=0.1, mu=1.0)
    else:  # log-decays
        x["g"] = torch.nn.functional.logsigmoid(n(B, h, L, dk, mu=3.0)).to(dt)
    return x


def _swiglu_inputs(case, seed):
    n, dt = _draws(seed), DTYPES[case["dtype"]]
    d, hid = case["d"], case["hidden"]
    return {"x": n(case["B"], case["H"] * case["W"], d).to(dt), "w_g": n(hid, d, std=d ** -0.5).to(dt),
            "w_v": n(hid, d, std=d ** -0.5).to(dt), "w_out": n(d, hid, std=hid ** -0.5).to(dt),
            "conv_w": n(hid, 3, 3, std=1 / 3), "conv_b": n(hid, std=0.1)}


def _block_inputs(case, seed):
    n, dt = _draws(seed), DTYPES[case["dtype"]]
    d, heads = BLOCK_SIZES[case["model"]]
    hid, ps = 4 * d, []
    x = n(case["B"], case["H"] * case["W"], d).to(dt)
    for _ in range(case["depth"]):
        ps.append({
            "ln1_w": n(d, std=0.1, mu=1.0), "ln1_b": n(d, std=0.1), "w_qkvr": n(4 * d, d, std=d ** -0.5).to(dt),
            "w_a1": n(GATE_RANK, d, std=d ** -0.5).to(dt), "w_a2": n(d, GATE_RANK, std=GATE_RANK ** -0.5).to(dt),
            "b_a": n(d, std=0.5, mu=2.0), "norm_w": n(d // heads, std=0.1, mu=1.0),
            "w_o": n(d, d, std=d ** -0.5).to(dt), "ln2_w": n(d, std=0.1, mu=1.0), "ln2_b": n(d, std=0.1),
            "w_g": n(hid, d, std=d ** -0.5).to(dt), "w_v": n(hid, d, std=d ** -0.5).to(dt),
            "w_out": n(d, hid, std=hid ** -0.5).to(dt), "conv_w": n(hid, 3, 3, std=1 / 3), "conv_b": n(hid, std=0.1)})
    return x, ps, heads


def _directions(case):
    """The scan direction of each block of a chain."""
    at = SCANS.index(case["first"])
    return [SCANS[(at + i) % 4] for i in range(case["depth"])]


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------
_capture_stream = None


def _captured(call):
    """`call` in a HIP graph, after one eager call on the capture stream."""
    global _capture_stream
    if _capture_stream is None:
        _capture_stream = torch.cuda.Stream()
    here = torch.cuda.current_stream()
    _capture_stream.wait_stream(here)
    with torch.cuda.stream(_capture_stream):
        call()
    here.wait_stream(_capture_stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=_capture_stream):
        out = call()
    return graph, out


def _op_call(case, seed):
    x = _op_inputs(case, seed)
    B, h, L, dk, dv = case["B"], case["heads"], case["H"] * case["W"], case["dk"], case["dv"]
    scans, ws = case["scans"].split(","), gtr.Workspace()
    outs = [torch.empty((B, h, L, dv), dtype=DTYPES[case["odtype"]], device="cuda") for _ in scans]
    finals = [torch.empty((B, h, dk, dv), device="cuda") if case["state"] else None for _ in scans]
    more = dict(gate_tau=TAU, out_gate=x["z"], norm_weight=x["w"], norm_eps=NORM_EPS) if case["fused"] else {}

    def call():
        for scan, o, sf in zip(scans, outs, finals):
            gtr.gtr_gla_fwd(x["q"], x["k"], x["v"], x["g"], H=case["H"], W=case["W"], scan=scan, s0=x["s0"], out=o,
                            s_final=sf, workspace=ws, **more)
        return outs, finals
    return call


def _swiglu_call(case, seed):
    x, ws = _swiglu_inputs(case, seed), gtr.Workspace()
    y = torch.empty_like(x["x"])
    return lambda: gtr.gtr_spatial_swiglu(x["x"], x["w_g"], x["w_v"], x["w_out"], x["conv_w"], x["conv_b"],
                                          H=case["H"], W=case["W"], out=y, workspace=ws)


def _block_call(case, seed):
    x, ps, heads = _block_inputs(case, seed)
    ready = [block.prepare(p) for p in ps]
    scans = _directions(case)

    def call():
        y = x
        for p, scan in zip(ready, scans):
            y = block.forward(y, p, H=case["H"], W=case["W"], heads=heads, scan=scan, tau=TAU, ln_eps=LN_EPS,
                              norm_eps=NORM_EPS)
        return y
    return call


def prepare(case, seed):
    call = {"op": _op_call, "swiglu": _swiglu_call}.get(case["kind"], _block_call)(case, seed)
    if not case["graph"]:
        return {"call": call}
    graph, out = _captured(call)
    return {"graph": graph, "out": out, "call": call}


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return state["call"]()


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _size(dtype):
    return 4 if dtype == "f32" else 2


def _op_flops(tokens, dk, dv, C=64):
    """Chunkwise GLA per token and head: the causal halves of the two intra-chunk products, summary and readout."""
    return tokens * ((dk + dv) * (C + 1) + 4 * dk * dv)


def work(case):
    M = case["B"] * case["H"] * case["W"]
    s = _size(case["dtype"])
    if case["kind"] == "op":
        n, dk, dv, calls = M * case["heads"], case["dk"], case["dv"], len(case["scans"].split(","))
        rows = (3 * dk + dv + (dv if case["fused"] else 0)) * s
        state = case["B"] * case["heads"] * dk * dv * 4 if case["state"] else 0
        return {"bytes": n * rows + state + calls * (n * dv * _size(case["odtype"]) + state),
                "flops": calls * _op_flops(n, dk, dv)}
    if case["kind"] == "swiglu":
        d, hid = case["d"], case["hidden"]
        return {"bytes": 2 * M * d * s + 3 * d * hid * s + 40 * hid, "flops": 6.0 * M * d * hid + 18.0 * M * hid}
    d, heads = BLOCK_SIZES[case["model"]]
    hid, dh = 4 * d, d // heads
    flops = 2.0 * M * d * 6 * d + _op_flops(M * heads, dh, dh) + 6.0 * M * d * hid + 18.0 * M * hid
    weights = (6 * d * d + 3 * d * hid) * s + (9 * d + 10 * hid) * 4
    return {"bytes": 2 * M * d * s + case["depth"] * weights, "flops": case["depth"] * flops}


def tolerance(case):
    # about four times the error of the results against 64 bits (rel / max seen: float32 2.2e-7 / 3.7e-6, the operator
    # 4.7e-4 / 6e-3 and 1.7e-3 with bf16 results, the mixer 4.4e-4 / 2.4e-3, a block 6.3e-4 / 4.5e-3 and in bf16 4.6e-3 /
    # 2.4e-2, twelve blocks 3.5e-3 / 2e-2, where the largest difference grows from block to block)
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "op":
        if case["dtype"] == "f32":
            return {"rel": 1e-6, "max": 1.5e-5}
        return {"rel": 7e-3, "max": 4e-2} if case["odtype"] == "bf16" else {"rel": 2e-3, "max": 2.5e-2}
    if case["kind"] == "swiglu":
        return {"rel": 7e-3, "max": 3e-2} if bf16 else {"rel": 1.8e-3, "max": 1e-2}
    if case["kind"] == "block":
        return {"rel": 1.8e-2, "max": 1e-1} if bf16 else {"rel": 2.5e-3, "max": 2e-2}
    return {"rel": 1.4e-2, "max": 3e-1}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
def _order(H, W, scan):
    """Row-major index of the token visited at each step of a scan."""
    i = torch.arange(H * W, device="cuda").reshape(H, W)
    i = (i.t() if scan.startswith("col") else i).reshape(-1)
    return i.flip(0) if scan.endswith("rev") else i


def _gla64(q, k, v, g, s0, H, W, scan):
    """The recurrence token by token; q .. g [B, heads, L, d] float64."""
    order = _order(H, W, scan)
    q, k, v, d = (t[:, :, order].permute(2, 0, 1, 3).contiguous() for t in (q, k, v, g.exp()))
    L, B, h, dk = q.shape
    dv = v.shape[-1]
    S = torch.zeros((B, h, dk, dv), dtype=torch.float64, device="cuda") if s0 is None else s0.double()
    o = torch.empty((L, B, h, dv), dtype=torch.float64, device="cuda")
    for t in range(L):
        S = S * d[t, :, :, :, None] + k[t, :, :, :, None] * v[t, :, :, None, :]
        torch.sum(S * q[t, :, :, :, None], dim=2, out=o[t])
    back = torch.empty_like(order)
    back[order] = torch.arange(L, device="cuda")
    return o[back].permute(1, 2, 0, 3) * dk ** -0.5, S


def _gate64(o, z, w):
    return z * torch.sigmoid(z) * o * torch.rsqrt((o * o).mean(-1, keepdim=True) + NORM_EPS) * w


def _swiglu64(x, w_g, w_v, w_out, conv_w, conv_b, H, W):
    B, L, _ = x.shape
    gate, val = x @ w_g.t(), (x @ w_v.t()).reshape(B, H, W, -1)
    pad = torch.nn.functional.pad(val, (0, 0, 1, 1, 1, 1))
    conv = conv_b + sum(pad[:, u:u + H, t:t + W] * conv_w[:, u, t] for u in range(3) for t in range(3))
    return (gate * torch.sigmoid(gate) * conv.reshape(B, L, -1)) @ w_out.t()


def _norm64(x, w, b):
    c = x - x.mean(-1, keepdim=True)
    return c * torch.rsqrt((c * c).mean(-1, keepdim=True) + LN_EPS) * w + b


def exact(case, seed):
    H, W = case["H"], case["W"]
    if case["kind"] == "op":
        x = {n: None if t is None else t.double() for n, t in _op_inputs(case, seed).items()}
        g = torch.nn.functional.logsigmoid(x["g"]) / TAU if case["fused"] else x["g"]
        got = [_gla64(x["q"], x["k"], x["v"], g, x["s0"], H, W, scan) for scan in case["scans"].split(",")]
        return ([_gate64(o, x["z"], x["w"]) if case["fused"] else o for o, _ in got],
                [S if case["state"] else None for _, S in got])
    if case["kind"] == "swiglu":
        x = {n: t.double() for n, t in _swiglu_inputs(case, seed).items()}
        return _swiglu64(x["x"], x["w_g"], x["w_v"], x["w_out"], x["conv_w"], x["conv_b"], H, W)
    x, ps, heads = _block_inputs(case, seed)
    x = x.double()
    B, L, d = x.shape
    split = lambda t: t.reshape(B, L, heads, d // heads).permute(0, 2, 1, 3)  # noqa: E731
    for p, scan in zip(ps, _directions(case)):
        p = {n: t.double() for n, t in p.items()}
        n1 = _norm64(x, p["ln1_w"], p["ln1_b"])
        q, k, v, z = ((n1 @ w.t()) for w in p["w_qkvr"].split(d))
        a = n1 @ p["w_a1"].t() @ p["w_a2"].t() + p["b_a"]
        o, _ = _gla64(split(q), split(k), split(v), torch.nn.functional.logsigmoid(split(a)) / TAU, None, H, W, scan)
        u = _gate64(o, split(z), p["norm_w"]).permute(0, 2, 1, 3).reshape(B, L, d)
        x = x + u @ p["w_o"].t()
        x = x + _swiglu64(_norm64(x, p["ln2_w"], p["ln2_b"]), p["w_g"], p["w_v"], p["w_out"], p["conv_w"], p["conv_b"], H, W)
    return x
