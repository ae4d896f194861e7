"""Timing cases of the sparse linear-layer path: what a training or inference program calls, at the sizes it calls it with.

A case is a dict of plain values.  Its "what" says which part of a program it stands for:

  layer   one linear layer's training step: re-projection of the weight, forward product, input gradient, weight
          gradient.  The unit everything else repeats.
  ffn     the feed-forward block's training step (two layers and the activation fused into their epilogues), in bf16 or
          in the 8-bit recipe (e4m3 weights and activations, e5m2 gradients, held scales, casts inside the step).
  block   the four linears of a transformer block (attention input and output, the two feed-forward layers), their
          weights re-projected by one multi-tensor launch, each with forward, input gradient and weight gradient.
  infer   the feed-forward block's forward pass alone on packed weights: a decode batch, a prompt.
  update  the end of an iteration: the dense-weight step and the re-projection of every sparse weight of a model in one
          multi-tensor launch.

Inputs have the distributions the synthetic workloads of this package state (W ~ N(0, 0.02), X ~ N(0, 1),
dY ~ N(0, 1e-3), weight steps ~ N(0, 1e-4)); weights, workspaces, outputs, scales and multi-tensor tables are what such
a program keeps from iteration to iteration.
"""
import torch

import paper_2409_09099_amd as sste
from paper_2409_09099_amd import workloads as WL

BETA = 1.4830322          # the frozen scale of a Gaussian weight
FMT_MAX = {"e4m3": 448.0, "e5m2": 57344.0}
MOST_WORK = 32768 * (3 + 1 + 4 + 4) * 1280 * 1280   # tokens x weights of the largest block


def listed():
    return [
        # the tiny layer of the first workload: every kernel is a few microseconds, launches and host time count
        dict(name="layer_tiny_bf16", what="layer", fmt="bf16", grad="bf16", out="bf16", T=512, O=256, I=1024),
        # first feed-forward layer of the 124M model, batch 8 x 1024
        dict(name="layer_124m_fc1_bf16", what="layer", fmt="bf16", grad="bf16", out="bf16", T=8192, O=3072, I=768),
        # odd widths and a token count that ends inside every tile
        dict(name="layer_ragged_bf16", what="layer", fmt="bf16", grad="bf16", out="bf16", T=2112, O=1544, I=832),
        # the same in 8 bits, e5m2 gradients, the output cast where it is produced
        dict(name="layer_ragged_fp8", what="layer", fmt="e4m3", grad="e5m2", out="e4m3", T=3200, O=1552, I=896),
        # feed-forward block of the 350M model, batch 16 x 1024
        dict(name="ffn_350m_bf16", what="ffn", fmt="bf16", grad="bf16", T=16384, d=1024),
        # feed-forward block of the 774M model in the 8-bit recipe
        dict(name="ffn_774m_fp8", what="ffn", fmt="e4m3", grad="e5m2", T=32768, d=1280),
        # the whole block of the 774M model, bf16 and e4m3 (the benchmark's two large workloads with their input gradients)
        dict(name="block_774m_bf16", what="block", fmt="bf16", grad="bf16", T=16384, d=1280),
        dict(name="block_774m_e4m3", what="block", fmt="e4m3", grad="e4m3", T=32768, d=1280),
        # decode: one token of each of 16 sequences
        dict(name="infer_decode_bf16", what="infer", fmt="bf16", T=16, d=1280),
        # a prompt of odd length
        dict(name="infer_prompt_e4m3", what="infer", fmt="e4m3", T=1021, d=1280),
        # every weight of the 124M model, float32 dense weights, 8-bit operands
        dict(name="update_124m_f32", what="update", fmt="e4m3", master="f32", layers=12, d=768),
        # every weight of the 774M model, bf16 dense weights
        dict(name="update_774m_bf16", what="update", fmt="bf16", master="bf16", layers=36, d=1280),
    ]


def draw(rng):
    def spread(lo, hi, step):
        v = lo * (hi / lo) ** rng.random()
        return int(min(max(round(v / step), -(-lo // step)), hi // step)) * step

    what = rng.choice(["layer"] * 4 + ["ffn"] * 2 + ["block"] * 2 + ["infer"] * 2 + ["update"] * 2)
    fmt = rng.choice(["bf16", "e4m3"])
    fp8 = fmt == "e4m3"
    ks = 128 if fp8 else 64                                # whole instruction steps along a contraction
    grad = rng.choice(["e4m3", "e5m2"]) if fp8 else "bf16"
    if what == "layer":
        O, I = spread(256, 5120, 16 if fp8 else 8), spread(256, 5120, ks)
        T = spread(512, max(512, min(32768, MOST_WORK // (O * I))), ks)
        return dict(what=what, fmt=fmt, grad=grad, out=rng.choice(["bf16", "e4m3"]) if fp8 else "bf16", T=T, O=O, I=I)
    if what == "infer":
        return dict(what=what, fmt=fmt, T=spread(1, 2048, 1), d=spread(256, 1280, ks))
    if what == "update":
        return dict(what=what, fmt=fmt, master=rng.choice(["bf16", "f32"]), layers=spread(1, 36, 1), d=spread(256, 1280, 128))
    return dict(what=what, fmt=fmt, grad=grad, T=spread(512, 32768, ks), d=spread(256, 1280, ks))


def _code(name):
    return {"bf16": sste.BF16, "e4m3": sste.F8E4M3, "e5m2": sste.F8E5M2}[name]


class _Inputs:
    """Gaussian tensors on the GPU, from the seed alone."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, rows, cols, std, dtype=torch.bfloat16):
        return torch.empty((rows, cols), dtype=dtype, device="cuda").normal_(0.0, std, generator=self.g)

    def operand(self, rows, cols, std, fmt):
        """(tensor, scale) of a GEMM operand: bf16 with scale 1, or 8-bit codes under the tensor's own scale."""
        x = self.normal(rows, cols, std)
        if fmt == "bf16":
            return x, 1.0
        scale = float(x.abs().max()) / FMT_MAX[fmt]
        return sste.cast_fp8(x, scale, _code(fmt))[0], scale


def _weight_scale(W, fmt):
    """Scale of the packed 8-bit weight: from the largest magnitude of the projection, 1 for bf16."""
    if fmt == "bf16":
        return 1.0
    amax = torch.zeros(1, dtype=torch.float32, device="cuda")
    sste.project_pack(W, BETA, sste.BF16, 1.0, amax_out=amax)
    return float(amax) / FMT_MAX["e4m3"]


def _linear(inp, T, O, I, case):
    """One linear layer's operands, outputs and workspace."""
    fmt, grad = case["fmt"], case["grad"]
    L = dict(O=O, I=I, W=inp.normal(O, I, WL.W_STD))
    L["X"], L["xs"] = inp.operand(T, I, WL.X_STD, fmt)
    L["dY"], L["dys"] = inp.operand(T, O, WL.DY_STD, grad)
    L["ws"] = _weight_scale(L["W"], fmt)
    L["vals"], L["meta"] = sste.packed_buffers(O, I, _code(fmt), "cuda")
    z8 = case.get("out", "bf16") == "e4m3"
    L["Z"] = torch.empty((T, O), dtype=torch.uint8 if z8 else torch.bfloat16, device="cuda")
    # a layer whose output is cast where it is produced takes its scale from earlier iterations
    L["zs"] = 6.0 * WL.X_STD * WL.W_STD * I ** 0.5 / FMT_MAX["e4m3"] if z8 else 1.0
    L["z_amax"] = torch.empty(1, dtype=torch.float32, device="cuda")
    L["dX"] = torch.empty((T, I), dtype=torch.bfloat16, device="cuda")
    L["dW"] = torch.empty((O, I), dtype=torch.float32, device="cuda")
    L["scratch"] = torch.empty(max(16, sste.wgrad_workspace_bytes(T, O, I, _code(grad))), dtype=torch.uint8, device="cuda")
    return L


def _prepare_ffn(inp, case):
    T, d, h, fmt, grad = case["T"], case["d"], 4 * case["d"], case["fmt"], case["grad"]
    f8, dt, gdt = fmt != "bf16", _code(fmt), _code(grad)
    new = lambda rows, cols, dtype=torch.bfloat16: torch.empty((rows, cols), dtype=dtype, device="cuda")  # noqa: E731
    s = dict(W1=inp.normal(h, d, WL.W_STD), W2=inp.normal(d, h, WL.W_STD), dYb=inp.normal(T, d, WL.DY_STD))
    s["X"], s["xs"] = inp.operand(T, d, WL.X_STD, fmt)
    for k, W in (("1", s["W1"]), ("2", s["W2"])):
        s["ws" + k] = _weight_scale(W, fmt)
        s["v" + k], s["m" + k] = sste.packed_buffers(W.shape[0], W.shape[1], dt, "cuda")
        s["dW" + k] = new(W.shape[0], W.shape[1], torch.float32)
        s["scratch" + k] = torch.empty(max(16, sste.wgrad_workspace_bytes(T, W.shape[0], W.shape[1], gdt)), dtype=torch.uint8, device="cuda")
    s["H"], s["dH"], s["Y"], s["dX"] = new(T, h), new(T, h), new(T, d), new(T, d)
    s["A"] = new(T, h, torch.uint8 if f8 else torch.bfloat16)
    if f8:
        s["dY8"], s["dH8"] = new(T, d, torch.uint8), new(T, h, torch.uint8)
        s["amax"] = [torch.empty(1, dtype=torch.float32, device="cuda") for _ in range(3)]
        # held scales, with head room over what these distributions reach
        s["a_scale"] = 7.0 * WL.W_STD * d ** 0.5 / FMT_MAX["e4m3"]
        s["dys"] = 7.0 * WL.DY_STD / FMT_MAX[grad]
        s["dhs"] = 9.0 * WL.DY_STD * WL.W_STD * d ** 0.5 / FMT_MAX[grad]
    return s


def _run_ffn(s):
    c = s["case"]
    d, h = c["d"], 4 * c["d"]
    if c["fmt"] == "bf16":
        sste.project_pack(s["W1"], BETA, vals=s["v1"], meta=s["m1"])
        sste.project_pack(s["W2"], BETA, vals=s["v2"], meta=s["m2"])
        sste.linear_fwd_act(s["X"], s["v1"], s["m1"], h, H=s["H"], A=s["A"])
        sste.linear_fwd(s["A"], s["v2"], s["m2"], d, Z=s["Y"])
        sste.linear_dgrad_act(s["dYb"], s["v2"], s["m2"], h, s["H"], dX=s["dH"])
        sste.linear_wgrad(s["dYb"], s["A"], seed=s["seed"], offset=0, dW=s["dW2"], workspace=s["scratch2"])
        sste.linear_wgrad(s["dH"], s["X"], seed=s["seed"], offset=1, dW=s["dW1"], workspace=s["scratch1"])
        sste.linear_dgrad(s["dH"], s["v1"], s["m1"], d, dX=s["dX"])
        return {k: s[k] for k in ("v1", "m1", "v2", "m2", "H", "A", "Y", "dH", "dW1", "dW2", "dX")}
    f8, g8, xs, ws1, ws2, a_s, dys, dhs = sste.F8E4M3, _code(c["grad"]), s["xs"], s["ws1"], s["ws2"], s["a_scale"], s["dys"], s["dhs"]
    sste.project_pack(s["W1"], BETA, f8, ws1, vals=s["v1"], meta=s["m1"])
    sste.project_pack(s["W2"], BETA, f8, ws2, vals=s["v2"], meta=s["m2"])
    sste.linear_fwd_act(s["X"], s["v1"], s["m1"], h, f8, xs, ws1, a_dtype=f8, a_scale=a_s, H=s["H"], A=s["A"], amax_out=s["amax"][0])
    sste.linear_fwd(s["A"], s["v2"], s["m2"], d, f8, a_s, ws2, Z=s["Y"])
    sste.cast_fp8(s["dYb"], dys, g8, Q=s["dY8"], amax_out=s["amax"][1])
    sste.linear_dgrad_act(s["dY8"], s["v2"], s["m2"], h, s["H"], g8, dys, ws2, dX=s["dH"])
    sste.cast_fp8(s["dH"], dhs, g8, Q=s["dH8"], amax_out=s["amax"][2])
    sste.linear_wgrad(s["dY8"], s["A"], seed=s["seed"], offset=0, dtype=g8, dy_scale=dys, x_scale=a_s, dW=s["dW2"], workspace=s["scratch2"])
    sste.linear_wgrad(s["dH8"], s["X"], seed=s["seed"], offset=1, dtype=g8, dy_scale=dhs, x_scale=xs, dW=s["dW1"], workspace=s["scratch1"])
    sste.linear_dgrad(s["dH8"], s["v1"], s["m1"], d, g8, dhs, ws1, dX=s["dX"])
    out = {k: s[k] for k in ("v1", "m1", "v2", "m2", "H", "A", "Y", "dY8", "dH", "dH8", "dW1", "dW2", "dX")}
    out["amax"] = s["amax"]
    return out


def _block_shapes(d):
    return [(3 * d, d), (d, d), (4 * d, d), (d, 4 * d)]


def _prepare_update(inp, case):
    """The weights of a model as one buffer per kind (dense weights, gradients, packed values, position bits), cut into tensors."""
    dt, f32 = _code(case["fmt"]), case["master"] == "f32"
    shapes = _block_shapes(case["d"]) * case["layers"]
    n = sum(O * I for O, I in shapes)
    s = dict(W=inp.normal(1, n, WL.W_STD, torch.float32 if f32 else torch.bfloat16).view(-1), G=inp.normal(1, n, WL.DY_STD, torch.float32).view(-1))
    s["vals"] = torch.empty(n // 2, dtype=torch.uint8 if dt == sste.F8E4M3 else torch.int16, device="cuda")
    s["meta"] = torch.empty(n // 8, dtype=torch.uint8, device="cuda")
    Ws, Gs, vs, ms, at = [], [], [], [], 0
    for O, I in shapes:
        m = O * I
        Ws.append(s["W"][at:at + m].view(O, I))
        Gs.append(s["G"][at:at + m].view(O, I))
        vs.append(s["vals"][at // 2:(at + m) // 2].view(O, I // 2))
        ms.append(s["meta"][at // 8:(at + m) // 8].view(O, I // 8))
        at += m
    scale = 1.0 if case["fmt"] == "bf16" else 5.0 * BETA * WL.W_STD / FMT_MAX["e4m3"]
    s["batch"] = sste.UpdateBatch(Ws, Gs, [BETA] * len(Ws), dt, [scale] * len(Ws), vals=vs, metas=ms)
    return s


def prepare(case, seed):
    inp = _Inputs(seed)
    what = case["what"]
    if what == "layer":
        s = dict(layers=[_linear(inp, case["T"], case["O"], case["I"], case)])
    elif what == "block":
        s = dict(layers=[_linear(inp, case["T"], O, I, case) for O, I in _block_shapes(case["d"])])
        L = s["layers"]
        s["pack"] = sste.PackBatch([x["W"] for x in L], [BETA] * 4, _code(case["fmt"]), [x["ws"] for x in L], [x["vals"] for x in L],
                                   [x["meta"] for x in L])
    elif what == "ffn":
        s = _prepare_ffn(inp, case)
    elif what == "infer":
        T, d, fmt = case["T"], case["d"], case["fmt"]
        s = dict(a_scale=7.0 * WL.W_STD * d ** 0.5 / FMT_MAX["e4m3"] if fmt == "e4m3" else 1.0)
        s["X"], s["xs"] = inp.operand(T, d, WL.X_STD, fmt)
        for k, (O, I) in (("1", (4 * d, d)), ("2", (d, 4 * d))):
            W = inp.normal(O, I, WL.W_STD)
            s["ws" + k] = _weight_scale(W, fmt)
            s["v" + k], s["m" + k] = sste.project_pack(W, BETA, _code(fmt), s["ws" + k])
        s["A"] = torch.empty((T, 4 * d), dtype=torch.uint8 if fmt == "e4m3" else torch.bfloat16, device="cuda")
        s["amax"] = torch.empty(1, dtype=torch.float32, device="cuda") if fmt == "e4m3" else None
        s["Y"] = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    else:
        s = _prepare_update(inp, case)
    s["case"], s["seed"] = case, seed
    return s


def run(s):
    c = s["case"]
    what = c["what"]
    if what in ("layer", "block"):
        dt, gdt = _code(c["fmt"]), _code(c["grad"])
        if what == "block":
            s["pack"].launch()
        out = []
        for k, L in enumerate(s["layers"]):
            if what == "layer":
                sste.project_pack(L["W"], BETA, dt, L["ws"], vals=L["vals"], meta=L["meta"])
            o = [L["vals"], L["meta"], L["Z"], L["dX"], L["dW"]]
            if c.get("out", "bf16") == "e4m3":
                sste.linear_fwd_ex(L["X"], L["vals"], L["meta"], L["O"], dt, L["xs"], L["ws"], sste.F8E4M3, L["zs"], Z=L["Z"], amax_out=L["z_amax"])
                o.append(L["z_amax"])
            else:
                sste.linear_fwd(L["X"], L["vals"], L["meta"], L["O"], dt, L["xs"], L["ws"], Z=L["Z"])
            sste.linear_dgrad(L["dY"], L["vals"], L["meta"], L["I"], gdt, L["dys"], L["ws"], dX=L["dX"])
            sste.linear_wgrad(L["dY"], L["X"], seed=s["seed"], offset=k, dtype=gdt, dy_scale=L["dys"], x_scale=L["xs"], dW=L["dW"],
                              workspace=L["scratch"])
            out.append(o)
        return out
    if what == "ffn":
        return _run_ffn(s)
    if what == "infer":
        d, dt = c["d"], _code(c["fmt"])
        sste.linear_fwd_act(s["X"], s["v1"], s["m1"], 4 * d, dt, s["xs"], s["ws1"], a_dtype=dt, a_scale=s["a_scale"], A=s["A"],
                            amax_out=s["amax"], store_pre=False)
        sste.linear_fwd(s["A"], s["v2"], s["m2"], d, dt, s["a_scale"], s["ws2"], Z=s["Y"])
        out = [s["A"], s["Y"]]
        return out + [s["amax"]] if dt == sste.F8E4M3 else out
    s["batch"].launch(WL.UPDATE_STD / WL.DY_STD)
    return [s["W"], s["vals"], s["meta"]]


def work(case):
    """Bytes: each input read once, each output written once (the sparsified gradient is no output and counts nothing).
    Flops: two per multiply-add with an element that is stored, i.e. T O I for the products with a 2:4 operand
    (forward, weight gradient) and 2 T O I for the dense one (input gradient)."""
    what, fmt = case["what"], case["fmt"]
    b = 1 if fmt == "e4m3" else 2                          # operand bytes
    packed = 0.5 * b + 0.125                               # packed operand bytes per weight
    if what == "update":
        n = case["layers"] * sum(O * I for O, I in _block_shapes(case["d"]))
        return {"bytes": n * (4 + 2 * (4 if case["master"] == "f32" else 2) + packed), "flops": 0.0}
    T = case["T"]
    if what == "infer":
        d = case["d"]
        return {"bytes": T * d * b + 2 * 4 * d * d * packed + T * 4 * d * b + T * d * 2, "flops": 2.0 * T * 4 * d * d}
    if what == "ffn":
        d, h = case["d"], 4 * case["d"]
        bytes_ = 2 * d * h * (2 + packed + 4) + T * d * (b + 2 + 2 + 2) + T * h * (2 + b + 2)
        if b == 1:
            bytes_ += T * (d + h)                          # the cast gradients
        return {"bytes": bytes_, "flops": 8.0 * T * d * h}
    shapes = [(case["O"], case["I"])] if what == "layer" else _block_shapes(case["d"])
    z = 1 if case.get("out", "bf16") == "e4m3" else 2
    bytes_ = sum(O * I * (2 + packed + 4) + T * I * (b + 2) + T * O * (b + z) for O, I in shapes)
    return {"bytes": bytes_, "flops": sum(4.0 * T * O * I for O, I in shapes)}


def tolerance(case):
    """Packed weights and updated dense weights are exact.  Products: float32 sums in any order, so bf16 results differ
    by single roundings here and there; an 8-bit code written from such a sum moves to its neighbour where the sum sits on
    a rounding boundary (the share the parity tests allow)."""
    if case["what"] == "update":
        return "exact"
    codes = case["fmt"] == "e4m3" and (case["what"] in ("ffn", "infer") or case.get("out") == "e4m3")
    return {"rel": 5e-3, "differ": 2e-3 if codes else 0.0}
