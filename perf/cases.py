"""What the fused MoE layer's speed is measured on: whole layer calls through
the package's public ``moe_forward``, over the formats, batch sizes and layer
shapes that a serving program runs.

The listed cases are the repository's benchmark workloads (plus two batches of
in-between size, one of them odd); ``draw`` spreads over the same layers, every
weight format, one to 8192 tokens, both output types, and logits given or
computed by the router in front.

Values: hidden ~ N(0, 1) in bf16, expert weights ~ N(0, 1/fan_in) quantised to
the format's storage (fp8: 128x128 blocks scaled to 448; int4: 128-groups
scaled to 7; MXFP4: OCP MX blocks of 32), logits ~ N(0, 1) plus the layer's own
routing bias, so experts are loaded as unevenly as the workloads have them.
"""
import functools
import math

import torch

import paper_2607_12875_amd as moe

# The layers: hidden size, experts, expert width, experts per token, scoring
# and routing bias ("normal": std of a per-expert logit bias; "zipf": its
# exponent; "sel": std of the sigmoid's selection-only bias).
LAYERS = {
    "tiny": dict(H=256, E=8, I=128, k=2, mode="softmax", scale=1.0, bias="none", amount=0.0),
    "wide64": dict(H=4096, E=64, I=1408, k=6, mode="softmax", scale=1.0, bias="normal", amount=0.5),
    "even64": dict(H=4096, E=64, I=1408, k=6, mode="softmax", scale=1.0, bias="none", amount=0.0),
    "zipf128": dict(H=4096, E=128, I=1536, k=8, mode="softmax", scale=1.0, bias="zipf", amount=1.1),
    "large256": dict(H=7168, E=256, I=2048, k=8, mode="sigmoid", scale=2.5, bias="sel", amount=0.1),
    "small60": dict(H=2048, E=60, I=1408, k=4, mode="softmax", scale=1.0, bias="normal", amount=0.5),
    "mid160": dict(H=5120, E=160, I=1536, k=6, mode="softmax", scale=1.0, bias="normal", amount=0.5),
}
WEIGHT_BYTES = {"bf16": 2.0, "fp8": 1.0 + 4.0 / 16384, "fp8a16": 1.0 + 4.0 / 16384, "int4": 0.5 + 2.0 / 128,
                "mxfp4": 0.5 + 1.0 / 32, "mxfp4x8": 0.5 + 1.0 / 32}


def _case(layer, T, wfmt, router=False, out="f32"):
    return dict(layer=layer, T=T, wfmt=wfmt, router=router, out=out)


def listed():
    return [
        # the smallest call: a toy layer, bound by launches and latency
        dict(name="tiny-bf16-64", **_case("tiny", 64, "bf16")),
        # one decode step of 16 sequences, router included, bf16 weights
        dict(name="decode-bf16-16", **_case("even64", 16, "bf16", router=True)),
        # a chunk of a prompt beside running sequences: between decode and prefill, odd
        dict(name="chunk-bf16-777", **_case("wide64", 777, "bf16", out="bf16")),
        # a whole prefill batch in bf16, unevenly loaded experts
        dict(name="prefill-bf16-4096", **_case("wide64", 4096, "bf16")),
        # the largest layer in block-scaled fp8: a prefill batch (the benchmark's default)
        dict(name="prefill-fp8-8192", **_case("large256", 8192, "fp8")),
        # the same layer and format serving a few hundred sequences, router included
        dict(name="batch-fp8-300", **_case("large256", 300, "fp8", router=True, out="bf16")),
        # int4 weights, skewed experts: a middle-sized batch
        dict(name="batch-int4-512", **_case("zipf128", 512, "int4")),
        # int4 weights, one decode step
        dict(name="decode-int4-16", **_case("zipf128", 16, "int4")),
        # fp8 weights with bf16 activations, one decode step
        dict(name="decode-fp8a16-16", **_case("large256", 16, "fp8a16")),
        # MXFP4 weights with bf16 activations: one decode step and a prefill batch
        dict(name="decode-mxfp4-16", **_case("large256", 16, "mxfp4")),
        dict(name="prefill-mxfp4-8192", **_case("large256", 8192, "mxfp4")),
        # MXFP4 weights with MXFP8 activations: a prefill batch
        dict(name="prefill-mxfp4x8-8192", **_case("large256", 8192, "mxfp4x8")),
    ]


def draw(rng):
    layer = rng.choice(sorted(LAYERS))
    wfmt = rng.choice(sorted(WEIGHT_BYTES))
    p = LAYERS[layer]
    top = 8192
    if wfmt == "fp8a16":  # a decode format: at most 32 routed rows per expert on average
        top = min(top, 32 * p["E"] // p["k"])
    T = int(round(math.exp(rng.uniform(0.0, math.log(top)))))
    return _case(layer, max(1, min(top, T)), wfmt, router=rng.random() < 0.3, out=rng.choice(["f32", "f32", "bf16"]))


# ------------------------------------------------------------------- inputs
def _gen(seed, sub, device):
    return torch.Generator(device=device).manual_seed((seed * 1000003 + sub) % (1 << 62))


def _routing(case, seed, device):
    """logits fp32 [T,E] (or the router's weights) and the selection bias."""
    p, T = LAYERS[case["layer"]], case["T"]
    E, H = p["E"], p["H"]
    gen = _gen(seed, 1, device)
    sel = None
    bias = torch.zeros(E, device=device)
    if p["bias"] == "normal":
        bias = torch.randn(E, generator=gen, device=device) * p["amount"]
    elif p["bias"] == "zipf":
        rank = torch.randperm(E, generator=gen, device=device) + 1
        bias = -p["amount"] * torch.log(rank.float())
    elif p["bias"] == "sel":
        sel = torch.randn(E, generator=gen, device=device) * p["amount"]
    if case["router"]:
        w = (torch.randn(E, H, generator=gen, device=device) / math.sqrt(H)).to(torch.bfloat16)
        return None, w, sel
    return torch.randn(T, E, generator=gen, device=device) + bias, None, sel


def _quantise(w, wfmt):
    """fp32 weights [n, N, K] in the storage of the format: (codes, scales)."""
    n, N, K = w.shape
    if wfmt == "bf16":
        return w.to(torch.bfloat16), None
    if wfmt in ("fp8", "fp8a16"):
        b = w.view(n, N // 128, 128, K // 128, 128)
        s = b.abs().amax(dim=(2, 4)).clamp_min(1e-10) / 448.0
        q = (b / s[:, :, None, :, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
        return q.view(torch.uint8).view(n, N, K), s
    if wfmt == "int4":
        b = w.view(n, N, K // 128, 128)
        s = (b.abs().amax(dim=3).clamp_min(1e-10) / 7.0).to(torch.bfloat16)
        q = (b / s.float()[..., None]).round_().clamp_(-8, 7).to(torch.int8).view(torch.uint8).view(n, N, K)
        q = (q & 15).view(n, N, K // 2, 2)
        return (q[..., 0] | (q[..., 1] << 4)).contiguous().view(torch.int32), s
    b = w.view(n, N, K // 32, 32)
    e = torch.floor(torch.log2(b.abs().amax(dim=3).clamp_min(1e-30))) - 2.0
    x = b / torch.exp2(e)[..., None]
    edges = torch.tensor([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0], device=w.device)
    q = torch.bucketize(x.abs(), edges, out_int32=True).to(torch.uint8) | ((x < 0).to(torch.uint8) << 3)
    q = q.view(n, N, K // 2, 2)
    return (q[..., 0] | (q[..., 1] << 4)).contiguous(), (e + 127.0).to(torch.uint8)


def _weights(case, seed, which, device):
    """All experts' stored weights of one product, made a few experts at a time."""
    p = LAYERS[case["layer"]]
    N, K = (2 * p["I"], p["H"]) if which == 1 else (p["H"], p["I"])
    gen = _gen(seed, 10 + which, device)
    per = max(1, (1 << 27) // (N * K))
    codes = scales = None
    for e in range(0, p["E"], per):
        n = min(per, p["E"] - e)
        w = torch.randn(n, N, K, generator=gen, device=device)
        c, s = _quantise(w.mul_(1.0 / math.sqrt(K)), case["wfmt"])
        if codes is None:
            codes = torch.empty((p["E"], *c.shape[1:]), dtype=c.dtype, device=device)
            scales = None if s is None else torch.empty((p["E"], *s.shape[1:]), dtype=s.dtype, device=device)
        codes[e:e + n] = c
        if s is not None:
            scales[e:e + n] = s
    return codes, scales


def _inputs(case, seed, device="cuda"):
    p, T = LAYERS[case["layer"]], case["T"]
    hidden = torch.randn(T, p["H"], generator=_gen(seed, 2, device), device=device).to(torch.bfloat16)
    logits, w_router, sel = _routing(case, seed, device)
    w1, s1 = _weights(case, seed, 1, device)
    w2, s2 = _weights(case, seed, 2, device)
    return dict(hidden=hidden, logits=logits, w_router=w_router, sel_bias=sel, w1=w1, w1_scale=s1, w2=w2, w2_scale=s2)


def prepare(case, seed):
    p, T = LAYERS[case["layer"]], case["T"]
    x = _inputs(case, seed)
    out = torch.empty(T, p["H"], dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device="cuda")
    ids = torch.empty(T, p["k"], dtype=torch.int32, device="cuda")
    wts = torch.empty(T, p["k"], dtype=torch.float32, device="cuda")
    logits_out = torch.empty(T, p["E"], dtype=torch.float32, device="cuda") if case["router"] else None
    kw = dict(mode=p["mode"], renormalize=True, routed_scale=p["scale"], wfmt=case["wfmt"], sel_bias=x["sel_bias"],
              w1_scale=x["w1_scale"], w2_scale=x["w2_scale"], out_dtype=case["out"], out=out, topk_ids_out=ids,
              topk_w_out=wts, w_router=x["w_router"], logits_out=logits_out)
    args = moe.make_args(T, p["H"], p["E"], p["I"], p["k"], mode=p["mode"], routed_scale=p["scale"],
                         wfmt=case["wfmt"], out_dtype=case["out"], w_router=x["w_router"])
    ws = torch.empty(max(moe.moe_workspace_bytes(args), 256), dtype=torch.uint8, device="cuda")
    return dict(x=x, k=p["k"], kw=kw, ws=ws)


def run(state):
    x, kw = state["x"], state["kw"]
    out, _ = moe.moe_forward(x["hidden"], x["logits"], x["w1"], x["w2"], state["k"], workspace=state["ws"], **kw)
    r = [out, kw["topk_ids_out"], kw["topk_w_out"]]
    return r if kw["logits_out"] is None else r + [kw["logits_out"]]


# ------------------------------------------------------- necessary work
@functools.lru_cache(maxsize=None)
def _active_experts(layer, T):
    """Experts that a batch reaches, from one draw of the layer's routing."""
    p = LAYERS[layer]
    logits, _, sel = _routing(dict(layer=layer, T=T, router=False), 0, "cpu")
    key = logits if p["mode"] == "softmax" else torch.sigmoid(logits) + (0.0 if sel is None else sel)
    return int(torch.topk(key, p["k"], dim=1).indices.unique().numel())


def work(case):
    p, T = LAYERS[case["layer"]], case["T"]
    H, E, I, k = p["H"], p["E"], p["I"], p["k"]
    per_expert = 3 * H * I * WEIGHT_BYTES[case["wfmt"]]
    nbytes = _active_experts(case["layer"], T) * per_expert
    nbytes += T * H * (2 + (4 if case["out"] == "f32" else 2)) + T * E * 4 + T * k * 8
    flops = 6 * T * k * H * I
    if case["router"]:
        nbytes += E * H * 2
        flops += 2 * T * E * H
    return {"bytes": int(nbytes), "flops": int(flops)}


# Largest relative errors (2-norm) of a correct implementation at each format's
# precision, about four times what the layer shows against `exact`: the
# bf16-activation formats differ by roundings of the intermediate that a
# different order of fp32 sums tips (5e-5), the tiled int4 route by bf16
# weights in its second product (1.4e-3), the e4m3-activation formats by their
# 16-bit rows before the weighted sum and by tipped codes (2.6e-3); a bf16
# output by its own rounding (1.7e-3).
REL = {"bf16": 2e-4, "fp8a16": 2e-4, "mxfp4": 2e-4, "int4": 6e-3, "fp8": 1e-2, "mxfp4x8": 1e-2}


def tolerance(case):
    t = {"rel": max(REL[case["wfmt"]], 7e-3 if case["out"] == "bf16" else 0.0)}
    if case["router"]:  # fp32 logits can tip a near tie of two experts
        t["differ"] = 1e-3
    return t


# ---------------------------------------------------------------- 64 bits
E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, -0.0, -0.5, -1.0, -1.5, -2.0, -3.0, -4.0, -6.0]


def _decode(codes, scales, wfmt):
    """One expert's stored weights [N, ...] as fp64 [N, K]."""
    if wfmt == "bf16":
        return codes.double()
    if wfmt in ("fp8", "fp8a16"):
        w = codes.view(torch.float8_e4m3fn).float().double()
        return w * scales.double().repeat_interleave(128, 0).repeat_interleave(128, 1)
    b = codes.view(torch.uint8)
    q = torch.stack((b & 15, b >> 4), dim=-1).view(b.shape[0], -1).long()
    if wfmt == "int4":
        v = torch.where(q >= 8, q - 16, q).double()
        return v * scales.double().repeat_interleave(128, 1)
    v = torch.tensor(E2M1, dtype=torch.float64, device=b.device)[q]
    return v * torch.exp2(scales.double() - 127.0).repeat_interleave(32, 1)


def _quant_rows(a, wfmt):
    """Activations as the format's products take them, in fp64.  The fp8 scale
    and quotient are fp32 by the format's definition (many bf16 values lie on
    exact ties there); the MXFP8 ones are powers of two."""
    if wfmt == "fp8":
        g = a.view(a.shape[0], -1, 128).float()
        amax = g.abs().amax(dim=2, keepdim=True).clamp_min(1e-10)
        s = amax / torch.full_like(amax, 448.0)
    elif wfmt == "mxfp4x8":
        g = a.view(a.shape[0], -1, 32)
        s = torch.exp2((torch.floor(torch.log2(g.abs().amax(dim=2, keepdim=True))) - 8.0).clamp_min(-127.0))
    else:
        return a.to(torch.bfloat16).double()
    q = (g / s).clamp(-448.0, 448.0).float().to(torch.float8_e4m3fn).float().double()
    return (q * s.double()).view(a.shape)


def exact(case, seed):
    p, T, wfmt = LAYERS[case["layer"]], case["T"], case["wfmt"]
    x = _inputs(case, seed)
    hidden = x["hidden"].double()
    logits = hidden @ x["w_router"].double().t() if case["router"] else x["logits"].double()
    score = logits if p["mode"] == "softmax" else torch.sigmoid(logits)
    key = score if x["sel_bias"] is None else score + x["sel_bias"].double()
    ids = torch.sort(key, dim=1, descending=True, stable=True).indices[:, :p["k"]]
    sel = score.gather(1, ids)
    wts = (torch.softmax(sel, 1) if p["mode"] == "softmax" else sel / sel.sum(1, keepdim=True)) * p["scale"]
    out = torch.zeros(T, p["H"], dtype=torch.float64, device=hidden.device)
    xq = _quant_rows(hidden, wfmt)
    for e in range(p["E"]):
        t, j = torch.nonzero(ids == e, as_tuple=True)
        if t.numel() == 0:
            continue
        s1 = None if x["w1_scale"] is None else x["w1_scale"][e]
        s2 = None if x["w2_scale"] is None else x["w2_scale"][e]
        g = xq[t] @ _decode(x["w1"][e], s1, wfmt).t()
        a = torch.nn.functional.silu(g[:, :p["I"]]) * g[:, p["I"]:]
        y = _quant_rows(a, wfmt) @ _decode(x["w2"][e], s2, wfmt).t()
        out.index_add_(0, t, y * wts[t, j][:, None])
    r = [out, ids.to(torch.int32), wts]
    return r + [logits] if case["router"] else r
