"""The work a user of the routed-LoRA layers has them do, as cases that can be timed.

Four kinds of case, each through the Python face of the C ABI with every buffer the caller would keep (weights,
pointer tables, workspaces, outputs) made beforehand:

  decode   one `milora_layer_decode` step of B requests through a layer's seven routed linears
  route    one `milora_route` call over the prompts of B requests
  linears  the seven `milora_routed_linear` calls of one layer for M rows: a prefill (row-major weights, rows mapped to
           requests prompt by prompt), beams of a decode step (packed weights), or plain fp32 layers

Sizes are those of `synth.CONFIGS` (LLaMA-2 7B and 13B layers, the fp32 toy layer), of the tests and of the benchmark,
or generic ones of the same ranges.
"""
import dataclasses

import torch

from paper_2410_18035_amd import binding as mb
from paper_2410_18035_amd import synth

DEV = "cuda:0"
SITES = range(mb.NUM_SITES)
# Coefficients of the rational router activation (a trained set is about this size).
RATIONAL = [0.1, 1.0, 0.3, -0.2, 0.05, 0.01, -0.003, 0.5, -0.25, 0.1, 0.02, -0.01]


def _decode(name, B, d, F, ranks, **kw):
    c = dict(kind="decode", B=B, d=d, F=F, ranks=ranks, T=B, dtype="bf16", packed=True, rmsnorm=False, attn=False,
             noalloc=False, top_k=1, up_down_skew=False)
    c.update(kw)
    return dict(c, name=name) if name else c


def _route(name, B, lo, hi, d, **kw):
    c = dict(kind="route", B=B, lo=lo, hi=hi, pad=0, d=d, T=B, dtype="bf16", pool="mean", act="gelu", top_k=1)
    c.update(kw)
    return dict(c, name=name) if name else c


def _linears(name, M, B, d, F, ranks, **kw):
    c = dict(kind="linears", M=M, B=B, d=d, F=F, ranks=ranks, T=B, dtype="bf16", packed=False, beams=False, bias=False,
             top_k=1)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call there is: a decode step of the fp32 toy layer, bound by launches and the host
        _decode("decode_toy_f32_b4", 4, 256, 688, "8", dtype="f32", packed=False),
        # one interactive user on a 7B layer: the time of a token is the time of the weights' stream
        _decode("decode_7b_b1", 1, 4096, 11008, "32"),
        # the benchmark's step: 32 tenants' requests, a 7B layer
        _decode("decode_7b_b32", 32, 4096, 11008, "32"),
        # a layer of the 64-request stack (RMS norm in front, tenants drawn with replacement)
        _decode("decode_7b_b64_norm", 64, 4096, 11008, "32", rmsnorm=True),
        # a layer of the 13B stack at the largest batch: mixed ranks, most requests routed to up and down
        _decode("decode_13b_b128_norm", 128, 5120, 13824, "8,16,64", rmsnorm=True, up_down_skew=True),
        # the benchmark's router call: 32 prompts of 256 tokens
        _route("route_7b_32x256_mean", 32, 256, 256, 4096),
        # the prefill configuration's prompts under the self-attention pooler and the learned activation, three sites each
        _route("route_7b_16x2048_selfattn", 16, 1024, 2048, 4096, pad=2048, pool="selfattn", act="rational", top_k=3),
        # time to first token of one short chat prompt
        _linears("prefill_7b_m45", 45, 1, 4096, 11008, "32"),
        # a few prompts of ordinary length prefilled together, ragged to the row
        _linears("prefill_7b_m777", 777, 5, 4096, 11008, "8,16,64"),
        # the benchmark's prefill: 16 prompts padded to 2048 rows
        _linears("prefill_7b_m32768", 32768, 16, 4096, 11008, "32"),
        # beam search with four beams on the decode weights: rows share requests, three sites per request
        _linears("beams_7b_m96_packed", 96, 24, 4096, 11008, "16", packed=True, beams=True, bias=True, top_k=3),
        # fp32 layers of sizes that are multiples of nothing (the any-shape path): validation runs, small models
        _linears("linears_f32_m300", 300, 6, 1000, 2730, "8,20", dtype="f32", bias=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _width(rng, unit):
    """(d, F) of a layer: the two LLaMA-2 sizes, or a width of its own with F near 2.7 d, multiples of `unit`."""
    if rng.random() < 0.5:
        return rng.choice([(4096, 11008), (5120, 13824)])
    d = unit * _log_int(rng, 1024 // unit, 5120 // unit)
    return d, unit * int(round(d * rng.uniform(2.3, 3.2) / unit))


def draw(rng):
    u = rng.random()
    ranks = rng.choice(["8", "16", "32", "64", "8,16,64", "5,12,16"])
    top_k = rng.choice([1, 1, 1, 2, 3])
    if u < 0.35:
        B = _log_int(rng, 1, 128)
        d, F = _width(rng, 32)
        return _decode(None, B, d, F, ranks, T=rng.randint((B + 1) // 2, B), rmsnorm=rng.random() < 0.5,
                       attn=rng.random() < 0.3, noalloc=B <= 32 and rng.random() < 0.25, top_k=top_k,
                       up_down_skew=rng.random() < 0.3)
    if u < 0.40:
        d = 8 * rng.randint(16, 64)
        return _decode(None, rng.randint(1, 16), d, 8 * int(d * 2.7 / 8), rng.choice(["4", "8"]), dtype="f32", packed=False)
    if u < 0.60:
        B = _log_int(rng, 1, 64)
        hi = _log_int(rng, 16, 2048)
        lo = rng.choice([hi, (hi + 1) // 2, max(1, hi // 8)])
        return _route(None, B, lo, hi, rng.choice([2048, 4096, 5120, 8 * rng.randint(100, 640)]),
                      pad=hi if rng.random() < 0.3 else 0, T=rng.randint((B + 1) // 2, B),
                      dtype=rng.choice(["bf16"] * 5 + ["f32"]), pool=rng.choice(["mean", "last", "max", "selfattn"]),
                      act=rng.choice(["identity", "tanh", "relu", "gelu", "rational"]), top_k=top_k)
    if u < 0.82:
        d, F = _width(rng, 64)
        M = _log_int(rng, 16, 32768)
        M = min(M, 32768 * 202_375_168 // (4 * d * d + 3 * d * F))
        return _linears(None, M, min(M, _log_int(rng, 1, 16)), d, F, ranks, bias=rng.random() < 0.2, top_k=top_k)
    if u < 0.92:
        d, F = _width(rng, 32)
        beams = rng.choice([1, 2, 4, 5])
        B = _log_int(rng, 1, 300 // beams)
        return _linears(None, B * beams, B, d, F, ranks, packed=True, beams=True, bias=rng.random() < 0.3, top_k=top_k)
    d = rng.randint(128, 1280)
    M = _log_int(rng, 8, 1000)
    return _linears(None, M, min(M, rng.randint(1, 8)), d, int(d * rng.uniform(2.3, 3.2)), rng.choice(["8", "3,8,17", "32"]),
                    dtype=rng.choice(["f32", "f32", "bf16"]), bias=rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------------- inputs
def _workload(case, seed):
    """The seeded draw behind a case.  Scales as in the serving configurations: about unit gain per linear and a
    low-rank term of the order of the base term."""
    d = case["d"]
    ranks = tuple(int(r) for r in case.get("ranks", "8").split(","))
    sigma_w = 0.02 * (4096 / d) ** 0.5
    return synth.Workload("case", case["dtype"], d, case.get("F", d), 1, case["T"], case["B"], ranks,
                          (case.get("lo", 1), case.get("hi", 1)), pad_to=case.get("pad", 0),
                          tenants="identity" if case["T"] == case["B"] else "uniform",
                          route_skew=(0.08, 0.08, 0.08, 0.08, 0.08, 0.30, 0.30) if case.get("up_down_skew") else None,
                          seed=int(seed) % 100_000, sigma_w=sigma_w,
                          sigma_lora=(sigma_w / (sum(ranks) / len(ranks)) ** 0.5) ** 0.5)


def _routes(wl, top_k):
    """Route bytes of the B requests: one site each, or sets of top_k sites."""
    if top_k == 1:
        return synth.constructed_routes(wl)[0]
    g = torch.Generator().manual_seed(wl.seed * 7 + 3)
    sets = torch.rand(wl.B, mb.NUM_SITES, generator=g).argsort(dim=1)[:, :top_k]
    return (mb.ROUTE_SET | (1 << sets).sum(1)).to(torch.uint8)


def _layer(case, wl):
    """Weights in the layout the case uses, and the pointer table of the tenants' adapters."""
    W = synth.base_weights(wl, 0, DEV)
    if case["packed"]:
        W = [mb.milora_pack_weight(w) for w in W]
    ad = synth.adapters(wl, 0, DEV)
    return W, mb.AdapterTable.from_tensors(ad.A, ad.B, ad.rank)


def _zeros(nbytes):
    return torch.zeros(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    wl = _workload(case, seed)
    tid = synth.tenant_ids(wl).to(DEV)
    dt = wl.torch_dtype
    if case["kind"] == "route":
        H, ss, sl = synth.prompts(wl, 0, DEV)
        selfattn = case["pool"] == "selfattn"
        return dict(case=case, H=H, ss=ss.to(DEV), sl=sl.to(DEV), tid=tid, Wr=synth.router_weights(wl, 0, DEV),
                    w_sa=synth.selfattn_query(wl, 0, DEV) if selfattn else None,
                    coef=RATIONAL if case["act"] == "rational" else None,
                    route=torch.empty(wl.B, dtype=torch.uint8, device=DEV),
                    ws=_zeros(mb.route_workspace_bytes(wl.B, wl.d, H.shape[0])))
    W, tab = _layer(case, wl)
    route = _routes(wl, case["top_k"]).to(DEV)
    st = dict(case=case, W=W, tab=tab, tid=tid, route=route)
    if case["kind"] == "decode":
        st.update(x=synth.decode_input(wl, 0, DEV), y=torch.empty(wl.B, wl.d, dtype=dt, device=DEV),
                  qkv=torch.empty(wl.B, 3 * wl.d, dtype=dt, device=DEV),
                  attn=synth.decode_input(wl, 1, DEV) if case["attn"] else None,
                  ws=None if case["noalloc"] else _zeros(mb.layer_decode_workspace_bytes(wl.B, wl.d, wl.F, tab.r_max)))
        return st
    M, B = case["M"], case["B"]
    if case["beams"]:
        r2r = torch.arange(M) // (M // B)
    else:  # prompts of uneven length, one after the other
        g = torch.Generator().manual_seed(wl.seed * 13 + 5)
        ends = torch.cumsum(torch.rand(B, generator=g) + 0.5, 0)
        r2r = torch.bucketize(torch.arange(M).double() / M * ends[-1].double(), ends.double(), right=True).clamp_(max=B - 1)
    gx = torch.Generator(device=DEV).manual_seed(wl.seed * 17 + 7)
    rows = lambda n: torch.empty(M, n, dtype=torch.float32, device=DEV).normal_(0, 1, generator=gx).to(dt)
    dims = [synth.site_dims(m, wl.d, wl.F) for m in SITES]
    st.update(x=rows(wl.d), xF=rows(wl.F), r2r=r2r.to(torch.int32).to(DEV), dims=dims,
              bias=[torch.empty(n, device=DEV).normal_(0, 0.1, generator=gx).to(dt) if case["bias"] else None for _, n in dims],
              out=[torch.empty(M, n, dtype=dt, device=DEV) for _, n in dims])
    # one workspace per weight shape (packed launches keep their hand-over flags in it)
    ws = {s: _zeros(mb.routed_linear_workspace_bytes(M, s[0], s[1], tab.r_max)) for s in set(dims)}
    st["ws"] = [ws[s] for s in dims]
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "route":
        return mb.milora_route(st["H"], st["ss"], st["sl"], st["tid"], st["Wr"], case["pool"], case["act"],
                               route_out=st["route"], workspace=st["ws"], w_sa=st["w_sa"], act_coef=st["coef"],
                               top_k=case["top_k"])
    layout = mb.W_PACKED if case["packed"] else mb.W_ROWMAJOR
    if case["kind"] == "decode":
        if case["noalloc"]:
            mb.milora_layer_decode_noalloc(st["x"], st["W"], st["tab"], st["tid"], st["route"], case["F"], st["y"],
                                           st["qkv"], rmsnorm=case["rmsnorm"], attn_out=st["attn"])
            return st["y"], st["qkv"]
        return mb.milora_layer_decode(st["x"], st["W"], st["tab"], st["tid"], st["route"], case["F"], w_layout=layout,
                                      rmsnorm=case["rmsnorm"], attn_out=st["attn"], y=st["y"], qkv_out=st["qkv"],
                                      workspace=st["ws"])
    return [mb.milora_routed_linear(st["xF"] if m == 6 else st["x"], st["W"][m], st["tab"], m, st["tid"], st["route"],
                                    row_to_req=st["r2r"], bias=st["bias"][m], w_layout=layout, d2=st["dims"][m][1],
                                    out=st["out"][m], workspace=st["ws"][m]) for m in SITES]


# ------------------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    s = 2 if case["dtype"] == "bf16" else 4
    d, B = case["d"], case["B"]
    if case["kind"] == "route":
        tokens = B * (1 if case["pool"] == "last" else (case["lo"] + case["hi"]) / 2)
        extra = d if case["pool"] == "selfattn" else 0
        return {"bytes": tokens * d * s + case["T"] * (7 * d + extra) * s + B * 29,
                "flops": tokens * d * (4 if extra else 1) + 14.0 * B * d}
    F = case["F"]
    P = 4 * d * d + 3 * d * F
    ranks = [int(r) for r in case["ranks"].split(",")]
    r = sum(ranks) / len(ranks)
    share = [0.08] * 5 + [0.30, 0.30] if case.get("up_down_skew") else [1 / 7] * 7
    dims = [synth.site_dims(m, d, F) for m in SITES]
    # low-rank pairs that some request uses, per request and per distinct tenant (mean over the draws)
    lora_row = case["top_k"] * sum(q * r * (a + b) for q, (a, b) in zip(share, dims))
    seen = 1 if case["T"] == B else (1 - (1 - 1 / case["T"]) ** B) * case["T"] / B
    M = case.get("M", B)
    act = 4 * d + F if case["kind"] == "decode" else sum(a + b for a, b in dims) - 5 * d  # in and out, x of six sites once
    if case["kind"] == "decode":
        act = 5 * d + (d if case["attn"] else 0)  # x, y, q, k, v
    return {"bytes": P * s + B * seen * lora_row * s + M * act * s, "flops": 2.0 * M * P + 2.0 * M * lora_row}


def tolerance(case):
    """About four times the distance of the results from the same path in 64 bits, the largest seen over these ranges:
    route logits rel 2.2e-7, max 4.5e-7; fp32 outputs 1.1e-6, 7.6e-6 (sums of up to a few thousand terms); bf16 linears
    1.7e-3, 3.9e-3 (one rounding); bf16 decode steps 4.4e-3, 2.4e-2 (four roundings in a chain)."""
    if case["kind"] == "route":
        return {"rel": 1e-6, "max": 2e-6, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 4.5e-6, "max": 3e-5}
    if case["kind"] == "linears":
        return {"rel": 6.6e-3, "max": 1.6e-2}
    return {"rel": 1.6e-2, "max": 9e-2}
