"""Performance cases of the MoE layer: what a user of this library has it do, through its
public entry points, from one decode step of a few sequences to the large combined
batch, in each data type.

A case is a dict of plain values:

    kind     "layer"     one whole layer step: MoELayer.run / MoELayerMXFP8.run
             "gate"      moe_router_topk: router GEMM and top-k from hidden states
             "dispatch"  moe_route, moe_permute with the row copy, moe_combine: the
                         steps around a caller's own expert computation
    dtype    "bf16", "f32" or "mxfp8" (layer); "bf16" elsewhere
    T, H, E, k           tokens, hidden size, experts, experts per token
    F, Fs                FFN size of the routed experts and of the shared one (0: none)
    skew     spread of the experts' popularity: popularity ~ lognormal(0, skew)
    gather   the layer's path: GEMM-1 reads token rows through the map, or x_perm
    renorm   gate weights normalised over the selected experts (1) or over all (0)

Every input is drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math

import torch

import paper_2606_21712_amd as moe

DEV = "cuda"


# --------------------------------------------------------------------------- the cases
def _case(name, kind, dtype, T, H, E, k, F=0, Fs=0, skew=0.0, gather=True, renorm=1):
    c = dict(name=name, kind=kind, dtype=dtype, T=T, H=H, E=E, k=k, F=F, Fs=Fs, skew=skew, gather=gather,
             renorm=renorm)
    return c if name else {f: v for f, v in c.items() if f != "name"}


def listed():
    return [
        # The smallest call: the tiny fp32 layer, where launches and latency are all there is.
        _case("f32_tiny", "layer", "f32", 256, 256, 8, 2, 512, gather=False),
        # An fp32 layer of some size: the run in full precision that a bf16 one is checked against.
        _case("f32_check", "layer", "f32", 2000, 1024, 8, 2, 2048),
        # Decoding with two dozen sequences on the Mixtral shape: the experts' weights are
        # read for a handful of rows each.
        _case("mixtral_decode24", "layer", "bf16", 24, 4096, 8, 2, 14336),
        # A short ragged batch on the Mixtral shape through the default (x_perm) path.
        _case("mixtral_509", "layer", "bf16", 509, 4096, 8, 2, 14336, gather=False),
        # Prefill of 4096 tokens, Mixtral shape.
        _case("mixtral_4k", "layer", "bf16", 4096, 4096, 8, 2, 14336),
        # Decoding on the fine-grained DeepSeek shape with its shared expert: 64 experts with
        # about a dozen rows each.
        _case("deepseek_decode96", "layer", "bf16", 96, 7168, 64, 8, 2048, 2048),
        # The DeepSeek shape at the batch that fills its experts.
        _case("deepseek_16k", "layer", "bf16", 16384, 7168, 64, 8, 2048, 2048),
        # The largest call: the memory-constrained combined batch, uneven expert loads.
        _case("memconstrained_128k", "layer", "bf16", 131072, 4096, 64, 4, 4096, skew=1.0),
        # MXFP8 expert GEMMs: a decode batch and a large uneven one.
        _case("mxfp8_deepseek_200", "layer", "mxfp8", 200, 7168, 64, 8, 2048, 2048),
        _case("mxfp8_memconstrained_32k", "layer", "mxfp8", 32768, 4096, 64, 4, 4096, skew=1.0),
        # The gate from hidden states: router GEMM and top-k.
        _case("gate_16k", "gate", "bf16", 16384, 7168, 64, 8, renorm=0),
        # Routing, grouping with the row copy, and combining, around a caller's own experts.
        _case("dispatch_32k", "dispatch", "bf16", 32768, 4096, 64, 4, skew=1.0),
    ]


# (H, E, k, F, Fs) of the repository's workloads
_SHAPES = [(4096, 8, 2, 14336, 0), (7168, 64, 8, 2048, 2048), (4096, 64, 4, 4096, 0)]

_MAX_FLOPS = 5.2e13            # of one layer pass: no more than the largest listed case
_MAX_WEIGHT_BYTES = 7.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["layer", "gate", "dispatch"], [8, 1, 1])[0]
    skew = rng.choice([0.0, 0.5, 1.0])
    renorm = rng.choice([1, 1, 0])
    if kind == "gate":
        return _case("", "gate", "bf16", _log_int(rng, 16, 131072), 64 * rng.randint(16, 112), rng.randint(4, 64),
                     rng.randint(1, 4), renorm=renorm)
    if kind == "dispatch":
        H = 64 * rng.randint(16, 112)
        return _case("", "dispatch", "bf16", _log_int(rng, 16, 65536 * 4096 // H), H, rng.choice([8, 16, 60, 64, 256]),
                     rng.randint(1, 8), skew=skew, renorm=renorm)
    dtype = rng.choices(["bf16", "mxfp8", "f32"], [4, 3, 1])[0]
    gather = rng.random() < 0.75
    if dtype == "f32":
        E = rng.choice([4, 8, 16])
        return _case("", "layer", "f32", _log_int(rng, 16, 4096), 64 * rng.randint(4, 24), E, rng.randint(1, 3),
                     64 * rng.randint(4, 40), skew=skew, gather=gather, renorm=renorm)
    while True:
        if rng.random() < 0.5:
            H, E, k, F, Fs = rng.choice(_SHAPES)
        else:
            step = 128 if dtype == "mxfp8" else 64
            H = step * rng.randint(1024 // step, 7168 // step)
            F = step * _log_int(rng, 512 // step, 14336 // step)
            E = rng.choice([4, 8, 16, 32, 60, 64, 128])
            k = rng.randint(1, min(8, E // 2))
            Fs = rng.choice([0, 0, F])
        T = _log_int(rng, 4, 65536)
        weights = 3 * H * (E * F + Fs) * (1 if dtype == "mxfp8" else 2)
        if weights <= _MAX_WEIGHT_BYTES and 6 * H * T * (k * F + Fs) <= _MAX_FLOPS:
            return _case("", "layer", dtype, T, H, E, k, F, Fs, skew, gather, renorm)


# --------------------------------------------------------------------------- inputs
def _inputs(c, seed):
    """The tensors a caller holds, from the seed alone.  x ~ N(0, 1) (normalised hidden
    states), weights ~ N(0, 1 / fan-in); logits are the experts' log popularity plus
    Gumbel noise, so that expert loads follow the popularity."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    T, H, E, k, F, Fs = (c[f] for f in ("T", "H", "E", "k", "F", "Fs"))
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16

    def normal(*shape, std=1.0):
        t = torch.empty(shape, dtype=dt, device=DEV)
        return t.normal_(0.0, std, generator=g)

    d = dict(x=normal(T, H))
    if c["kind"] == "gate":
        d["w_router"] = normal(E, H, std=H ** -0.5)
        return d
    pop = torch.empty(E, device=DEV).normal_(0.0, 1.0, generator=g) * c["skew"]
    u = torch.empty((T, E), device=DEV).exponential_(generator=g)
    d["logits"] = pop - u.clamp_min_(1e-30).log_()
    if c["kind"] == "dispatch":
        d["y_perm"] = normal(T * k, H)
        return d
    d["w"] = [normal(E, F, H, std=H ** -0.5), normal(E, F, H, std=H ** -0.5), normal(E, H, F, std=F ** -0.5)]
    d["ws"] = [normal(1, Fs, H, std=H ** -0.5), normal(1, Fs, H, std=H ** -0.5),
               normal(1, H, Fs, std=Fs ** -0.5)] if Fs else []
    return d


def prepare(case, seed):
    c = case
    d = _inputs(c, seed)
    T, H, E, k = (c[f] for f in ("T", "H", "E", "k"))
    i32 = dict(dtype=torch.int32, device=DEV)
    if c["kind"] == "gate":
        return dict(case=c, x=d["x"], w=d["w_router"], ids=torch.empty((T, k), **i32),
                    weights=torch.empty((T, k), dtype=torch.float32, device=DEV))
    if c["kind"] == "dispatch":
        out = dict(counts=torch.empty(E, **i32), offsets=torch.empty(E + 1, **i32),
                   sorted_token_ids=torch.empty(T * k, **i32), dest_rows=torch.empty((T, k), **i32),
                   x_perm=torch.empty((T * k, H), dtype=d["x"].dtype, device=DEV))
        ws = torch.empty(max(1, moe.moe_permute_workspace_bytes(T, E, k)), dtype=torch.uint8, device=DEV)
        return dict(case=c, x=d["x"], logits=d["logits"], y_perm=d["y_perm"], out=out, ws=ws,
                    y=torch.empty_like(d["x"]), ids=torch.empty((T, k), **i32),
                    weights=torch.empty((T, k), dtype=torch.float32, device=DEV))
    if c["dtype"] == "mxfp8":
        layer = moe.MoELayerMXFP8(T, H, E, k, c["F"], c["Fs"], device=DEV, gather=c["gather"])
        w = [moe.quantize_weights_mxfp8(t) for t in d["w"] + d["ws"]]
    else:
        layer = moe.MoELayer(T, H, E, k, c["F"], c["Fs"], dtype=d["x"].dtype, device=DEV, gather=c["gather"])
        w = d["w"] + d["ws"]
    return dict(case=c, layer=layer, x=d["x"], logits=d["logits"], w=w)


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "layer":
        layer = s["layer"]
        y = layer.run(s["x"], s["logits"], *s["w"], renormalize=c["renorm"])
        return dict(y=y, ids=layer.topk_ids, weights=layer.topk_weights)
    if c["kind"] == "gate":
        moe.moe_router_topk(s["x"], s["w"], c["k"], c["renorm"], topk_ids=s["ids"], topk_weights=s["weights"])
        return dict(ids=s["ids"], weights=s["weights"])
    moe.moe_route(s["logits"], c["k"], c["renorm"], s["ids"], s["weights"])
    out = moe.moe_permute(s["ids"], s["x"], c["E"], out=s["out"], ws=s["ws"])
    y = moe.moe_combine(s["y_perm"], out["dest_rows"], s["weights"], y=s["y"])
    return dict(y=y, ids=s["ids"], weights=s["weights"], x_perm=out["x_perm"], counts=out["counts"],
                sorted_token_ids=out["sorted_token_ids"], dest_rows=out["dest_rows"])


# --------------------------------------------------------------------------- what a pass needs
def work(case):
    c = case
    T, H, E, k, F, Fs = (c[f] for f in ("T", "H", "E", "k", "F", "Fs"))
    R = T * k
    b = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "gate":
        return dict(bytes=T * H * b + E * H * b + R * 8, flops=2 * T * H * E)
    if c["kind"] == "dispatch":
        return dict(bytes=T * E * 4 + R * 16 + (T + R) * H * b + (R + T) * H * b, flops=2 * R * H)
    # experts that see a token, when T tokens each pick k of E
    active = E * (1.0 - (1.0 - k / E) ** T)
    per = 3 * H * F
    wb = (per * active + 3 * H * Fs) * (33 / 32 if c["dtype"] == "mxfp8" else b)
    return dict(bytes=wb + 2 * T * H * b + T * E * 4 + R * 8, flops=6 * H * F * R + 6 * H * Fs * T)


def tolerance(case):
    """About four times the error against exact() (measured: fp32 y 0.6-1.2e-6, bf16 and MXFP8 y
    2.5-2.9e-3, gate weights 3e-7, combine alone one bf16 rounding)."""
    c = case
    if c["kind"] == "gate":
        # fp32 sums of bf16 products: the selection may differ where two logits tie to fp32 rounding
        return dict(rel=4e-6, max=4e-4, differ=1e-3)
    if c["kind"] == "dispatch":
        # fp32 sums of at most 8 rows, rounded to bf16 once: another order moves few roundings
        return dict(rel=1e-4, max=2e-2, differ=0.0)
    if c["dtype"] == "f32":
        return dict(rel=6e-6, max=1e-4, differ=0.0)
    return dict(rel=1.2e-2, max=1e-1, differ=0.0)


# --------------------------------------------------------------------------- 64-bit values
def _mx(v):
    """v (float64 [..., K]) as MXFP8 represents it: per 32 elements one power-of-two scale,
    E4M3 elements rounded to nearest even, clamped to +-448."""
    b = v.reshape(-1, 32)
    amax = b.abs().amax(1, keepdim=True)
    e = torch.frexp(amax)[1].to(torch.float64) - 1.0          # floor(log2 amax)
    e = torch.where(amax > 0, (e - 8.0).clamp(-127.0, 127.0), torch.full_like(e, -127.0))
    s = torch.exp2(e)
    q = b / s
    step = torch.exp2((torch.frexp(q)[1].to(torch.float64) - 1.0).clamp_min(-6.0) - 3.0)
    q = (torch.round(q / step) * step).clamp(-448.0, 448.0)
    return (q * s).reshape(v.shape)


def _ffn64(x, wg, wu, wd, mx):
    """SwiGLU FFN in 64 bits; mx: on the values that the MXFP8 path computes with."""
    z = _mx if mx else (lambda t: t)
    g = x @ z(wg.double()).T
    u = x @ z(wu.double()).T
    h = z(g * torch.sigmoid(g) * u)
    return h @ z(wd.double()).T


def _route64(logits, k, renorm):
    p = torch.softmax(logits.double(), 1)
    top, ids = torch.topk(logits, k, 1)
    w = p.gather(1, ids)
    return ids, w / w.sum(1, keepdim=True) if renorm else w


def exact(case, seed):
    c = case
    d = _inputs(c, seed)
    k, mx = c["k"], c["dtype"] == "mxfp8"
    if c["kind"] == "gate":
        logits = d["x"].double() @ d["w_router"].double().T
        return dict(ids=None, weights=_route64(logits, k, c["renorm"])[1])
    ids, w = _route64(d["logits"], k, c["renorm"])
    if c["kind"] == "dispatch":
        order = torch.sort(ids.reshape(-1), stable=True)[1]
        dest = torch.empty_like(order)
        dest[order] = torch.arange(order.numel(), device=DEV)
        dest = dest.reshape(ids.shape)
        y = sum(w[:, j:j + 1] * d["y_perm"][dest[:, j]].double() for j in range(k))
        return dict(y=y, ids=None, weights=w, x_perm=d["x"][order // k].double(), counts=None, sorted_token_ids=None,
                    dest_rows=None)
    x = d["x"].double()
    if mx:
        x = _mx(x)
    y = _ffn64(x, *(t[0] for t in d["ws"]), mx) if c["Fs"] else torch.zeros_like(x)
    for e in range(c["E"]):
        tok, slot = torch.nonzero(ids == e, as_tuple=True)
        if tok.numel():
            y.index_add_(0, tok, w[tok, slot, None] * _ffn64(x[tok], *(t[e] for t in d["w"]), mx))
    return dict(y=y, ids=None, weights=w)
