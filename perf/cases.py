"""The calls whose speed matters to a user of this package, over the sizes such users have.

A case is a dict of plain values; its ``kind`` names the public entry points it goes through:

  step     ``GroupStep.run``: pack, shared backbone, per-tenant heads forward + backward, unpack
  infer    ``InferStep.replay`` / ``launch``: the resident decode-only step of the inference queue
  layer    ``jn_backbone_forward``: layers of the frozen backbone over a packed batch
  heads    ``jn_tenant_heads_fwd_bwd``: pooling, MLP heads forward, loss, weight gradients
  experts  ``jn_tenant_experts_fwd_bwd``: action experts forward, loss, weight gradients
  adamw    ``jn_tenant_adamw_step``: per-tenant optimizer step
  pack     ``jn_pack_group`` and ``jn_unpack``: requests to the physical batch and back

Lengths and tenant sizes of a case follow from its own numbers (``shape_seed``), values from the seed that
``prepare`` gets. ``exact`` evaluates the same definitions in float64 torch, one sample and one tenant at a time.
"""
from __future__ import annotations

import functools
import math
from types import SimpleNamespace
from typing import Dict, List

import numpy as np
import torch

import paper_2607_16074_amd as jn
from paper_2607_16074_amd import step as jstep

DEV = "cuda"
EPS = 1e-6
SIG = 0x4A4E5056_4C414631
F64 = torch.float64

# Backbones of the repository's workloads: the tiny one of the end-to-end check, the 12-layer base one, and the
# 2B-shaped one with its multi-query and grouped-query variants.
_BACKBONES = {
    "tiny": dict(d=128, heads=4, ffn=512, glu=False, kv=0, causal=False, rope=0.0),
    "base": dict(d=768, heads=12, ffn=3072, glu=False, kv=0, causal=False, rope=0.0),
    "2b": dict(d=2048, heads=8, ffn=16384, glu=True, kv=0, causal=False, rope=0.0),
    "2b_mqa": dict(d=2048, heads=8, ffn=16384, glu=True, kv=1, causal=False, rope=10000.0),
    "2b_gqa": dict(d=2048, heads=16, ffn=16384, glu=True, kv=2, causal=True, rope=1000000.0),
}
# (action_dim, chunk) of the tenants, cycled over a group
_SCHEMAS = ((7, 1), (7, 10), (7, 50), (14, 1), (14, 10), (14, 50), (32, 10), (32, 50))
# an action expert's width, heads and MLP width; action tokens per sample
_EXPERT = dict(d=1024, heads=8, ffn=4096, chunk=50)
_D_TIME = 1024


# ------------------------------------------------------------------ cases ---


def listed() -> List[dict]:
    return [
        # The smallest training step a user runs (the end-to-end check's two tenants x eight short samples): bound
        # by launches and the calls' own host work.
        dict(name="step_tiny_2x8", kind="step", bb="tiny", layers=2, tenants=2, samples=16, len_lo=20, len_hi=32,
             skew=0.0, hidden=256, hidden_layers=1, align=1, shape_seed=1),
        # Serving one robot: one observation through the whole 2B-shaped model, replayed as a captured graph.
        dict(name="infer_2b_1x1", kind="infer", bb="2b", layers=18, tenants=1, samples=1, len_lo=272, len_hi=320,
             skew=0.0, hidden=1024, hidden_layers=2, align=1, graph=True, shape_seed=2),
        # A layer of the same model for the batch that the inference queue collects from eight tenants.
        dict(name="layer_2b_8x1", kind="layer", bb="2b", layers=1, tenants=8, samples=8, len_lo=272, len_hi=320,
             skew=0.0, align=1, shape_seed=3),
        # A layer at the headline training batch, 8 tenants x 32 samples: the largest matrix products.
        dict(name="layer_2b_8x32", kind="layer", bb="2b", layers=1, tenants=8, samples=256, len_lo=272, len_hi=320,
             skew=0.0, align=1, shape_seed=4),
        # A decoder-style backbone (causal, rotary, grouped key/value heads) at one tenant's local batch, its
        # samples aligned to 16 rows.
        dict(name="layer_2b_gqa_causal", kind="layer", bb="2b_gqa", layers=1, tenants=1, samples=32, len_lo=272,
             len_hi=320, skew=0.0, align=16, shape_seed=5),
        # A layer of the base model over four tenants of 32 single-camera samples.
        dict(name="layer_base_4x32", kind="layer", bb="base", layers=1, tenants=4, samples=128, len_lo=204,
             len_hi=244, skew=0.0, align=1, shape_seed=6),
        # The base model's layer over 32 tenants with Zipf sample counts and one to three cameras: long samples.
        dict(name="layer_base_skewed_32", kind="layer", bb="base", layers=1, tenants=32, samples=512, len_lo=272,
             len_hi=832, skew=1.2, align=1, shape_seed=7),
        # The MLP heads' training stage of the headline batch.
        dict(name="heads_8x32", kind="heads", d=2048, tenants=8, samples=256, len_lo=272, len_hi=320, skew=0.0,
             hidden=1024, hidden_layers=2, align=1, shape_seed=8),
        # Action-expert tenants of unequal sizes and camera counts, two blocks of each expert.
        dict(name="experts_16_mixed", kind="experts", d=768, layers=2, tenants=16, samples=288, len_lo=272,
             len_hi=864, skew=0.5, flow=False, align=1, shape_seed=9),
        # One tenant fine-tuning alone with the flow-matching objective and a small local batch.
        dict(name="experts_flow_1x8", kind="experts", d=768, layers=2, tenants=1, samples=8, len_lo=272, len_hi=352,
             skew=0.0, flow=True, align=1, shape_seed=10),
        # The optimizer step after the headline batch: every tenant's head, fp32 in place.
        dict(name="adamw_8_heads", kind="adamw", what="heads", d=2048, hidden=1024, hidden_layers=2, layers=0,
             tenants=8, bf16=False),
        # Intake and hand-back of the headline batch: padded requests to packed rows and hidden rows back.
        dict(name="pack_unpack_8x32", kind="pack", d=2048, tenants=8, samples=256, len_lo=272, len_hi=320, skew=0.0,
             pad=0, align=1, requests_per_tenant=1, shape_seed=12),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_group(rng, most_samples: int, most_tenants: int) -> dict:
    samples = _log_int(rng, 1, most_samples)
    lo = _log_int(rng, 16, 560)
    return dict(samples=samples, tenants=_log_int(rng, 1, min(samples, most_tenants)), len_lo=lo,
                len_hi=lo + rng.choice((rng.randint(0, 280), 560)), skew=rng.choice((0.0, 0.0, 0.5, 1.2)),
                align=rng.choice((1, 1, 1, 16)), shape_seed=rng.randrange(1 << 30))


def _draw(rng) -> dict:
    kind = rng.choice(("step", "infer", "layer", "layer", "layer", "heads", "experts", "experts", "adamw", "pack"))
    if kind == "step":
        bb = rng.choice(("tiny", "base"))
        return dict(_draw_group(rng, 96, 6), kind=kind, bb=bb, layers=rng.randint(1, 4),
                    hidden=rng.choice((256, 512, 1024)), hidden_layers=rng.randint(1, 2))
    if kind == "infer":
        return dict(_draw_group(rng, 8, 8), kind=kind, bb=rng.choice(("base", "2b", "2b_mqa", "2b_gqa")),
                    layers=rng.randint(2, 12), hidden=1024, hidden_layers=rng.randint(1, 2),
                    graph=rng.random() < 0.5)
    if kind == "layer":
        bb = rng.choice(("base", "base", "2b", "2b_mqa", "2b_gqa"))
        return dict(_draw_group(rng, 512 if bb == "base" else 128, 32), kind=kind, bb=bb, layers=1)
    if kind == "heads":
        return dict(_draw_group(rng, 512, 30), kind=kind, d=rng.choice((768, 2048)),
                    hidden=rng.choice((256, 512, 1024)), hidden_layers=rng.randint(1, 2))
    if kind == "experts":
        return dict(_draw_group(rng, 192, 8), kind=kind, d=768, layers=rng.randint(1, 2), flow=rng.random() < 0.5)
    if kind == "adamw":
        if rng.random() < 0.5:
            return dict(kind=kind, what="heads", d=rng.choice((768, 2048)), hidden=rng.randint(200, 1100),
                        hidden_layers=rng.randint(1, 2), layers=0, tenants=_log_int(rng, 1, 16), bf16=False)
        return dict(kind=kind, what="experts", d=768, hidden=0, hidden_layers=0, layers=rng.randint(1, 2),
                    tenants=_log_int(rng, 1, 8), bf16=True)
    return dict(_draw_group(rng, 256, 16), kind=kind, d=rng.choice((768, 2048)), pad=rng.randint(0, 48),
                requests_per_tenant=rng.randint(1, 3))


def draw(rng) -> dict:
    """One more case of the ranges the listed ones stand for, no dearer than the largest of them."""
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


def _cost(case: dict) -> float:
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 0.8e15)


# ----------------------------------------------------------------- shapes ---


def _counts(case: dict) -> List[int]:
    """Samples of every tenant: even, or a Zipf split with at least one each."""
    n, g, s = case["samples"], case["tenants"], case["skew"]
    if not s:
        return [n // g + (k < n % g) for k in range(g)]
    w = np.array([(k + 1) ** -s for k in range(g)])
    c = np.maximum(1, np.floor(n * w / w.sum()).astype(int))
    k = 0
    while c.sum() != n:
        if c.sum() < n:
            c[k % g] += 1
        elif c[k % g] > 1:
            c[k % g] -= 1
        k += 1
    return [int(x) for x in np.random.default_rng(case["shape_seed"]).permutation(c)]


def _lengths(case: dict) -> List[np.ndarray]:
    """Valid rows of every sample, per tenant: with a wide range a tenant draws its camera count first."""
    rng = np.random.default_rng(case["shape_seed"] + 1)
    lo, hi = case["len_lo"], case["len_hi"]
    out = []
    for n in _counts(case):
        a, b = lo, hi
        if hi - lo >= 512:
            a = lo + 256 * int(rng.integers(0, 3))
            b = min(hi, a + 48)
        out.append(rng.integers(a, b + 1, size=n).astype(np.int32))
    return out


def _schema(case: dict, g: int):
    return _SCHEMAS[(g * 3 + case["tenants"]) % len(_SCHEMAS)]


def _head_dims(case: dict, d: int, g: int) -> List[int]:
    a, c = _schema(case, g)
    return [d] + [case["hidden"]] * case["hidden_layers"] + [a * c]


def _expert_shapes(case: dict, g: int) -> Dict[str, tuple]:
    """Weights of tenant g's expert, in a fixed order."""
    d, f, a = _EXPERT["d"], _EXPERT["ffn"], _schema(case, g)[0]
    out = {"w_in": (d, a), "w_out": (a, d), "gf": (d,)}
    if case.get("flow"):
        out["w_time"] = (d, _D_TIME)
    for i in range(case["layers"]):
        for k, s in (("wqkv_s", (3 * d, d)), ("wo_s", (d, d)), ("wq_c", (d, d)), ("wkv_c", (2 * d, case["d"])),
                     ("wo_c", (d, d)), ("w_up", (f, d)), ("w_down", (d, f)), ("g1", (d,)), ("g2", (d,)),
                     ("g3", (d,))):
            out[f"{i}.{k}"] = s
    return out


def _split(flat: torch.Tensor, shapes: List[tuple]) -> List[torch.Tensor]:
    """Tensors of the given shapes inside a flat bucket, each starting on 256 bytes of fp32."""
    out, at = [], 0
    for s in shapes:
        n = math.prod(s)
        out.append(flat[at: at + n].view(s))
        at += -(-n // 64) * 64
    return out


def _bucket(shapes: List[tuple], dtype=torch.float32) -> torch.Tensor:
    return torch.zeros(sum(-(-math.prod(s) // 64) * 64 for s in shapes), dtype=dtype, device=DEV)


# ----------------------------------------------------------------- values ---


class _Draw:
    """Seeded values on the GPU."""

    def __init__(self, seed: int):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def f32(self, shape, std=1.0):
        return torch.randn(shape, generator=self.g, device=DEV).mul_(std)

    def bf16(self, shape, std=1.0):
        return self.f32(shape, std).to(torch.bfloat16)

    def gain(self, d):
        return (1 + 0.1 * self.f32((d,))).to(torch.bfloat16)

    def uniform(self, n):
        return torch.rand(n, generator=self.g, device=DEV)


def _backbone(case: dict, rnd: _Draw):
    b = _BACKBONES[case["bb"]]
    d, f = b["d"], b["ffn"]
    rows = d + 2 * (b["kv"] or b["heads"]) * (d // b["heads"])
    layers = []
    for _ in range(case["layers"]):
        w = {"wqkv": rnd.bf16((rows, d), 0.02), "wo": rnd.bf16((d, d), 0.02), "w_up": rnd.bf16((f, d), 0.02),
             "w_down": rnd.bf16((d, f), 0.02), "g1": rnd.gain(d), "g2": rnd.gain(d)}
        if b["glu"]:
            w["w_gate"] = rnd.bf16((f, d), 0.02)
        layers.append(w)
    return layers, rnd.gain(d)


def _requests(case: dict, d: int, rnd: _Draw, pad: int = 0, per_tenant: int = 1):
    """Padded observations, every tenant's samples cut into ``per_tenant`` requests; rows past a length are filler."""
    out = []
    for g, lens in enumerate(_lengths(case)):
        for part in np.array_split(lens, min(per_tenant, len(lens))):
            out.append(jn.Request(g, rnd.bf16((len(part), int(lens.max()) + pad, d)), part))
    return out


def _heads(case: dict, d: int, rnd: _Draw):
    out = []
    for g in range(case["tenants"]):
        dims = _head_dims(case, d, g)
        out.append(([rnd.f32((o, i), i ** -0.5) for i, o in zip(dims[:-1], dims[1:])],
                    [rnd.f32((o,), 0.02) for o in dims[1:]]))
    return out


def _targets(case: dict, rnd: _Draw):
    return [rnd.f32((n, math.prod(_schema(case, g)))) for g, n in enumerate(_counts(case))]


def _inputs(case: dict, seed: int) -> SimpleNamespace:
    """What both ``prepare`` and ``exact`` start from."""
    rnd, s = _Draw(seed), SimpleNamespace()
    kind = case["kind"]
    if kind in ("step", "infer", "layer"):
        s.b = _BACKBONES[case["bb"]]
        s.d = s.b["d"]
        s.layers, s.gf = _backbone(case, rnd)
        s.requests = _requests(case, s.d, rnd)
    if kind == "pack":
        s.d = case["d"]
        s.requests = _requests(case, s.d, rnd, case["pad"], case["requests_per_tenant"])
    if kind in ("heads", "experts"):
        s.d = case["d"]
        # the rows themselves come from the backbone: the requests only carry sizes
        s.requests = [jn.Request(g, None, lens, int(lens.max())) for g, lens in enumerate(_lengths(case))]
        s.hidden = rnd.bf16((int(sum(_rows(r.lengths, case["align"]).sum() for r in s.requests)), s.d))
    if kind in ("step", "infer", "heads"):
        s.heads = _heads(case, s.d, rnd)
    if kind in ("step", "heads"):
        s.targets = _targets(case, rnd)
    if kind == "experts":
        s.shapes = [_expert_shapes(case, g) for g in range(case["tenants"])]
        s.weights = [{k: rnd.gain(v[0]) if len(v) == 1 else rnd.bf16(v, 0.02) for k, v in sh.items()}
                     for sh in s.shapes]
        sizes = [(n, _EXPERT["chunk"], _schema(case, g)[0]) for g, n in enumerate(_counts(case))]
        s.noisy = [rnd.f32(x) for x in sizes]
        s.targets = [rnd.f32(x) for x in sizes]
        s.flow_t = [0.001 + 0.999 * rnd.uniform(x[0]) ** (1 / 1.5) for x in sizes] if case["flow"] else None
    if kind == "adamw":
        s.shapes = []
        for g in range(case["tenants"]):
            if case["what"] == "heads":
                dims = _head_dims(case, case["d"], g)
                s.shapes.append([(o, i) for i, o in zip(dims[:-1], dims[1:])] + [(o,) for o in dims[1:]])
            else:
                s.shapes.append(list(_expert_shapes(case, g).values()))
        s.p, s.g, s.m, s.v = [], [], [], []
        for sh in s.shapes:
            n = _bucket(sh).numel()
            s.p.append(rnd.f32((n,), 0.03))
            s.g.append(rnd.f32((n,), 1e-3))
            s.m.append(rnd.f32((n,), 3e-4))
            s.v.append(rnd.f32((n,), 1e-3).square_())
        s.hyper = [dict(lr=1e-4 * (1 + g % 3), weight_decay=0.01 * (g % 2)) for g in range(case["tenants"])]
    return s


def _rows(lens: np.ndarray, align: int) -> np.ndarray:
    return -(-lens // align) * align


# ------------------------------------------------------------ entry points ---


def prepare(case: dict, seed: int) -> SimpleNamespace:
    s = _inputs(case, seed)
    s.case, kind = case, case["kind"]
    if kind in ("step", "infer"):
        _prepare_model(case, s)
        return s
    s.ctx = jn.Context()
    if kind == "adamw":
        _prepare_adamw(case, s)
        return s
    if kind in ("heads", "experts"):
        # an MLP or expert stage follows a pack of some rows: the packed values are not read by it
        for r in s.requests:
            r.embeds = torch.zeros((r.n, r.max_len, s.d), dtype=torch.bfloat16, device=DEV)
    s.table = [jn.Tenant(SIG, s.d) for _ in range(case["tenants"])]
    size = jn.jn_pack_plan(s.requests, s.table, s.d, case["align"])
    s.maps = torch.empty(int(size.map_bytes), dtype=torch.uint8, device=DEV)
    s.tokens = torch.empty((size.T, s.d), dtype=torch.bfloat16, device=DEV)
    s.packed = jn.jn_pack_group(s.ctx, s.requests, s.table, s.d, case["align"], s.maps, s.tokens)
    if kind == "layer":
        s.bb = _make_backbone(s)
        s.hidden = torch.empty_like(s.tokens)
        s.ws = torch.empty(jn.jn_backbone_workspace_size(s.bb, size.T), dtype=torch.uint8, device=DEV)
    elif kind == "pack":
        s.out = [torch.empty_like(r.embeds) for r in s.requests]
    elif kind == "heads":
        _prepare_heads(case, s)
    else:
        _prepare_experts(case, s)
    return s


def _make_backbone(s) -> jn.Backbone:
    return jn.Backbone(s.layers, s.gf, s.b["heads"], EPS, s.b["kv"], s.b["causal"], s.b["rope"])


@functools.lru_cache(maxsize=None)
def _serving_stream():
    """A server runs its resident plans one after another on one stream (a captured graph needs its own)."""
    return torch.cuda.Stream()


def _prepare_model(case: dict, s):
    meta = [dict(zip(("action_dim", "chunk"), _schema(case, g))) for g in range(case["tenants"])]
    heads = [jn.Head(W, b, m["action_dim"], m["chunk"]) for (W, b), m in zip(s.heads, meta)]
    model = jstep.Model(_make_backbone(s), heads, meta, SIG)
    tenants = list(range(case["tenants"]))
    if case["kind"] == "infer":
        s.step = jstep.InferStep(model, s.requests, tenants, case["align"], stream=_serving_stream())
        packed, hidden = s.step.plan.packed()
        at = hidden - s.step.ws.data_ptr()
        s.hidden = s.step.ws[at: at + packed.T * s.d * 2].view(torch.bfloat16).view(packed.T, s.d)
        if case["graph"]:
            s.step.capture()
    else:
        s.step = jstep.GroupStep(model, s.requests, {g: t.cpu().numpy() for g, t in enumerate(s.targets)}, tenants,
                                 case["align"])


def _prepare_heads(case: dict, s):
    s.mlps, s.ios, s.grads = [], [], []
    s.loss = torch.zeros(case["tenants"], device=DEV)
    for g, (W, b) in enumerate(s.heads):
        a, c = _schema(case, g)
        s.mlps.append(jn.Head(W, b, a, c))
        shapes = [tuple(t.shape) for t in W + b]
        s.grads.append(_bucket(shapes))
        views = _split(s.grads[-1], shapes)
        s.ios.append(jn.HeadIO(s.targets[g], torch.empty_like(s.targets[g]), s.loss[g:], views[:len(W)],
                               views[len(W):]))
    s.pooled = torch.empty((s.packed.N, s.d), device=DEV)
    s.ws = torch.empty(jn.jn_heads_workspace_size(s.packed, s.mlps), dtype=torch.uint8, device=DEV)


def _prepare_experts(case: dict, s):
    n_s, rows = jn.jn_pack_tenant_sizes(s.requests, s.table, s.d, case["align"])
    s.experts, s.ios, s.grads = [], [], []
    s.loss = torch.zeros(case["tenants"], device=DEV)

    def by_layer(t):
        return [{k: t[f"{i}.{k}"] for k in jn.EXPERT_LAYER_FIELDS} for i in range(case["layers"])]

    for g, w in enumerate(s.weights):
        s.experts.append(jn.Expert(w["w_in"], w["w_out"], w["gf"], by_layer(w), _EXPERT["heads"], _EXPERT["chunk"],
                                   s.d, EPS, w.get("w_time")))
        shapes = list(s.shapes[g].values())
        s.grads.append(_bucket(shapes))
        dw = dict(zip(s.shapes[g], _split(s.grads[-1], shapes)))
        s.ios.append(jn.ExpertIO(int(n_s[g]), int(rows[g]), s.noisy[g], s.targets[g], torch.empty_like(s.targets[g]),
                                 s.loss[g:], dw["w_in"], dw["w_out"], dw["gf"], by_layer(dw),
                                 s.flow_t[g] if case["flow"] else None, dw.get("w_time")))
    s.ws = torch.empty(jn.jn_experts_workspace_size(s.packed, s.experts, s.ios), dtype=torch.uint8, device=DEV)


def _prepare_adamw(case: dict, s):
    s.tenants, s.bf16 = [], []
    for g, sh in enumerate(s.shapes):
        copies = torch.zeros(s.p[g].numel(), dtype=torch.bfloat16, device=DEV) if case["bf16"] else None
        s.bf16.append(copies)
        s.tenants.append(jn.AdamWTenant(*(_split(x[g], sh) for x in (s.p, s.g, s.m, s.v)), step=9,
                                        bf16_out=_split(copies, sh) if case["bf16"] else None, **s.hyper[g]))
    s.ws = torch.empty(jn.jn_adamw_workspace_size(s.tenants), dtype=torch.uint8, device=DEV)


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "step":
        st = s.step
        st.run()
        return {"hidden": st.out_hidden, "pooled": st.pooled, "actions": [io.actions for io in st.ios],
                "loss": [io.loss for io in st.ios], "dW": [io.dW for io in st.ios], "db": [io.db for io in st.ios]}
    if kind == "infer":
        s.step.replay() if case["graph"] else s.step.launch()
        return {"actions": s.step.actions, "hidden": s.hidden}
    if kind == "layer":
        jn.jn_backbone_forward(s.ctx, s.bb, s.packed, s.hidden, s.ws)
        return s.hidden
    if kind == "heads":
        jn.jn_tenant_heads_fwd_bwd(s.ctx, s.packed, s.hidden, s.mlps, s.ios, s.ws, s.pooled)
        return {"pooled": s.pooled, "loss": s.loss, "grads": s.grads, "actions": [io.actions for io in s.ios]}
    if kind == "experts":
        jn.jn_tenant_experts_fwd_bwd(s.ctx, s.packed, s.hidden, s.experts, s.ios, s.ws)
        return {"pred": [io.pred for io in s.ios], "loss": s.loss, "grads": s.grads}
    if kind == "adamw":
        for t in s.tenants:
            t.struct.step += 1
        jn.jn_tenant_adamw_step(s.ctx, s.tenants, s.ws)
        return {"p": s.p, "m": s.m, "v": s.v, "bf16": [x for x in s.bf16 if x is not None]}
    s.packed = jn.jn_pack_group(s.ctx, s.requests, s.table, s.d, case["align"], s.maps, s.tokens)
    jn.jn_unpack(s.ctx, s.packed, s.requests, s.tokens, s.d * 2, s.out)
    return {"tokens": s.tokens, "rows": s.out}


# -------------------------------------------------------------- accounting ---


def work(case: dict) -> dict:
    """Bytes each input once in and each output once out; operations on valid rows only."""
    kind = case["kind"]
    by = fl = 0.0
    if kind == "adamw":
        if case["what"] == "heads":
            n = sum(i * o + o for g in range(case["tenants"])
                    for i, o in zip(_head_dims(case, case["d"], g)[:-1], _head_dims(case, case["d"], g)[1:]))
        else:
            n = sum(math.prod(v) for g in range(case["tenants"]) for v in _expert_shapes(case, g).values())
        return {"bytes": n * (30.0 if case["bf16"] else 28.0), "flops": 15.0 * n}
    lens = _lengths(case)
    every = np.concatenate(lens).astype(np.float64)
    rows, pairs = every.sum(), (every ** 2).sum()
    d = _BACKBONES[case["bb"]]["d"] if "bb" in case else case["d"]
    if kind in ("step", "infer", "layer"):
        b = _BACKBONES[case["bb"]]
        qkv = d + 2 * (b["kv"] or b["heads"]) * (d // b["heads"])
        weights = qkv * d + d * d + (3 if b["glu"] else 2) * b["ffn"] * d
        by += case["layers"] * weights * 2 + rows * d * 4
        fl += case["layers"] * (2 * rows * weights + 4 * pairs * d * (0.5 if b["causal"] else 1))
    if kind in ("step", "infer", "heads"):
        for g, n in enumerate(_counts(case)):
            dims = _head_dims(case, d, g)
            for k, (i, o) in enumerate(zip(dims[:-1], dims[1:])):
                train = kind != "infer"
                by += (i + 1) * o * (8 if train else 4)
                fl += 2.0 * n * i * o * (1 + (2 if k else 1) * train)
            by += 4.0 * n * dims[-1] * (2 if kind != "infer" else 1)
    if kind == "heads":
        by += rows * d * 2 + len(every) * d * 4
    if kind == "step":
        by += sum(x.size * int(x.max()) for x in lens) * d * 2 + len(every) * d * 4
    if kind == "pack":
        by += rows * d * 6 + sum(x.size * (int(x.max()) + case["pad"]) for x in lens) * d * 2
    if kind == "experts":
        e = _EXPERT
        by += rows * d * 2
        for g, x in enumerate(lens):
            a, na = _schema(case, g)[0], x.size * e["chunk"]
            by += sum(math.prod(v) for v in _expert_shapes(case, g).values()) * 6 + na * a * 12
            per_row = 6 * e["d"] ** 2 + 2 * e["d"] * e["ffn"]
            fl += 6.0 * case["layers"] * na * per_row
            fl += 4.0 * case["layers"] * x.sum() * 2 * e["d"] * d  # the prefix gets no gradient
            fl += 12.0 * case["layers"] * e["d"] * (x.size * e["chunk"] ** 2 + e["chunk"] * float(x.sum()))
            fl += 10.0 * na * a * e["d"] + (4.0 * na * _D_TIME * e["d"] if case["flow"] else 0)
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case: dict):
    """About four times the distance to ``exact`` that was measured for each kind (in brackets), which is what
    another rounding of the same bf16 values, or summation order of the same fp32 ones, gives."""
    kind = case["kind"]
    if kind == "pack":
        return "exact"  # copies
    if kind == "adamw":
        # fp32 updates (4e-8); a bf16 copy may round to the other side
        return {"rel": 1e-4, "max": 1e-2} if case["bf16"] else {"rel": 3e-7, "max": 1e-5}
    if kind == "heads":
        return {"rel": 3e-6, "max": 1e-3}  # (4e-7)
    if kind in ("layer", "step"):
        return {"rel": 1.2e-2, "max": 0.2}  # one layer (3e-3), a few of them and a head (2e-3)
    if kind == "experts":
        return {"rel": 2e-2, "max": 0.4}  # two blocks and their gradients (5e-3)
    return {"rel": 3e-2, "max": 0.5}  # a whole model of up to 18 layers (1.1e-2)


# ------------------------------------------------------------------- exact ---


def _rms(x, g):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g.to(F64)


def _gelu(u):
    return 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))


def _rotate(x, theta):
    """Rotary positions of [heads, rows, hd], pairs (i, i + hd/2)."""
    hd = x.shape[-1]
    at = torch.arange(x.shape[1], device=x.device, dtype=F64)[:, None]
    ang = at * theta ** (-2 * torch.arange(hd // 2, device=x.device, dtype=F64) / hd)
    a, b = x[..., : hd // 2], x[..., hd // 2:]
    return torch.cat((a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()), -1)


def _attend(q, k, v, causal=False):
    """[heads, rows, hd] each."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if causal:
        s = s.masked_fill(torch.ones(s.shape[1:], dtype=torch.bool, device=s.device).triu(1), -math.inf)
    return torch.matmul(torch.softmax(s, -1), v)


def _exact_backbone(s, samples: List[torch.Tensor]) -> List[torch.Tensor]:
    """The frozen backbone in float64 over samples of valid rows."""
    b, d = s.b, s.d
    hd, kv = d // b["heads"], b["kv"] or b["heads"]
    lens = [x.shape[0] for x in samples]
    x = torch.cat(samples).to(F64)
    for w in s.layers:
        w = {k: v.to(F64) for k, v in w.items()}
        qkv = _rms(x, w["g1"]) @ w["wqkv"].T
        parts, at = [], 0
        for n in lens:
            t = qkv[at: at + n].view(n, -1, hd).transpose(0, 1)
            q, k, v = t[: b["heads"]], t[b["heads"]: b["heads"] + kv], t[b["heads"] + kv:]
            if b["rope"]:
                q, k = _rotate(q, b["rope"]), _rotate(k, b["rope"])
            r = b["heads"] // kv
            o = _attend(q, k.repeat_interleave(r, 0), v.repeat_interleave(r, 0), b["causal"])
            parts.append(o.transpose(0, 1).reshape(n, d))
            at += n
        del qkv
        x = x + torch.cat(parts) @ w["wo"].T
        del parts
        for i in range(0, x.shape[0], 16384):  # the MLP's rows are independent
            h = _rms(x[i: i + 16384], w["g2"])
            u = h @ w["w_up"].T
            u = _gelu(h @ w["w_gate"].T) * u if b["glu"] else _gelu(u)
            x[i: i + 16384] += u @ w["w_down"].T
    return list(_rms(x, s.gf).split(lens))


def _padded(parts: List[torch.Tensor], align: int) -> torch.Tensor:
    out = []
    for x in parts:
        out.append(x)
        fill = -x.shape[0] % align
        if fill:
            out.append(x.new_zeros((fill, x.shape[1])))
    return torch.cat(out)


def _exact_head(W, b, p, targets=None):
    """(actions, loss, gradients of W then b) of one tenant."""
    leaves = [t.to(F64).requires_grad_(targets is not None) for t in list(W) + list(b)]
    h = p
    for k in range(len(W)):
        h = h @ leaves[k].T + leaves[len(W) + k]
        if k + 1 < len(W):
            h = _gelu(h)
    if targets is None:
        return h, None, None
    loss = (h - targets.to(F64).view_as(h)).square().mean()
    return h.detach(), loss.detach(), torch.autograd.grad(loss, leaves)


def _into_bucket(values, shapes) -> torch.Tensor:
    flat = _bucket(shapes, F64)
    for dst, src in zip(_split(flat, shapes), values):
        dst.copy_(src)
    return flat


def _exact_expert(case, w, n, hidden, noisy, targets, flow_t):
    """(predictions, loss, gradients in the weights' order) of one tenant; ``hidden``: its samples' valid rows."""
    d, hd, L = _EXPERT["d"], _EXPERT["d"] // _EXPERT["heads"], _EXPERT["chunk"]
    w = {k: v.to(F64).requires_grad_(True) for k, v in w.items()}
    x, t = noisy.to(F64), targets.to(F64)
    if flow_t is not None:
        tau = flow_t.to(F64)[:, None, None]
        x, t = tau * x + (1 - tau) * t, x - t
    h = x @ w["w_in"].T
    if flow_t is not None:
        freq = 10000.0 ** (-torch.arange(_D_TIME // 2, device=DEV, dtype=F64) / (_D_TIME // 2))
        ang = 1000 * flow_t.to(F64)[:, None] * freq
        h = h + (torch.cat((ang.sin(), ang.cos()), -1) @ w["w_time"].T)[:, None]

    def split(y):
        return y.view(y.shape[0], -1, hd).transpose(0, 1)

    for i in range(case["layers"]):
        def W(k):
            return w[f"{i}.{k}"]
        qkv = _rms(h, W("g1")) @ W("wqkv_s").T
        q, k, v = (split(y.reshape(n * L, d)).reshape(-1, n, L, hd).flatten(0, 1) for y in qkv.split(d, -1))
        o = _attend(q, k, v).view(-1, n, L, hd).permute(1, 2, 0, 3).reshape(n, L, d)
        h = h + o @ W("wo_s").T
        q = _rms(h, W("g2")) @ W("wq_c").T
        o = []
        for j, rows in enumerate(hidden):
            kv = rows.to(F64) @ W("wkv_c").T
            o.append(_attend(split(q[j]), split(kv[:, :d]), split(kv[:, d:])).transpose(0, 1).reshape(L, d))
        h = h + torch.stack(o) @ W("wo_c").T
        h = h + _gelu(_rms(h, W("g3")) @ W("w_up").T) @ W("w_down").T
    pred = _rms(h, w["gf"]) @ w["w_out"].T
    loss = (pred - t).square().mean()
    return pred.detach(), loss.detach(), torch.autograd.grad(loss, list(w.values()))


def exact(case: dict, seed: int):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "pack":
        return None  # copies: nothing is computed
    if kind == "adamw":
        return _exact_adamw(case, s)
    if kind in ("step", "infer", "layer"):
        hidden = _exact_backbone(s, [r.embeds[i, : r.lengths[i]] for r in s.requests for i in range(r.n)])
        if kind == "layer":
            return _padded(hidden, case["align"])
    else:
        hidden, at = [], 0
        for r in s.requests:
            for n, m in zip(r.lengths, _rows(r.lengths, case["align"])):
                hidden.append(s.hidden[at: at + int(n)])
                at += int(m)
    by_tenant = [[hidden.pop(0) for _ in range(r.n)] for r in s.requests]  # one request per tenant, in order
    if kind == "experts":
        got = [_exact_expert(case, s.weights[g], len(rows), rows, s.noisy[g], s.targets[g],
                             s.flow_t[g] if case["flow"] else None) for g, rows in enumerate(by_tenant)]
        # a loss's distance to 64 bits is the chance sum of its predictions' roundings, which are compared themselves
        return {"pred": [x[0] for x in got], "loss": None,
                "grads": [_into_bucket(x[2], list(sh.values())) for x, sh in zip(got, s.shapes)]}
    pooled = [torch.stack([x.to(F64).mean(0) for x in rows]) for rows in by_tenant]
    got = [_exact_head(W, b, p, s.targets[g] if kind != "infer" else None)
           for g, ((W, b), p) in enumerate(zip(s.heads, pooled))]
    actions = [x[0] for x in got]
    if kind == "infer":
        return {"actions": actions, "hidden": _padded([x for rows in by_tenant for x in rows], case["align"])}
    if kind == "heads":
        return {"pooled": torch.cat(pooled), "loss": torch.stack([x[1] for x in got]), "actions": actions,
                "grads": [_into_bucket(x[2], [tuple(t.shape) for t in W + b])
                          for x, (W, b) in zip(got, s.heads)]}
    out = []
    for rows, r in zip(by_tenant, s.requests):
        full = torch.zeros((r.n, r.max_len, s.d), dtype=F64, device=DEV)
        for i, x in enumerate(rows):
            full[i, : x.shape[0]] = x
        out.append(full)
    return {"hidden": out, "pooled": torch.cat(pooled), "actions": actions, "loss": None,  # as above
            "dW": [list(x[2][: len(W)]) for x, (W, _) in zip(got, s.heads)],
            "db": [list(x[2][len(W):]) for x, (W, _) in zip(got, s.heads)]}


def _exact_adamw(case: dict, s):
    out = {"p": [], "m": [], "v": [], "bf16": []}
    for g, sh in enumerate(s.shapes):
        b1, b2, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-8))
        lr, wd = (float(np.float32(s.hyper[g][k])) for k in ("lr", "weight_decay"))
        step, copies = 10, torch.zeros(s.p[g].numel(), dtype=F64, device=DEV)
        views = [[t for t in _split(x[g].to(F64), sh)] for x in (s.p, s.g, s.m, s.v)]
        flat = [x[g].to(F64) for x in (s.p, s.m, s.v)]
        dst = [_split(x, sh) for x in flat] + [_split(copies, sh)]
        for i, (p, gr, m, v) in enumerate(zip(*views)):
            m = b1 * m + (1 - b1) * gr
            v = b2 * v + (1 - b2) * gr * gr
            p = p * (1 - lr * wd) - lr / (1 - b1 ** step) * m / ((v / (1 - b2 ** step)).sqrt() + eps)
            for t, x in zip(dst, (p, m, v, p)):
                t[i].copy_(x)
        for k, x in zip(("p", "m", "v"), flat):
            out[k].append(x)
        if case["bf16"]:
            out["bf16"].append(copies)
    return out
