"""Edges of the GEMM tile shapes and of the K split, through the backbone call.
Every test asks the plan which shape its sizes get, so none passes on another one.

Short batches run 64x96 tiles (weight rows x tokens): row counts around its and the
other shapes' heights, and a down projection (K = 2,176 = 34 slabs) split into
ranges of unequal length, its reduction fused with the next norm.  Every other
shape, per epilogue: one row fewer than, exactly and one more than whole tiles, weight
widths that end inside a 256-wide tile, unsplit and split.  Hidden rows against the
fp64 oracle at the 2e-2 max-relative bar of the other backbone tests (bf16
operands); a sample alone (64x96 for the most part) equals the same sample in batches
of other shapes bitwise where no contraction is split (K < 2,048)."""
import numpy as np
import pytest

import workloads as W
from test_gemm_plan import BF16, GEGLU, GELU, RESID, gemm_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROWS = (1, 17, 64, 95, 96, 97, 128, 129, 159, 161, 257, 320, 513)


def spec(lens, d, ffn, glu, layers=2):
    ten = tuple(W.TenantSpec(1, n, 0, 0, n, (d, 64, 6), 3, 2) for n in lens)
    return W.WorkloadSpec(97, W.BackboneSpec(layers, d, d // 128, ffn, glu), ten, 0, "tile edges")


def plans(rows, d, ffn, glu):
    """(leading rows on 256x256 tiles, shape of the others, K ranges) of the four projections."""
    import paper_2607_16074_amd as lib
    return {"qkv": gemm_plan(lib, BF16, rows, 3 * d, d), "o": gemm_plan(lib, RESID, rows, d, d),
            "up": gemm_plan(lib, GEGLU if glu else GELU, rows, ffn, d), "down": gemm_plan(lib, RESID, rows, d, ffn)}


def hidden(wl, tenants):
    from paper_2607_16074_amd import step as jstep
    model, reqs, targets = jstep.from_workload(wl)
    st = jstep.GroupStep(model, [r for r in reqs if r.tenant in tenants], targets, list(tenants))
    st.run()
    torch.cuda.synchronize()
    return st


def check_hidden(wl, lens):
    import oracle
    got = hidden(wl, range(len(lens))).hidden.float().cpu().numpy().astype(np.float64)
    by = oracle.step.isolated(wl, heads=False)["hidden"]
    ref = np.concatenate([by[(r, 0)] for r in range(len(lens))])
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) / np.max(np.abs(ref)) < 2e-2


@pytest.mark.parametrize("ffn,glu", [(2176, False), (640, True)])
@pytest.mark.parametrize("rows", ROWS)
def test_rows_at_tile_edges(rows, ffn, glu):
    print(f"rows {rows} ffn {ffn} glu {glu}", flush=True)
    p = plans(rows, 384, ffn, glu)
    assert all(x[:2] == (0, "64x96") for x in p.values()) and (p["down"][2] > 1) == (ffn > 2048), p
    check_hidden(W.make_workload(spec((rows,), 384, ffn, glu)), (rows,))


@pytest.mark.parametrize("gemm,shape,split,d,ffn,glu,tiles", [
    ("qkv", "128x96", False, 256, 128, False, 22), ("qkv", "128x160", False, 256, 128, False, 26),
    ("qkv", "256x128", False, 384, 128, False, 36), ("qkv", "256x160", False, 640, 128, False, 26),
    ("qkv", "256x256", False, 640, 128, False, 21),
    ("up", "128x96", False, 128, 4224, False, 4), ("up", "128x160", False, 128, 4224, False, 5),
    ("up", "256x128", False, 128, 4224, False, 9), ("up", "256x160", False, 128, 2176, False, 23),
    ("up", "256x256", False, 128, 2176, False, 18), ("up", "64x96", True, 2048, 128, False, 1),
    ("up", "128x96", False, 128, 4224, True, 2), ("up", "128x160", False, 128, 4224, True, 2),
    ("up", "256x128", False, 128, 4224, True, 4), ("up", "256x160", False, 128, 4224, True, 6),
    ("up", "256x256", False, 128, 4224, True, 5),
    ("o", "128x128", False, 128, 128, False, 1), ("o", "128x96", False, 1280, 128, False, 13),
    ("o", "128x160", False, 768, 128, False, 34), ("o", "256x160", False, 1536, 128, False, 34),
    ("down", "256x128", False, 1280, 2176, False, 32),
    ("down", "128x96", True, 256, 4224, False, 33), ("down", "128x160", True, 384, 3072, False, 26),
    ("down", "256x256", True, 1280, 4224, False, 16),
])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_every_shape_at_its_edges(gemm, shape, split, d, ffn, glu, tiles, more):
    rows = tiles * int(shape.split("x")[1]) + more
    print(f"{gemm} {shape} split {split} d {d} ffn {ffn} glu {glu} rows {rows}", flush=True)
    m1, got, ranges = plans(rows, d, ffn, glu)[gemm]
    assert (m1, got, ranges > 1) == (0, shape, split)
    lens = (97,) * (rows // 97) + ((rows % 97,) if rows % 97 else ())
    check_hidden(W.make_workload(spec(lens, d, ffn, glu, layers=1)), lens)


@pytest.mark.parametrize("d,ffn,glu,lens,shapes", [
    (384, 1920, True, (97, 161, 33, 320, 256, 33) + (300,) * 12, ["256x128", "128x128", "256x160", "128x96"]),
    (512, 1920, False, (97, 161, 33) + (330,) * 7, ["128x160", "64x96", "128x160", "64x96"]),
    (1024, 1920, True, (97, 161, 33, 320, 289, 400), ["128x160", "64x96", "256x128", "64x96"]),
    # leading rows on 256x256 tiles and a tail
    (768, 1920, False, (300,) * 30, ["128x160", "128x128", "256x160", "128x128"]),
])
def test_sample_alone_equals_sample_in_a_batch_bitwise(d, ffn, glu, lens, shapes):
    print(f"d {d} ffn {ffn} glu {glu} rows {sum(lens)}", flush=True)
    p = plans(sum(lens), d, ffn, glu)
    assert [x[1] for x in p.values()] == shapes and all(x[2] == 1 for x in p.values()), p
    wl = W.make_workload(spec(lens, d, ffn, glu))
    full, at = hidden(wl, range(len(lens))).hidden, 0
    for g, n in enumerate(lens):
        if g < 6 or g >= len(lens) - 6:
            alone = plans(n, d, ffn, glu)
            assert all(x[2] == 1 for x in alone.values()) and alone["up"][1] != p["up"][1], alone
            assert torch.equal(hidden(wl, [g]).hidden, full[at: at + n]), g
        at += n


@pytest.mark.parametrize("d,glu,lens,gemm,joined", [
    (384, False, (313,) * 31 + (300,) * 34, "qkv", True),    # 78 x 5 tiles of six slabs
    (128, True, (313,) * 31 + (300,) * 34, "up", False),     # 78 x 15 tiles of two
    (128, False, (300,) * 100, "up", False),                 # 118 x 8
])
def test_workgroups_with_several_tiles_bitwise(d, glu, lens, gemm, joined):
    """Launches of more than 256 tiles of 256x256, whose workgroups take several in
    turn, joined (three K slabs or more: the next tile's first slabs are fetched
    under the last ones) and not: samples at both ends and the middle equal
    themselves alone, where no tile follows another."""
    ffn, rows = 1920, sum(lens)
    print(f"d {d} glu {glu} rows {rows}", flush=True)
    m1, shape, ranges = plans(rows, d, ffn, glu)[gemm]
    columns = 3 * d if gemm == "qkv" else ffn * (2 if glu else 1)
    assert (m1, shape, ranges) == (0, "256x256", 1) and -(-rows // 256) * -(-columns // 256) > 256
    assert (d // 64 >= 3) == joined
    wl = W.make_workload(W.WorkloadSpec(
        96, W.BackboneSpec(1, d, d // 128, ffn, glu),
        tuple(W.TenantSpec(1, n, 0, 0, n, (d, 64, 6), 3, 2) for n in lens), 0, "many tiles"))
    full, at = hidden(wl, range(len(lens))).hidden, 0
    assert full.shape[0] == rows
    last = len(lens) - 1
    for g, n in enumerate(lens):
        if g in (0, 1, 30, 31, 47, last - 1, last):
            print(f"sample {g}", flush=True)
            assert torch.equal(hidden(wl, [g]).hidden, full[at: at + n]), g
        at += n


@pytest.mark.parametrize("hidden_dims,rows", [
    ((33, 1), (1,)), ((31, 65), (2, 33)), ((300, 257), (32, 1, 31)), ((64, 1030), (65, 7)), ((515,), (40, 24))])
def test_head_tiles_at_edges(hidden_dims, rows):
    """Head widths that end inside a 32-wide tile, a 64 x 256 weight-gradient
    tile, a wave's K range or a 16-byte vector, and row counts around one tile.
    fp32 throughout: a sum of K <= 1,030 products grows by about sqrt(K) 2^-24
    = 2e-6, over at most five chained products (three forward, two backward)."""
    import oracle
    print(f"widths {hidden_dims} rows {rows}", flush=True)
    d, act, chunk = 640, 3, 5
    ten = tuple(W.TenantSpec(n, 0, 1, 9, 9, (d,) + hidden_dims + (act * chunk,), act, chunk) for n in rows)
    wl = W.make_workload(W.WorkloadSpec(98, W.BackboneSpec(1, d, 5, 256, False), ten, 0, "head edges"))
    st = hidden(wl, range(len(rows)))
    pooled, off = st.pooled.cpu().numpy().astype(np.float64), 0

    def rel(t, ref):
        return np.linalg.norm(t.cpu().numpy().astype(np.float64) - ref) / max(np.linalg.norm(ref), 1e-30)

    for g, n in enumerate(rows):
        ref = oracle.step.tenant_from_pooled(wl, g, pooled[off: off + n])
        off += n
        io = st.ios[g]
        assert rel(io.actions, ref["actions"]) < 1e-5
        assert abs(float(io.loss) - ref["loss"]) <= 1e-5 * abs(ref["loss"])
        for layer, (dw, db) in enumerate(ref["grads"]):
            assert rel(io.dW[layer], dw) < 1e-5 and rel(io.db[layer], db) < 1e-5, (g, layer)
