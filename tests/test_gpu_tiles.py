"""Edges of the GEMM tile shapes and of the K split, through the backbone call:
row counts around every tile height (96, 128, 160, 256), weight widths that end
inside a tile, and a down projection (K = 2,176 = 34 slabs) that short batches
split into ranges of unequal length, its reduction fused with the next norm.
Hidden rows against the fp64 oracle at the 2e-2 max-relative bar of the other
backbone tests (bf16 operands); a sample alone equals the same sample in a
longer batch bitwise where no contraction is split (K < 2,048)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROWS = (1, 17, 64, 95, 96, 97, 128, 129, 159, 161, 257, 320, 513)


def spec(lens, d, ffn, glu):
    ten = tuple(W.TenantSpec(1, n, 0, 0, n, (d, 64, 6), 3, 2) for n in lens)
    return W.WorkloadSpec(97, W.BackboneSpec(2, d, 3, ffn, glu), ten, 0, "tile edges")


def hidden(wl, tenants):
    from paper_2607_16074_amd import step as jstep
    model, reqs, targets = jstep.from_workload(wl)
    st = jstep.GroupStep(model, [r for r in reqs if r.tenant in tenants], targets, list(tenants))
    st.run()
    torch.cuda.synchronize()
    return st


@pytest.mark.parametrize("ffn,glu", [(2176, False), (640, True)])
@pytest.mark.parametrize("rows", ROWS)
def test_rows_at_tile_edges(rows, ffn, glu):
    import oracle
    print(f"rows {rows} ffn {ffn} glu {glu}", flush=True)
    wl = W.make_workload(spec((rows,), 384, ffn, glu))
    got = hidden(wl, [0]).hidden.float().cpu().numpy().astype(np.float64)
    ref = oracle.step.isolated(wl, heads=False)["hidden"][(0, 0)]
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) / np.max(np.abs(ref)) < 2e-2


def test_sample_alone_equals_sample_in_a_batch_bitwise():
    lens = (97, 161, 33, 320, 256)
    wl = W.make_workload(spec(lens, 384, 640, True))
    full, at = hidden(wl, range(len(lens))).hidden, 0
    for g, n in enumerate(lens):
        assert torch.equal(hidden(wl, [g]).hidden, full[at: at + n]), g
        at += n


@pytest.mark.parametrize("d", [128, 384])
def test_workgroups_with_several_tiles_bitwise(d):
    """Launches whose workgroups take several 256x256 tiles in turn (19,903
    rows, 1,920 columns: 632 tiles), joined (384 columns are six K slabs) and
    not (128 are two): samples at both ends and the middle equal themselves
    alone, where no tile follows another."""
    lens = (313,) * 31 + (300,) * 34
    wl = W.make_workload(W.WorkloadSpec(
        96, W.BackboneSpec(1, d, d // 128, 1920, False),
        tuple(W.TenantSpec(1, n, 0, 0, n, (d, 64, 6), 3, 2) for n in lens), 0, "many tiles"))
    full, at = hidden(wl, range(len(lens))).hidden, 0
    assert full.shape[0] == sum(lens)
    for g, n in enumerate(lens):
        if g in (0, 1, 30, 31, 47, 63, 64):
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
