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
