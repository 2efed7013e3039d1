"""Head gradients of tenants with many rows: above 256 rows (512 where the gradient
has more than 32 tiles of 64 x 256: 1,088 x 384) the eight waves of a workgroup
share a 32 x 64 part of the weight gradient, each a range of the rows.  Row counts
around those lines and around a range's 16-row slabs, widths that end inside a
part.  fp32 throughout against float64: a sum of K rows grows by about
sqrt(K) 2^-24, 4e-6 at 4,097, over at most five chained products."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [((256,), (255, 256, 257)), ((33, 70), (1, 300, 129)), ((300, 257), (513,)), ((64,), (4097, 40)),
          ((1088,), (512, 513)), ((31,), (1000, 384))]


def run(wl, tenants):
    from paper_2607_16074_amd import step as jstep
    model, reqs, targets = jstep.from_workload(wl)
    st = jstep.GroupStep(model, [r for r in reqs if r.tenant in tenants], targets, list(tenants))
    st.run()
    torch.cuda.synchronize()
    return st


@pytest.mark.parametrize("dims,rows", SHAPES)
def test_gradients_over_many_rows(dims, rows):
    import oracle
    print(f"widths {dims} rows {rows}", flush=True)
    d, act, chunk = 384, 3, 5
    ten = tuple(W.TenantSpec(n, 0, 1, 2, 2, (d,) + dims + (act * chunk,), act, chunk) for n in rows)
    wl = W.make_workload(W.WorkloadSpec(95, W.BackboneSpec(1, d, 3, 256, False), ten, 0, "head rows"))
    st = run(wl, range(len(rows)))
    pooled, off = st.pooled.cpu().numpy().astype(np.float64), 0

    def rel(t, ref):
        return np.linalg.norm(t.cpu().numpy().astype(np.float64) - ref) / max(np.linalg.norm(ref), 1e-30)

    for g, n in enumerate(rows):
        ref = oracle.step.tenant_from_pooled(wl, g, pooled[off: off + n])
        off += n
        io = st.ios[g]
        assert abs(float(io.loss) - ref["loss"]) <= 1e-5 * abs(ref["loss"])
        for layer, (dw, db) in enumerate(ref["grads"]):
            assert rel(io.dW[layer], dw) < 2e-5 and rel(io.db[layer], db) < 2e-5, (g, layer)
        # the order of the sums is the tenant's own
        alone = run(wl, [g]).ios[0]
        for a, b in zip(list(io.dW) + list(io.db), list(alone.dW) + list(alone.db)):
            assert torch.equal(a, b), g
