"""Weight gradients of tenants of unequal sizes, launched longest first: sizes on
both sides of the rule (the longest a quarter over the mean), the largest tenant
first, last and in between, small tiles and, for the wide expert's many tiles,
the larger ones. Materialised transposes keep the tenants' order and issue the
same MFMA sequence per output element, so every output agrees bitwise."""
import pytest

import workloads as W
from test_gpu_expert import _expert_outputs_equal, expert_spec, run_experts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SMALL, WIDE = (1, 256, 4, 512), (1, 1024, 8, 4096)


@pytest.mark.parametrize("expert,chunk,samples", [
    (SMALL, 10, (5, 3)), (SMALL, 10, (6, 3)), (SMALL, 10, (1, 7, 2)), (SMALL, 1, (1, 1, 1, 130)),
    (WIDE, 50, (9, 1, 2, 30)), (WIDE, 50, (2, 16, 4, 1, 3, 24, 5, 1))])
def test_unequal_tenants_bitwise(expert, chunk, samples):
    import paper_2607_16074_amd as jn
    from paper_2607_16074_amd import _abi
    from paper_2607_16074_amd import step as jstep
    print(f"expert {expert} chunk {chunk} samples {samples}", flush=True)
    wl = W.make_workload(expert_spec(expert, chunk, [(n, 7 + k) for k, n in enumerate(samples)]))
    st, targets, noisy = run_experts(wl)
    ctx = jn.Context()
    ctx.set_option(_abi.JN_OPT_EXPERT_TRANSPOSES, 1)
    alt = jstep.GroupStep(st.model, jstep.from_workload(wl)[1], targets, st.tenants, 1, ctx=ctx, noisy=noisy,
                          flow_t=jstep.flow_times(wl))
    alt.run()
    torch.cuda.synchronize()
    for k, g in enumerate(st.tenants):
        _expert_outputs_equal(st.ios[k], alt.ios[k], g)
