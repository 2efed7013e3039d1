"""Data and weight gradients of an expert layer in one launch: row counts
around the 96-row data-gradient tile and the 64-row slab, and weight gradients
of exactly and of more than two rounds of tiles (512: pair; 768: two launches).
Materialised transposes never run as a pair and issue the same MFMA sequence
per output element, so every output agrees bitwise."""
import pytest

import workloads as W
from test_gpu_expert import _expert_outputs_equal, expert_spec, run_experts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SMALL, WIDE = (1, 256, 4, 512), (1, 1024, 8, 4096)


@pytest.mark.parametrize("expert,chunk,samples", [
    (SMALL, 1, (1,)), (SMALL, 1, (96, 97)), (SMALL, 5, (19, 1)), (SMALL, 64, (1, 2, 3)), (SMALL, 13, (5, 15)),
    (WIDE, 7, (3, 2)), (WIDE, 9, (1, 2, 1))])
def test_paired_gradients_bitwise(expert, chunk, samples):
    import paper_2607_16074_amd as jn
    from paper_2607_16074_amd import _abi
    from paper_2607_16074_amd import step as jstep
    print(f"expert {expert} chunk {chunk} samples {samples}", flush=True)
    wl = W.make_workload(expert_spec(expert, chunk, [(n, 7) for n in samples]))
    st, targets, noisy = run_experts(wl)
    ctx = jn.Context()
    ctx.set_option(_abi.JN_OPT_EXPERT_TRANSPOSES, 1)
    alt = jstep.GroupStep(st.model, jstep.from_workload(wl)[1], targets, st.tenants, 1, ctx=ctx, noisy=noisy,
                          flow_t=jstep.flow_times(wl))
    alt.run()
    torch.cuda.synchronize()
    for k, g in enumerate(st.tenants):
        _expert_outputs_equal(st.ios[k], alt.ios[k], g)
