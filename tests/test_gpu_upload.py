"""Host tables on the device: small ones by a kernel that reads the pinned
staging buffer, ones above 64 KB by a copy.  Packs back to back, each with
other lengths, so that every staging buffer is rewritten while earlier packs
are still queued; the maps are whole numbers and equal the host's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5, 2300, 2345, 2500])  # 28 bytes of tables per sample: 64 KB lie at 2,339
def test_tables_arrive(n):
    import paper_2607_16074_amd as jn
    print(f"samples {n}", flush=True)
    ctx, d, rng = jn.Context(), 8, np.random.default_rng(n)
    tenants = [jn.Tenant(7, d)]
    embeds = torch.ones((n, 4, d), dtype=torch.bfloat16, device="cuda")
    runs = []
    for _ in range(12):
        reqs = [jn.Request(0, embeds, rng.integers(1, 5, n))]
        sz = jn.jn_pack_plan(reqs, tenants, d, 1)
        maps = torch.zeros(int(sz.map_bytes), dtype=torch.uint8, device="cuda")
        tokens = torch.zeros((int(sz.T), d), dtype=torch.bfloat16, device="cuda")
        runs.append((jn.jn_pack_group(ctx, reqs, tenants, d, 1, maps, tokens),
                     jn.jn_pack_maps_host(reqs, tenants, d), tokens))
    torch.cuda.synchronize()
    for packed, host, tokens in runs:
        for name in ("seqlens", "cu_seqlens", "sample_request", "sample_local", "tenant_perm", "sample_tenant_rank",
                     "token_sample", "token_pos"):
            assert np.array_equal(packed.map_tensor(name).cpu().numpy(), host[name]), name
        assert bool((tokens == 1).all())  # read through the request table
