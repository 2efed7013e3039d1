"""Few long samples among many short ones: pack, unpack and the experts' prefix
copy then walk the packed rows, the requests or the prefix rows instead of as many
workgroups for every sample.  Rows of one 16-byte element, rows that end inside a
workgroup's 512 elements and rows of whole ones; padding, alignment rows, the 4-byte
form of unpack.  Copies: bitwise, against the host's maps."""
import numpy as np
import pytest

import workloads as W
from test_gpu_expert import _expert_outputs_equal, run_experts

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GROUPS = [  # (lengths, padded length) per request
    [([1] * 300, 1), ([700], 701), ([2, 1, 3] * 40, 3)],
    [([5000], 5000), ([1] * 999, 2)],
    [([100] * 40, 103), ([600], 600), ([1, 30], 33)],  # the longest goes round its blocks several times
    [([5] * 90 + [600], 600), ([1], 1)],  # one request: the padding is as long as its rows
    [([17, 16, 15] * 30, 20), ([1030, 1], 1031), ([33] * 50, 34), ([900], 900)],
]


@pytest.mark.parametrize("group", range(len(GROUPS)))
@pytest.mark.parametrize("d,align", [(8, 1), (8, 16), (768, 1), (768, 4), (2048, 1), (1160, 16)])
def test_copies(group, d, align):
    import paper_2607_16074_amd as jn
    print(f"group {group} d {d} align {align}", flush=True)
    ctx, rng = jn.Context(), np.random.default_rng(group)
    host = [rng.integers(0, 1 << 15, (len(x), m, d)).astype(np.int16) for x, m in GROUPS[group]]
    reqs = [jn.Request(0, torch.from_numpy(h).cuda().view(torch.bfloat16), np.array(x, np.int32))
            for h, (x, _) in zip(host, GROUPS[group])]
    tenants = [jn.Tenant(7, d)]
    sz = jn.jn_pack_plan(reqs, tenants, d, align)
    maps = torch.zeros(int(sz.map_bytes), dtype=torch.uint8, device="cuda")
    tokens = torch.full((int(sz.T) + 1, d), -1, dtype=torch.int16, device="cuda")
    packed = jn.jn_pack_group(ctx, reqs, tenants, d, align, maps, tokens[:-1])
    m = jn.jn_pack_maps_host(reqs, tenants, d, align)
    for name in ("token_sample", "token_pos"):
        assert np.array_equal(packed.map_tensor(name).cpu().numpy(), m[name]), name
    want = np.zeros((int(sz.T), d), np.int16)
    where = list(zip(m["sample_request"], m["sample_local"], m["cu_seqlens"], m["seqlens"]))
    for r, s, at, n in where:
        want[at:at + n] = host[r][s, :n]
    assert np.array_equal(tokens[:-1].cpu().numpy(), want) and bool((tokens[-1] == -1).all())
    for width in (d * 2, 12):
        rows = want.view(np.uint8) if width == d * 2 else rng.integers(0, 256, (int(sz.T), width), dtype=np.uint8)
        outs = [torch.full((h.shape[0], h.shape[1], width), 255, dtype=torch.uint8, device="cuda") for h in host]
        jn.jn_unpack(ctx, packed, reqs, torch.from_numpy(rows).cuda(), width, outs)
        back = [np.zeros((h.shape[0], h.shape[1], width), np.uint8) for h in host]
        for r, s, at, n in where:
            back[r][s, :n] = rows[at:at + n]
        for r, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy(), back[r]), (width, r)


@pytest.mark.parametrize("samples", [64, 65])  # 256 MB are plain stores' last, 65 samples beyond
def test_copies_around_the_last_level_cache(samples):
    import paper_2607_16074_amd as jn
    print(f"samples {samples}", flush=True)
    ctx, d, rows = jn.Context(), 2048, 1024
    x = torch.randint(-32768, 32767, (samples, rows, d), dtype=torch.int16, device="cuda")
    lens = np.arange(rows, rows - samples, -1, dtype=np.int32)
    for i, n in enumerate(lens):
        x[i, n:] = 0
    reqs, tenants = [jn.Request(0, x.view(torch.bfloat16), lens)], [jn.Tenant(7, d)]
    sz = jn.jn_pack_plan(reqs, tenants, d, rows)  # aligned: every sample's rows and zeros
    maps = torch.zeros(int(sz.map_bytes), dtype=torch.uint8, device="cuda")
    tokens = torch.full((int(sz.T), d), -1, dtype=torch.int16, device="cuda")
    packed = jn.jn_pack_group(ctx, reqs, tenants, d, rows, maps, tokens)
    assert torch.equal(tokens.view_as(x), x)
    out = torch.full_like(x, -1)
    jn.jn_unpack(ctx, packed, reqs, tokens, d * 2, [out])
    assert torch.equal(out, x)


def test_expert_prefix_of_unlike_lengths():
    """Each tenant's own samples are alike, the group's are not: the same bits."""
    from paper_2607_16074_amd import step as jstep
    ten = tuple(W.TenantSpec(n, 0, lo, lo, lo, (128, 64, 12), 3, 4, expert=(1, 256, 4, 512))
                for n, lo in ((60, 2), (1, 640), (30, 3)))
    wl = W.make_workload(W.WorkloadSpec(94, W.BackboneSpec(1, 128, 4, 256, False), ten, 0, "unlike lengths"))
    full, targets, noisy = run_experts(wl)
    reqs = jstep.from_workload(wl)[1]
    for g in range(3):
        print(f"tenant {g}", flush=True)
        alone = jstep.GroupStep(full.model, [r for r in reqs if r.tenant == g], targets, [g], 1, noisy=noisy)
        alone.run()
        torch.cuda.synchronize()
        _expert_outputs_equal(full.ios[g], alone.ios[0], g)
