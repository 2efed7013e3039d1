"""Pack and unpack move a sample's rows as runs of 512 elements: lengths that end
just before, at and after a run, zero rows behind a sample (alignment, padded
requests), and the 4-byte form of unpack. Copies: bitwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,lens,pad,align", [
    (8, [1, 511, 512, 513, 1025], 3, 1),       # one 16-byte element per row
    (8, [1, 511, 512, 513, 700], 900, 16),     # whole runs of padding
    (768, [5, 6, 11, 16, 17], 0, 16),          # 96 per row: 5.33 rows per run
    (2048, [1, 2, 3, 64], 1, 1),               # 256 per row
    (4096, [1, 2, 33], 2, 16),
])
@pytest.mark.parametrize("row_bytes", [0, 4, 12, 2064])  # 0: the packed rows themselves
def test_runs(d, lens, pad, align, row_bytes):
    import paper_2607_16074_amd as jn
    print(f"d {d} lens {lens} pad {pad} align {align} row bytes {row_bytes}", flush=True)
    ctx, rng = jn.Context(), np.random.default_rng(d + pad)
    cut = len(lens) // 2
    reqs, host = [], []
    for t, part in enumerate((lens[:cut], lens[cut:])):
        x = rng.integers(0, 1 << 15, (len(part), max(part) + pad, d)).astype(np.int16)
        host.append(x)
        reqs.append(jn.Request(t, torch.from_numpy(x).cuda().view(torch.bfloat16), np.array(part, dtype=np.int32)))
    tenants = [jn.Tenant(7, d)] * 2
    sz = jn.jn_pack_plan(reqs, tenants, d, align)
    maps = torch.zeros(int(sz.map_bytes), dtype=torch.uint8, device="cuda")
    tokens = torch.full((int(sz.T), d), -1, dtype=torch.int16, device="cuda")
    packed = jn.jn_pack_group(ctx, reqs, tenants, d, align, maps, tokens)
    m = jn.jn_pack_maps_host(reqs, tenants, d, align)
    for name in ("token_sample", "token_pos"):
        assert np.array_equal(packed.map_tensor(name).cpu().numpy(), m[name]), name
    want = np.zeros((int(sz.T), d), np.int16)
    where = [(i, int(m["sample_request"][i]), int(m["sample_local"][i]), int(m["cu_seqlens"][i]), int(m["seqlens"][i]))
             for i in range(len(lens))]
    for _, r, s, at, n in where:
        want[at:at + n] = host[r][s, :n]
    assert np.array_equal(tokens.cpu().numpy(), want)

    rows = want.view(np.uint8) if row_bytes == 0 else rng.integers(0, 256, (int(sz.T), row_bytes), dtype=np.uint8)
    width = rows.shape[1]
    outs = [torch.full((len(x), x.shape[1], width), 255, dtype=torch.uint8, device="cuda") for x in host]
    jn.jn_unpack(ctx, packed, reqs, torch.from_numpy(rows).cuda(), width, outs)
    back = [np.zeros((len(x), x.shape[1], width), np.uint8) for x in host]
    for _, r, s, at, n in where:
        back[r][s, :n] = rows[at:at + n]
    for r, o in enumerate(outs):
        assert np.array_equal(o.cpu().numpy(), back[r]), r
