"""GPU: the merge that finds its own bucket offsets (calls of few buckets)
against the one that reads them from the offsets kernel (the same head among
many), bit for bit."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", ["bucket", "bucket_nearest"])
@pytest.mark.parametrize("n,B,rho,lump", [(33, 32, 0.5, False), (100, 1, 0.3, False), (257, 64, 1.0, False),
                                          (1025, 32, 0.25, True), (4100, 64, 0.9, False), (9000, 3, 0.25, False),
                                          (120000, 64, 0.9, True), (120000, 32, 0.02, True)])
def test_offsets_found_in_the_merge(n, B, rho, lump, route):
    from paper_2607_16213_amd import selkv as S
    d = 64
    gen = torch.Generator(device="cuda").manual_seed(n + B)
    m = int(rho * n)
    key = torch.rand((n,), generator=gen, device="cuda")
    if lump:                       # runs of buckets that keep everything, and runs that keep nothing
        key = key * 0.1 + (torch.arange(n, device="cuda") // 700 % 3 == 0)
    order = key.argsort(descending=True)
    kept, ev = order[:m].sort().values.int(), order[m:].sort().values.int()
    V = torch.randn((n, d), generator=gen, device="cuda").bfloat16()
    K = torch.randn((n, d), generator=gen, device="cuda").bfloat16()
    attn = torch.rand((n,), generator=gen, device="cuda") + 0.1
    nb = (n + B - 1) // B
    outs = []
    for heads in (1, 4097 // nb + 2):
        if heads == 1 and nb > 4096:
            continue
        p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=d, seq_len=n, window=1, kv_dtype="bf16",
                     budget_ratio=rho, bucket=B, route_mode=route)
        assert S.budget(p)[0] == m
        rep = lambda x: x[None, None].expand(1, heads, *x.shape).contiguous()
        o = [torch.empty((1, heads, m, d), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        o += [torch.full((1, heads, n - m), -9, dtype=torch.int32, device="cuda"),
              torch.full((1, heads, n - m), -9.0, device="cuda"), torch.full((1, heads, m), -9.0, device="cuda")]
        ws = torch.randint(0, 256, (S.workspace_bytes(p, S.CALL_MERGE_BIAS),), dtype=torch.uint8, device="cuda")
        S.merge_bias(p, rep(K), rep(V), rep(attn), rep(V.float().norm(dim=-1)), rep(kept), rep(ev), *o, ws)
        outs.append([x[0, -1].cpu() for x in o])
    assert len(outs) == 2 and all(torch.equal(x, y) for x, y in zip(*outs))
    t = outs[0][2].long()
    routed = t >= 0
    assert (t < m).all() and (route == "bucket_nearest") <= bool(routed.all())
    if route == "bucket":          # a routed token's target lies in its bucket
        assert torch.equal(kept.cpu().long()[t[routed]] // B, ev.cpu().long()[routed] // B)
