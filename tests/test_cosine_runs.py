"""GPU: the bf16 all-pairs match with the kept range split into runs of few
tiles and with runs past the last tile, against torch in float64."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,n,rho", [(1, 300, 0.25), (1, 520, 0.5), (2, 2000, 0.25), (1, 2700, 0.5), (1, 4500, 0.3),
                                         (8, 1100, 0.25), (3, 9000, 0.1), (40, 700, 0.4)])
def test_match_runs(heads, n, rho):
    from paper_2607_16213_amd import selkv as S
    d = 128
    gen = torch.Generator(device="cuda").manual_seed(n + heads)
    p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=d, seq_len=n, window=1, kv_dtype="bf16",
                 budget_ratio=rho, route_mode="full_cosine")
    m, mr, ms = S.budget(p)
    V = torch.randn((1, heads, n, d), generator=gen, device="cuda").bfloat16()
    perm = torch.rand((1, heads, n), generator=gen, device="cuda").argsort(-1)
    kept, ev = perm[..., :m].sort(-1).values.int().contiguous(), perm[..., m:].sort(-1).values.int().contiguous()
    attn = torch.rand((1, heads, n), generator=gen, device="cuda") + 0.1
    vnorm = V.float().norm(dim=-1)
    o = dict(K_out=torch.empty((1, heads, m, d), dtype=torch.bfloat16, device="cuda"))
    o["V_out"] = torch.empty_like(o["K_out"])
    target = torch.full((1, heads, n - m), -9, dtype=torch.int32, device="cuda")
    gate, bias = torch.empty((1, heads, n - m), device="cuda"), torch.empty((1, heads, m), device="cuda")
    ws = torch.randint(0, 256, (S.workspace_bytes(p, S.CALL_MERGE_BIAS),), dtype=torch.uint8, device="cuda")
    S.merge_bias(p, V, V, attn, vnorm, kept, ev, o["K_out"], o["V_out"], target, gate, bias, ws)
    for h in range(heads):
        u = V[0, h].double()
        u = u / u.norm(dim=-1, keepdim=True)
        cos = u[ev[0, h].long()] @ u[kept[0, h].long()].T
        best = cos.max(1).values
        t = target[0, h].long()
        assert ((t >= 0) & (t < m)).all(), h
        # the chosen slot's cosine is the largest up to fp32 rounding of a sum of d products of unit-norm rows
        assert (best - cos.gather(1, t[:, None])[:, 0]).max().item() < 1e-6, h
        assert (gate[0, h].double() - best.clamp(0, 1)).abs().max().item() < 2e-6, h
