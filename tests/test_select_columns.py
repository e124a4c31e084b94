"""GPU: selection against a stable sort, at the sizes where the kernel changes
its split over workgroups, its staging or its path, and for scores that force
the whole-head path."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIZES = [(1, 17), (3, 79), (2, 80), (2, 81), (5, 1040), (8, 2063), (8, 4113), (8, 8192), (1, 20496), (8, 20497), (9, 24593),
         (130, 1600), (300, 700), (40, 32768), (8, 102400), (2, 131088), (2, 131089), (1, 300017)]
KINDS = ["lognormal", "ties", "equal", "negative", "minus_inf", "few_finite", "clumped", "denormal", "zeros"]


def scores(kind, heads, n, ms, rng):
    x = np.exp(0.7 * rng.standard_normal((heads, n))).astype(np.float32)
    if kind == "ties":
        x = np.round(x * 4).astype(np.float32)
    elif kind == "equal":
        x[:] = 0.5
    elif kind == "negative":
        x = rng.standard_normal((heads, n)).astype(np.float32)
    elif kind == "minus_inf":          # as the union's second selection sees it
        x[rng.random((heads, n)) < 0.6] = -np.inf
    elif kind == "few_finite":         # fewer than ms above -inf
        x[:, max(ms - 3, 0):] = -np.inf
    elif kind == "clumped":            # the band's scores all in a few columns of one wave
        x = np.where(np.arange(n) % 64 < 2, 1.0 + 1e-6 * rng.random((heads, n)), rng.random((heads, n)) * 0.5).astype(np.float32)
    elif kind == "denormal":
        x = (rng.integers(0, 1 << 22, (heads, n)).astype(np.uint32)).view(np.float32)
    elif kind == "zeros":              # +0 and -0 are equal scores
        x = np.where(rng.random((heads, n)) < 0.5, np.float32(0.0), np.float32(-0.0))
        x[:, ::7] = 1e-3
    return x


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads,n", SIZES)
def test_select_matches_stable_sort(heads, n, kind):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=64, seq_len=n, window=1, kv_dtype="bf16",
                 budget_ratio=0.25 if n > 100 else 0.9)
    m, mr, ms = S.budget(p)
    rng = np.random.default_rng(n * 31 + heads)
    x = scores(kind, heads, n - mr, ms, rng)
    kept = torch.full((1, heads, m), -7, dtype=torch.int32, device="cuda")
    ev = torch.full((1, heads, n - m), -7, dtype=torch.int32, device="cuda")
    S.select(p, torch.from_numpy(x)[None].cuda(), kept, ev)
    kept, ev = kept[0].cpu().numpy(), ev[0].cpu().numpy()
    for h in range(heads):
        order = np.argsort(-x[h], kind="stable")[:ms]         # equal scores: the lower position first
        mask = np.zeros(n, bool)
        mask[order] = True
        mask[n - mr:] = True
        assert np.array_equal(kept[h], np.nonzero(mask)[0]), h
        assert np.array_equal(ev[h], np.nonzero(~mask)[0]), h


@pytest.mark.parametrize("batch,heads,n", [(1, 8, 8192), (3, 2, 1000), (1, 8, 102400), (4, 8, 20500), (1, 3, 140000)])
def test_union_select_matches_numpy(batch, heads, n):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=batch, n_heads_kv=heads, group=2, head_dim=64, seq_len=n, window=1, select_mode="union")
    m, mr, ms = S.budget(p)
    rng = np.random.default_rng(n + batch)
    x = np.exp(0.5 * rng.standard_normal((batch, heads, n - mr))).astype(np.float32)
    x[:, :, ::5] = np.round(x[:, :, ::5] * 8) / 8
    kept = torch.full((batch, heads, m), -7, dtype=torch.int32, device="cuda")
    ev = torch.full((batch, heads, n - m), -7, dtype=torch.int32, device="cuda")
    ws = torch.randint(0, 256, (S.workspace_bytes(p, S.CALL_SELECT),), dtype=torch.uint8, device="cuda")
    S.select(p, torch.from_numpy(x).cuda(), kept, ev, ws)
    for b in range(batch):
        union = np.zeros(n - mr, bool)
        mean = np.zeros(n - mr, np.float32)
        for h in range(heads):
            union[np.argsort(-x[b, h], kind="stable")[:ms]] = True
            mean = mean + x[b, h]                             # the fp32 sum in head order, divided by the heads
        key = np.where(union, mean / np.float32(heads), -np.inf)
        mask = np.zeros(n, bool)
        mask[np.argsort(-key, kind="stable")[:ms]] = True
        mask[n - mr:] = True
        for h in range(heads):
            assert np.array_equal(kept[b, h].cpu().numpy(), np.nonzero(mask)[0]), (b, h)
            assert np.array_equal(ev[b, h].cpu().numpy(), np.nonzero(~mask)[0]), (b, h)
