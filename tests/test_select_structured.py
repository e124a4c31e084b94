"""GPU: selection where the scores have structure along the sequence or defeat
the sample that places the band."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def check(p, x, name):
    """selkv.select on the scores x [heads, n_cand] against a stable sort."""
    from paper_2607_16213_amd import selkv as S
    m, mr, ms = S.budget(p)
    heads, n = p.n_heads_kv, p.seq_len
    kept = torch.full((1, heads, m), -7, dtype=torch.int32, device="cuda")
    ev = torch.full((1, heads, n - m), -7, dtype=torch.int32, device="cuda")
    S.select(p, torch.from_numpy(x)[None].cuda(), kept, ev)
    kept, ev = kept[0].cpu().numpy(), ev[0].cpu().numpy()
    for h in range(heads):
        order = np.argsort(-x[h], kind="stable")[:ms]         # equal scores: the lower position first
        mask = np.zeros(n, bool)
        mask[order] = True
        mask[n - mr:] = True
        assert np.array_equal(kept[h], np.nonzero(mask)[0]), (name, h)
        assert np.array_equal(ev[h], np.nonzero(~mask)[0]), (name, h)


# the sample takes 4096 evenly spaced scores of heads too long to stage whole; here all of them are -inf
@pytest.mark.parametrize("keep", ["fewer_finite", "more_finite"])
@pytest.mark.parametrize("heads,n", [(1, 24700), (8, 32768), (3, 102400), (130, 40000)])
def test_sample_without_a_finite_score(heads, n, keep):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=64, seq_len=n, window=1,
                 budget_ratio=0.25 if keep == "fewer_finite" else 51.0 / n)
    n_cand = n - S.budget(p)[1]
    rng = np.random.default_rng(n)
    x = rng.random((heads, n_cand)).astype(np.float32)
    x[rng.random((heads, n_cand)) < 0.9] = -np.inf
    x[:, np.arange(4096) * n_cand // 4096] = -np.inf
    assert np.isfinite(x).sum(1).min() > 35
    check(p, x, keep)
