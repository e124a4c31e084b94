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
@pytest.mark.parametrize("heads,n", [(1, 9000), (1, 24700), (8, 32768), (3, 102400), (130, 40000)])
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


def sorted_keys(x):
    """Order keys of fp32 scores: as the scores, -0 equal to +0, NaN beyond the infinity of its sign."""
    u = x.view(np.uint32).copy()
    u[u == 0x80000000] = 0
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.int64)


# heads that leave the column path (NaN; more candidates than the columns take; many equal scores), shared between
# several workgroups and not
@pytest.mark.parametrize("kind", ["nan", "some_nan", "plateau", "iid"])
@pytest.mark.parametrize("heads,n", [(1, 2049), (8, 8208), (8, 8209), (9, 24593), (1, 102400), (130, 33000), (300, 5000), (1, 131089),
                                     (2, 300017), (1, 1000003)])
def test_whole_head_path(heads, n, kind):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=64, seq_len=n, window=1)
    m, mr, ms = S.budget(p)
    rng = np.random.default_rng(n + heads)
    x = np.exp(0.7 * rng.standard_normal((heads, n - mr))).astype(np.float32)
    if kind == "nan":
        x[:, (n - mr) // 2] = np.nan
        x[:, 5] = -np.float32(np.nan)
    elif kind == "some_nan":                     # heads of one call go different ways
        x[::2, ::777] = np.nan
    elif kind == "plateau":
        x[x < 1.8] = 0.0
    kept = torch.full((1, heads, m), -7, dtype=torch.int32, device="cuda")
    ev = torch.full((1, heads, n - m), -7, dtype=torch.int32, device="cuda")
    S.select(p, torch.from_numpy(x)[None].cuda(), kept, ev)
    kept, ev = kept[0].cpu().numpy(), ev[0].cpu().numpy()
    for h in range(heads):
        mask = np.zeros(n, bool)
        mask[np.argsort(-sorted_keys(x[h]), kind="stable")[:ms]] = True
        mask[n - mr:] = True
        assert np.array_equal(kept[h], np.nonzero(mask)[0]), h
        assert np.array_equal(ev[h], np.nonzero(~mask)[0]), h


def union_lists(x, ms):
    """The union rule for one cache: x [heads, n_cand] -> mask of the shared picks."""
    heads, n_cand = x.shape
    union = np.zeros(n_cand, bool)
    mean = np.zeros(n_cand, np.float32)
    for h in range(heads):
        union[np.argsort(-x[h], kind="stable")[:ms]] = True
        mean = mean + x[h]                       # the fp32 sum in head order, divided by the heads
    mask = np.zeros(n_cand, bool)
    mask[np.argsort(-np.where(union, mean / np.float32(heads), -np.inf), kind="stable")[:ms]] = True
    return mask


@pytest.mark.parametrize("kind", ["iid", "plateau"])
@pytest.mark.parametrize("batch,heads,n", [(1, 8, 140016), (2, 3, 131089), (1, 8, 102400), (1, 40, 5000), (40, 8, 1100)])
def test_union_whole_head_path(batch, heads, n, kind):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=batch, n_heads_kv=heads, group=2, head_dim=64, seq_len=n, window=1, select_mode="union")
    m, mr, ms = S.budget(p)
    rng = np.random.default_rng(n)
    x = np.exp(0.5 * rng.standard_normal((batch, heads, n - mr))).astype(np.float32)
    if kind == "plateau":
        x[x < 1.5] = 0.0
    kept = torch.full((batch, heads, m), -7, dtype=torch.int32, device="cuda")
    ev = torch.full((batch, heads, n - m), -7, dtype=torch.int32, device="cuda")
    S.select(p, torch.from_numpy(x).cuda(), kept, ev, S.workspace(p, S.CALL_SELECT, "cuda"))
    for b in range(batch):
        mask = np.ones(n, bool)
        mask[:n - mr] = union_lists(x[b], ms)
        want = torch.from_numpy(np.nonzero(mask)[0].astype(np.int32)).cuda()
        rest = torch.from_numpy(np.nonzero(~mask)[0].astype(np.int32)).cuda()
        assert bool((kept[b] == want).all()) and bool((ev[b] == rest).all()), b


def call_us(p, x):
    """Median time of a selkv.select call on the scores x [batch, heads, n_cand]."""
    from paper_2607_16213_amd import selkv as S
    m = S.budget(p)[0]
    kept = torch.empty((p.batch, p.n_heads_kv, m), dtype=torch.int32, device="cuda")
    ev = torch.empty((p.batch, p.n_heads_kv, p.seq_len - m), dtype=torch.int32, device="cuda")
    ws = S.workspace(p, S.CALL_SELECT, "cuda")
    times = []
    for i in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            S.select(p, x, kept, ev, ws)
        b.record()
        b.synchronize()
        if i:
            times.append(a.elapsed_time(b) * 100.0)
    return sorted(times)[len(times) // 2]


def test_union_of_a_long_cache_costs_what_its_lists_do():
    # 140000 candidates pass the columns' 131072; the same call with 1% fewer than those stays inside.  Writing the
    # eight heads' lists entry by entry from one workgroup made the longer call 12 times the shorter; 1.8 measured now
    from paper_2607_16213_amd import selkv as S
    gen = torch.Generator(device="cuda").manual_seed(3)
    us = []
    for n in (129800, 140016):
        p = S.params(batch=1, n_heads_kv=8, group=2, head_dim=64, seq_len=n, window=1, select_mode="union")
        x = torch.randn((1, 8, n - 16), generator=gen, device="cuda").mul_(0.7).exp_()
        us.append(call_us(p, x))
    assert us[1] < 5 * us[0], us


def shaped(kind, shape, gen):
    """Positive scores with a course along the sequence."""
    z = torch.randn(shape, generator=gen, device="cuda")
    t = torch.arange(shape[-1], device="cuda") / shape[-1]
    if kind == "iid":
        return (0.7 * z).exp()
    if kind == "grow2":
        return (0.3 * z + 0.693 * t).exp()
    if kind == "grow10":
        return (0.3 * z + 2.303 * t).exp()
    if kind == "fall":                           # every score above the next
        return (2.0 - t).expand(shape).contiguous()
    level = torch.randn(shape[:-1] + (24,), generator=gen, device="cuda")      # 24 passages of their own level
    return (0.3 * z + level.repeat_interleave(shape[-1] // 24 + 1, -1)[..., :shape[-1]]).exp()


@pytest.mark.parametrize("kind", ["grow2", "grow10", "fall", "passages"])
@pytest.mark.parametrize("heads,n", [(2, 8208), (2, 8209), (40, 9001), (2, 16400), (2, 24591), (2, 24593), (3, 40001), (1, 65552), (8, 102400), (2, 131088), (300, 26000)])
def test_scores_with_a_course(heads, n, kind):
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=1, n_heads_kv=heads, group=1, head_dim=64, seq_len=n, window=1)
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = shaped(kind, (heads, n - S.budget(p)[1]), gen)
    check(p, x.cpu().numpy(), kind)


def test_scores_with_a_course_cost_no_more():
    # the band's scores spread over all columns wherever they lie: 27 - 28 us for every kind; the columns of one wave
    # used to take those of a passage, and a full one cost 6.5 times as much
    from paper_2607_16213_amd import selkv as S
    p = S.params(batch=1, n_heads_kv=8, group=1, head_dim=64, seq_len=102400, window=1)
    gen = torch.Generator(device="cuda").manual_seed(4)
    us = {k: call_us(p, shaped(k, (1, 8, 102384), gen)) for k in ("iid", "grow2", "grow10", "fall", "passages")}
    assert max(us.values()) < 2 * us["iid"], us
