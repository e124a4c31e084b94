"""GPU: the shared-tile score passes at the edges of their configurations
(window rows per wave layout, tiles, chunks, merge of the partials) against
plain torch in float64."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def reference(K, V, Q, G, W, mr, pool):
    """score, attn, vnorm of one KV head in float64 (K, V [n, d], Q [G * W, d])."""
    n, d = K.shape
    x = (Q @ K.T) / math.sqrt(d)
    row = torch.arange(G * W, device=K.device) % W
    x.masked_fill_(torch.arange(n, device=K.device)[None] > (n - W + row)[:, None], -math.inf)
    a = torch.softmax(x, -1).sum(0) / G
    vn = V.norm(dim=-1)
    c = torch.nn.functional.pad((a * vn)[:n - mr], (pool // 2, pool // 2))
    return sum(c[i:i + n - mr] for i in range(pool)) / pool, a, vn


CASES = [  # batch, heads, group, window, d, n
    (1, 2, 1, 1, 128, 33), (1, 2, 1, 16, 128, 31), (1, 2, 1, 32, 64, 32), (1, 2, 3, 11, 128, 500),      # 32 rows
    (1, 2, 1, 33, 128, 200), (1, 3, 2, 32, 64, 1025), (1, 2, 7, 9, 128, 129),                            # 64 rows
    (1, 2, 5, 13, 128, 97), (1, 2, 4, 32, 128, 4099), (1, 2, 8, 16, 64, 4096),                           # 128 rows
    (1, 2, 3, 43, 128, 64), (1, 2, 8, 32, 128, 2047), (1, 2, 4, 64, 64, 6145), (1, 2, 8, 17, 128, 65),   # 256 rows
    (1, 2, 8, 33, 128, 300),                                                                            # general passes
    (64, 4, 1, 8, 64, 8225), (64, 4, 2, 32, 64, 8225),   # many heads (bf16: partials merged by their own kernel)
]

# Calls so large that a kernel of its own merges the partials: more than 128 tiles of 32 keys per workgroup of pass 2,
# or 64 of 64 keys with more than 128 rows.  512 workgroups share a call (fp32 at d = 64: 768; more than 128 rows: 256).
MERGED = [  # dtype, batch, heads, group, window, d, n
    ("fp32", 4, 4, 1, 32, 64, 200001), ("fp32", 4, 4, 2, 40, 64, 200001),      # 100016 tiles of 32, over 98304
    ("fp32", 4, 4, 2, 32, 128, 131300), ("fp32", 2, 8, 4, 32, 128, 131300),    # 65664 tiles, over 65536
    ("bf16", 4, 4, 4, 32, 128, 131300), ("bf16", 4, 4, 1, 16, 64, 131300),
    ("bf16", 1, 4, 8, 32, 64, 262400), ("bf16", 1, 4, 4, 64, 128, 262399),     # 256 rows: 16400 tiles of 64, over 16384
    ("fp32", 1, 4, 8, 32, 64, 262400), ("fp32", 1, 4, 3, 50, 128, 262399),
    ("bf16", 2, 4, 1, 32, 64, 525000),   # 131256 tiles: pass 1 too leaves one round of workgroups for short chunks
]


def check_scores(case, dtype, heads_checked):
    from paper_2607_16213_amd import selkv as S
    B, H, G, W, d, n = case
    gen = torch.Generator(device="cuda").manual_seed(n * 1000 + G * W)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").div_(math.sqrt(d) / 2).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    K, V, Q = rnd(B, H, n, d), rnd(B, H, n, d), rnd(B, H * G, W, d)
    p = S.params(batch=B, n_heads_kv=H, group=G, head_dim=d, seq_len=n, window=W, kv_dtype=dtype, scale=0.0)
    m, mr, _ = S.budget(p)
    nan = float("nan")
    score = torch.full((B, H, n - mr), nan, device="cuda")
    attn, vnorm = torch.full((B, H, n), nan, device="cuda"), torch.full((B, H, n), nan, device="cuda")
    S.score(p, K, V, Q, score, attn, vnorm, S.workspace(p, S.CALL_SCORE, "cuda"))
    for b, h in heads_checked:
        rs, ra, rv = reference(K[b, h].double(), V[b, h].double(), Q[b].reshape(H, G * W, d)[h].double(), G, W, mr,
                               p.pool_kernel)
        # logits stay below 4, so their fp32 sums of d products carry a few 1e-7 into the exponent; the
        # G * W <= 264 addends of a column add as much again: 3e-6 relative covers each output
        for name, got, ref in (("attn", attn[b, h], ra), ("vnorm", vnorm[b, h], rv), ("score", score[b, h], rs)):
            err = ((got.double() - ref).abs() / ref.clamp_min(1e-30)).max().item() if ref.numel() else 0.0
            assert err < 3e-6, (name, b, h, err)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("case", CASES, ids=["b%d_h%d_g%d_w%d_d%d_n%d" % c for c in CASES])
def test_shared_tile_scores(case, dtype):
    B, H = case[:2]
    check_scores(case, dtype, [(b, h) for b in sorted({0, B // 2, B - 1}) for h in range(H)])


@pytest.mark.parametrize("case", MERGED, ids=["%s_b%d_h%d_g%d_w%d_d%d_n%d" % c for c in MERGED])
def test_scores_of_calls_that_merge_their_partials_first(case):
    B, H = case[1:3]
    check_scores(case[1:], case[0], [(0, 0), (B // 2, H // 2), (B - 1, H - 1)])
