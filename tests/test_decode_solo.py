"""GPU: decode steps on either side of the lengths where one workgroup takes a
head by itself, against torch in float64."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

LENGTHS = [1, 16, 31, 64, 127, 128, 129, 255, 256, 257, 300, 511, 512, 513, 1000]


@pytest.mark.parametrize("append", [False, True], ids=["fixed", "append"])
@pytest.mark.parametrize("dtype,tol", [("bf16", 2e-6), ("fp32", 2e-6)])
@pytest.mark.parametrize("heads,G,d", [(2, 1, 128), (8, 4, 64), (3, 8, 128), (70, 2, 64), (300, 3, 128)])
def test_decode_lengths(heads, G, d, dtype, tol, append):
    # tol: relative 2-norm per query head.  fp32 logits of d products and the running softmax carry a few 1e-7
    # (measured at most 3e-7); the output is fp32 whatever the cache's type
    from paper_2607_16213_amd import selkv as S
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(heads * 1000 + d)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(dt)
    p = S.params(batch=1, n_heads_kv=heads, group=G, head_dim=d, kv_dtype=dtype)
    for L in LENGTHS:
        cap = L + 3
        K, V, q = rnd(1, heads, cap, d), rnd(1, heads, cap, d), rnd(1, heads * G, d)
        bias = torch.rand((1, heads, cap), generator=gen, device="cuda")
        out = torch.full((1, heads * G, d), float("nan"), device="cuda")
        ws = torch.randint(0, 256, (S.workspace_bytes(p, S.CALL_DECODE, cap),), dtype=torch.uint8, device="cuda")
        if append:
            kn, vn = rnd(1, heads, d), rnd(1, heads, d)
            Kr, Vr, br = K.clone(), V.clone(), bias.clone()
            Kr[:, :, L - 1], Vr[:, :, L - 1], br[:, :, L - 1] = kn, vn, 0
            S.decode_append(p, q, kn, vn, K, V, bias, L - 1, out, ws)
            assert torch.equal(K, Kr) and torch.equal(V, Vr) and torch.equal(bias, br), L
        else:
            K, V, bias = K[:, :, :L].contiguous(), V[:, :, :L].contiguous(), bias[:, :, :L].contiguous()
            S.decode_attn(p, q, K, V, bias, out, ws)
        x = torch.matmul(q.double().view(heads, G, d), K[0, :, :L].double().transpose(1, 2).contiguous()) / math.sqrt(d)
        w = torch.softmax(x + bias[0, :, None, :L].double(), -1)
        ref = torch.matmul(w, V[0, :, :L].double()).view(heads * G, d)
        err = ((out[0].double() - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item()
        assert err < tol, (L, err)
