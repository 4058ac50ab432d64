"""bf16 scores whose products have so few tiles that k is cut into parts: against the same formulas in fp64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


@pytest.mark.parametrize("weights", ["qk", "q", "k", ""])
@pytest.mark.parametrize("B,N,d,T", [(1, 300, 1024, 16), (2, 130, 2048, 5), (1, 64, 512, 1), (1, 700, 1536, 33), (3, 90, 520, 2)],
                         ids=["four-parts", "batch-odd-keywords", "one-keyword", "two-tiles", "width-not-cut"])
@pytest.mark.parametrize("mode", ["cosine", "softmax"])
def test_scores_with_k_in_parts(C, mode, B, N, d, T, weights):
    import torch
    g = torch.Generator().manual_seed(N + T)
    X, Q = torch.randn(B, N, d, generator=g).bfloat16().cuda(), torch.randn(B, T, d, generator=g).bfloat16().cuda()
    Wq, Wk = (torch.randn(2, d, d, generator=g) / d ** 0.5).bfloat16().cuda()
    Wq, Wk = Wq if "q" in weights else None, Wk if "k" in weights else None
    H = 2 if d % 8 == 0 else 1
    p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=H, dtype=C.BF16, keep_k=4, preselect_m=8, rank_r=2,
                 rel_mode=C.REL_COSINE_MAX if mode == "cosine" else C.REL_ATTN_SOFTMAX)
    got = C.score(p, X, None, Q, Wq, Wk)[0].double().cpu()
    v, q = X.double().cpu(), Q.double().cpu()
    v = v @ Wk.double().cpu() if Wk is not None else v
    q = q @ Wq.double().cpu() if Wq is not None else q
    if mode == "cosine":
        ref = (torch.nn.functional.normalize(v, dim=-1) @ torch.nn.functional.normalize(q, dim=-1).transpose(1, 2)).amax(2)
        # fp32 sums of d products: a rounding of 2^-24 per addition, adding up like a random walk, four times over
        assert (got - ref).abs().max() < 4 * d ** 0.5 * 2 ** -24
    else:
        dh = d // H
        ref = sum(torch.softmax(q[..., a:a + dh] @ v[..., a:a + dh].transpose(1, 2) / dh ** 0.5, 2).mean(1) for a in range(0, d, dh)) / H
        # the same error in a logit of size up to ~ sqrt(dh) (unscaled ~ dh), relative in a probability
        assert ((got - ref).abs() / ref).max() < 4 * d ** 0.5 * 2 ** -24 * max(1.0, dh ** 0.5)
