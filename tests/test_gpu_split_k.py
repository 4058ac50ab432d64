"""bf16 scores and Gram matrices of few tiles (smaller tiles than those of large products): against the same formulas in fp64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


@pytest.mark.parametrize("weights", ["qk", "q", "k", ""])
@pytest.mark.parametrize("B,N,d,T", [(1, 300, 1024, 16), (2, 130, 2048, 5), (1, 64, 512, 1), (1, 700, 1536, 33), (3, 90, 520, 2), (2, 200, 544, 3)],
                         ids=["two-row-tiles", "batch-odd-keywords", "one-keyword", "two-tiles", "width-not-64", "width-32"])
@pytest.mark.parametrize("mode", ["cosine", "softmax"])
def test_scores_of_few_tiles(C, mode, B, N, d, T, weights):
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


@pytest.mark.parametrize("B,N,M,d", [(1, 40, 33, 256), (3, 200, 129, 320), (1, 400, 288, 1088), (2, 600, 600, 512)],
                         ids=["remainder-tiles", "five-steps-over-four-waves", "one-image", "more-tiles"])
def test_gram_matrix_of_few_tiles(C, B, N, M, d):
    """The energies of rank M - 1 ... of the pre-selected rows sum to nearly the trace of their Gram matrix, row by row |z_i|^2
    less the last eigenpair's part: compared with the fp64 eigen-decomposition."""
    import torch
    g = torch.Generator().manual_seed(M)
    scale = 0.97 ** torch.arange(d, dtype=torch.float32)
    X = (torch.randn(B, N, d, generator=g) * scale).bfloat16().cuda()
    s = torch.rand(B, N, generator=g).cuda()
    r = min(20, M // 2)
    p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=1, dtype=C.BF16, keep_k=8, preselect_m=M, rank_r=r)
    out = C.select(p, X, s)
    for b in range(B):
        rows = out["idx_m"][b].long()
        Z = X[b][rows].double().cpu()
        lam, V = torch.linalg.eigh(Z @ Z.t())
        ref = (V[:, -r:] ** 2 * lam[-r:]).sum(1)
        err = (out["c"][b].double().cpu() - ref).abs() / ref.clamp_min(1e-3 * ref.max())
        # fp32 sums over 256 products (2^-24 each, random walk), magnified by the gap at the cut (relative 1 - 0.97^2, 0.06)
        assert err.max() < 4 * 16 * 2 ** -24 / 0.06


@pytest.mark.parametrize("m,d", [(128, 320), (100, 448), (128, 1088), (128, 1536), (128, 256)])
def test_gram_matrix_does_not_depend_on_the_number_of_tiles(C, m, d):
    """One video alone (few tiles) and as one of 64 (many): the same fp32 sums over 256 products each, so that only the order of
    a handful of fp64 additions differs."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(m + d)
    X, s = torch.randn(64, 160, d, generator=g, device="cuda").bfloat16(), torch.rand(64, 160, generator=g, device="cuda")
    got = []
    for B in (1, 64):
        p = C.StreamParams(batch=B, n_frame=160, d_model=d, frame_m=m, keep_k=m, rank_r=8, dtype=C.BF16)
        out = C.stream_alloc_state(p)
        C.stream_step(p, 0, 0, X[:B].contiguous(), s[:B].contiguous(), None, out)
        got.append(out[1][0].clone())
    torch.cuda.synchronize()
    assert got[0].diagonal().min() > 0
    assert (got[0] - got[1]).abs().max() < 1e-14 * got[0].max()
