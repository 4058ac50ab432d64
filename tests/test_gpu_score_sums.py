"""Scores are one sum over the width per element, in one order, whatever the size of the product: an image scores the same
alone and in any batch, copies of a token score and weigh the same, and the kept tokens are the fp64 oracle's."""
import numpy as np
import pytest

import covspec_inputs as I
import util as U
from oracle import covspec_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


@pytest.mark.parametrize("mode", ["cosine", "softmax"])
@pytest.mark.parametrize("N,d,T,weights", [(200, 1024, 16, True), (130, 64, 5, True), (200, 192, 11, True), (190, 320, 33, True), (200, 4096, 16, False)],
                         ids=["width-1024", "one-k-tile", "three-k-tiles", "remainders", "width-4096"])
def test_an_image_scores_the_same_alone_and_in_a_batch(C, mode, N, d, T, weights):
    """1, 80 and 96 images: the inner products are fewer 64 x 64 tiles than compute units, more than that, and enough 128 x 128
    tiles for those.  Equal to the bit (all row norms stay below the size of the 256 x 256 kernel, which adds rows up in another
    order).  The softmax variant's inner products are fp32 ones; only its e(q) is at stake."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d + T)
    X, Q = (torch.randn(96, n, d, generator=g, device="cuda").bfloat16() for n in (N, T))
    Wq, Wk = [(torch.randn(d, d, generator=g, device="cuda") / d ** 0.5).bfloat16() for _ in range(2)] if weights else (None, None)
    got = []
    for B in (1, 80, 96):
        p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=2, dtype=C.BF16, keep_k=4, preselect_m=8, rank_r=2,
                     rel_mode=C.REL_COSINE_MAX if mode == "cosine" else C.REL_ATTN_SOFTMAX)
        got.append(C.score(p, X[:B].contiguous(), None, Q[:B].contiguous(), Wq, Wk)[0])
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1][:1]) and torch.equal(got[1], got[2][:80])


@pytest.mark.parametrize("d", [64, 192, 1024])
def test_scores_on_both_sides_of_the_one_wave_products(C, d):
    """36 images of 200 tokens and 16 query rows: 504 tiles of 32 x 32 of the inner products, a wave each; one image more: 518, and
    tiles of 64 x 64.  1, 3 and 16 k-tiles.  Equal to the bit."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d)
    X, Q = (torch.randn(37, n, d, generator=g, device="cuda").bfloat16() for n in (200, 16))
    got = []
    for B in (36, 37):
        p = C.Params(batch=B, n_tokens=200, d_model=d, n_query=16, n_heads=2, dtype=C.BF16, keep_k=4, preselect_m=8, rank_r=2, rel_mode=C.REL_COSINE_MAX)
        got.append(C.score(p, X[:B].contiguous(), None, Q[:B].contiguous(), None, None)[0])
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1][:36])


@pytest.mark.parametrize("N,d,T", [(100, 320, 20), (97, 64, 17)])
def test_fp32_scores_on_both_sides_of_the_16_x_16_tiles(C, N, d, T):
    """fp64 products of 14 tiles of 16 x 16 an image: 252 tiles, one per compute unit, and 266, which are tiles of 32 x 32; alone the
    query projection is on the small ones too.  Remainders in both directions, 1 and 5 steps of 16 k per wave.  Equal to the bit."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(d)
    X, Q = (torch.randn(19, n, d, generator=g, device="cuda") for n in (N, T))
    Wq, Wk = (torch.randn(d, d, generator=g, device="cuda") / d ** 0.5 for _ in range(2))
    got = []
    for B in (1, 18, 19):
        p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=1, dtype=C.FP32, keep_k=4, preselect_m=8, rank_r=2, rel_mode=C.REL_COSINE_MAX)
        got.append(C.score(p, X[:B].contiguous(), None, Q[:B].contiguous(), Wq, Wk)[0])
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1][:1]) and torch.equal(got[1], got[2][:18])
    x, q = X[0].double().cpu().numpy(), Q[0].double().cpu().numpy()
    ref = O.query_score_cosine(O.embed(x, Wk.double().cpu().numpy()), O.embed(q, Wq.double().cpu().numpy()))
    np.testing.assert_allclose(got[0][0].cpu().numpy(), ref, rtol=2.0 ** -23)      # fp64 inside, rounded once


def test_copies_and_kept_tokens_of_a_single_image(C):
    """576 x 4096 images with exact copies and 20x outliers, one at a time: copies have bit-equal scores and energies, and wherever
    the fp64 values at both cuts are further apart than rounding can move them the kept tokens are the oracle's."""
    import torch
    w = I.small_workload(cid=41, name="single", batch=8, n_tokens=576, d_model=4096, dtype=I.BF16, n_query=32, n_heads=32, keep_k=144,
                         preselect_m=288, rank_r=72, factor_rank=256, n_act_layers=2, structure="dups+outliers")
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    op, p = U.oracle_params(w), U.lib_params(C, w, 1)
    decided = pairs = 0
    for b in range(w.batch):
        x, h, q = (dev[n][b:b + 1].contiguous() for n in ("X", "hidden", "Q"))
        sq, sa, sf = C.score(p, x, h, q, dev["Wq"], dev["Wk"])
        out = C.select(p, x, sf)
        idx, _ = C.reduce(p, x, h, q, dev["Wq"], dev["Wk"])
        sq, sf, c, idx_m = (t[0].cpu().numpy() for t in (sq, sf, out["c"], out["idx_m"]))
        assert torch.equal(idx, out["idx"])
        groups = np.unique(batch["X"][b], axis=0, return_inverse=True)[1].ravel()
        for gid in np.flatnonzero(np.bincount(groups) > 1):
            same = np.flatnonzero(groups == gid)
            assert len(set(sf[same])) == 1
            energies = c[np.isin(idx_m, same)]
            pairs += energies.size > 1
            assert len(set(energies)) <= 1
        ref = U.oracle_image(w, batch, b, op)
        # a cosine: fp32 roundings (2^-24) of d additions, adding up like a random walk; after min-max normalisation relative to
        # the scores' range; both neighbours at the cut move
        eps = 2 * w.d_model ** 0.5 * 2.0 ** -24
        assert np.abs(sq - ref["s_query"]).max() < eps
        eps *= 2 * w.lam / (ref["s_query"].max() - ref["s_query"].min())
        v, e = np.sort(ref["s_fused"])[::-1], np.sort(ref["c"])[::-1]
        # an energy: fp32 sums of 256 products (16 x 2^-24 of |z|^2), tenfold
        if v[w.preselect_m - 1] - v[w.preselect_m] > eps and e[w.keep_k - 1] - e[w.keep_k] > 1e-5 * e[w.keep_k]:
            decided += 1
            np.testing.assert_array_equal(idx[0].cpu().numpy(), ref["idx"])
    assert decided >= 3 and pairs >= 20


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("N,T,H", [(9, 1, 1), (63, 15, 1), (65, 4, 4), (129, 17, 1), (1025, 8, 16), (577, 125, 1)])
def test_attention_scores_over_few_and_many_rows(C, dtype, N, T, H):
    """The mean of the softmax over H * T rows, which sixteen waves share: fewer rows than waves, a row more than that, eight rows a
    wave, a wave left without rows; tokens on both sides of a workgroup's 64.  Odd numbers of tokens: the form of multiples of four
    is another one for bf16."""
    import torch
    d, B = 64, 2
    rng = np.random.default_rng(N)
    X, Q = ((0.5 * rng.standard_normal((B, n, d))).astype(np.float32) for n in (N, T))
    Xd, Qd = (torch.from_numpy(a).cuda() for a in (X, Q))
    if dtype == "bf16":
        Xd, Qd = Xd.bfloat16(), Qd.bfloat16()
    p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=H, dtype=C.BF16 if dtype == "bf16" else C.FP32, keep_k=1, preselect_m=4, rank_r=2,
                 rel_mode=C.REL_ATTN_SOFTMAX)
    sq = C.score(p, Xd, None, Qd, None, None)[0].cpu().numpy()
    for b in range(B):
        ref = O.query_score_attention(Xd[b].double().cpu().numpy(), Qd[b].double().cpu().numpy(), H)
        # fp32: fp64 inside, one rounding of the result and the exponential's.  bf16: a logit is an fp32 sum of d / H products, off by at
        # most d / H roundings of their absolute sum (below 10 / 8 behind the scale), and its difference from the row's maximum by three
        np.testing.assert_allclose(sq[b], ref, rtol=2e-7 if dtype == "fp32" else (d / H + 3) * 2.0 ** -24 * 2.5 + 3e-7)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("T", [1, 3, 7, 16, 17, 33, 47, 48, 64, 65, 79, 96, 111, 112, 113, 128, 150])
def test_attention_scores_of_few_and_many_images(C, dtype, T):
    """The mean over the rows: sixteen waves for 64 tokens of one image, a thread for all rows of a token of 330 (660 waves, up to 16 rows) and 1030
    images (2060 waves).  Shares of 1 to 8 rows and more, whole and cut off.  Equal to the bit, and to the oracle."""
    import torch
    N, d = 65, 64
    g = torch.Generator(device="cuda").manual_seed(T)
    X, Q = (torch.randn(1030, n, d, generator=g, device="cuda") for n in (N, T))
    if dtype == "bf16":
        X, Q = X.bfloat16(), Q.bfloat16()
    got = []
    for B in (1, 330, 1030):
        p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=1, dtype=C.BF16 if dtype == "bf16" else C.FP32, keep_k=1, preselect_m=4, rank_r=2,
                     rel_mode=C.REL_ATTN_SOFTMAX)
        got.append(C.score(p, X[:B].contiguous(), None, Q[:B].contiguous(), None, None)[0])
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1][:1]) and torch.equal(got[1], got[2][:330])
    ref = O.query_score_attention(X[0].double().cpu().numpy(), Q[0].double().cpu().numpy(), 1)
    # as above; logits of width 64 are below 5 behind the scale
    np.testing.assert_allclose(got[0][0].cpu().numpy(), ref, rtol=2e-7 if dtype == "fp32" else (d + 3) * 2.0 ** -24 * 2.5 + 3e-7)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("mode", ["cosine", "softmax"])
def test_scores_with_weights_of_any_alignment(C, dtype, mode):
    """Each weight on a 16-byte boundary and an element behind one: the two are transposed together where they are alike, otherwise each in its own
    form.  Against the oracle, and the same to rounding in all four."""
    import torch
    N, d, T, B = 90, 192, 7, 2
    g = torch.Generator(device="cuda").manual_seed(3)
    X, Q = (torch.randn(B, n, d, generator=g, device="cuda") for n in (N, T))
    W = [torch.randn(d, d, generator=g, device="cuda") / d ** 0.5 for _ in range(2)]
    if dtype == "bf16":
        X, Q, W = X.bfloat16(), Q.bfloat16(), [w.bfloat16() for w in W]
    p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, n_heads=2, dtype=C.BF16 if dtype == "bf16" else C.FP32, keep_k=4, preselect_m=8, rank_r=2,
                 rel_mode=C.REL_COSINE_MAX if mode == "cosine" else C.REL_ATTN_SOFTMAX)
    x, q, wq, wk = (t.double().cpu().numpy() for t in (X[0], Q[0], W[0], W[1]))
    score = O.query_score_cosine if mode == "cosine" else lambda v, e: O.query_score_attention(v, e, 2)
    ref = score(O.embed(x, wk), O.embed(q, wq))
    for shift in (0, 1, 2, 3):
        ws = []
        for i in range(2):
            base = torch.zeros(d * d + 8, dtype=W[i].dtype, device="cuda")
            at = base[shift >> i & 1:][:d * d].view(d, d)
            at.copy_(W[i])
            assert at.data_ptr() % 16 == (shift >> i & 1) * at.element_size()
            ws.append(at)
        got = C.score(p, X, None, Q, ws[0], ws[1])[0][0].cpu().numpy()
        # fp32: fp64 inside.  bf16: fp32 sums of 192 products twice over, against scores from 0.1 (cosine) and mean softmax weights of 1 / 90
        np.testing.assert_allclose(got, ref, rtol=3e-7 if dtype == "fp32" else 3e-4, atol=0 if dtype == "fp32" else 2e-6, err_msg="shift %d" % shift)
