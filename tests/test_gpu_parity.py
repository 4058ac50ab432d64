"""GPU parity: the HIP path behind the C ABI against the CPU oracle, element by element.

Bars: indices bit-exact (ties -> lower index); scores within 1e-5 relative for fp32
inputs and 2e-2 for bf16 inputs (denominator floored at 1e-3 of the largest reference
magnitude).  Inputs are seeded and synthetic (covspec_inputs); expected values come
from the oracle only.
"""
import numpy as np
import pytest

import covspec_inputs as I
from oracle import covspec_oracle as O
from tests import util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


SMALL = {
    "fp32-ragged": I.small_workload(cid=11, name="s-fp32", batch=2, n_tokens=300, d_model=192, dtype=I.FP32,
                                    n_query=5, n_heads=3, keep_k=20, preselect_m=50, rank_r=8, factor_rank=32,
                                    n_act_layers=3),
    "bf16-ragged": I.small_workload(cid=12, name="s-bf16", batch=3, n_tokens=333, d_model=256, dtype=I.BF16,
                                    n_query=7, n_heads=2, keep_k=24, preselect_m=56, rank_r=10, factor_rank=48,
                                    n_act_layers=4, structure="dups+outliers"),
    "bf16-tiles": I.small_workload(cid=13, name="m-bf16", batch=2, n_tokens=700, d_model=512, dtype=I.BF16,
                                   n_query=33, n_heads=4, keep_k=150, preselect_m=300, rank_r=40, factor_rank=96,
                                   n_act_layers=2, structure="neardups"),
}


def _cpu(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("rel_mode", [0, 1])
def test_score_matches_oracle(C, name, rel_mode):
    w = SMALL[name]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch, rel_mode=rel_mode)
    sq, sa, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    sq, sa, sf = _cpu(sq), _cpu(sa), _cpu(sf)
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, U.oracle_params(w, rel_mode=rel_mode))
        U.assert_scores_close(sq[b], ref["s_query"], w.dtype, "%s s_query[%d]" % (name, b))
        U.assert_scores_close(sa[b], ref["s_act"], w.dtype, "%s s_act[%d]" % (name, b))
        U.assert_scores_close(sf[b], ref["s_fused"], w.dtype, "%s s_fused[%d]" % (name, b))
        if rel_mode == 1:
            assert abs(float(sq[b].astype(np.float64).sum()) - 1.0) < 1e-4


def test_large_product_path_with_an_odd_number_of_k_tiles_and_ragged_edges(C):
    """The 256x256-tile kernel of the large bf16 products (taken from 512 tiles up) on a shape none of the five
    workloads has: K = 320 is five 64-wide k-tiles (an odd count), 300 token rows and 320 / 270 output columns end inside
    a tile in both directions (rows beyond the end load zeros), with the row-norm epilogue (projection) and the store
    epilogue (token x folded-query products)."""
    w = I.small_workload(cid=15, name="ring-edges", batch=128, n_tokens=300, d_model=320, dtype=I.BF16, n_query=90,
                         n_heads=4, keep_k=40, preselect_m=80, rank_r=16, factor_rank=64, n_act_layers=1)
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch)
    sq, sa, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    sq, sf = _cpu(sq), _cpu(sf)
    op = U.oracle_params(w)
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, op)
        U.assert_scores_close(sq[b], ref["s_query"], w.dtype, "ring-edges s_query[%d]" % b)
        U.assert_scores_close(sf[b], ref["s_fused"], w.dtype, "ring-edges s_fused[%d]" % b)


@pytest.mark.parametrize("name", ["fp32-ragged", "bf16-tiles"])
def test_zero_tokens_and_zero_keywords_score_zero(C, name):
    """A token or a query keyword that is the zero vector has no direction: its cosine is 0 (the denominator is
    floored, Sec. III-A.1's score is undefined there).  One image gets two zero tokens and a zero keyword, another
    only zero keywords but one."""
    w = SMALL[name]
    batch = {k: (v.copy() if hasattr(v, "copy") else v) for k, v in U.gen_batch(w).items()}
    batch["X"][0, 3] = 0
    batch["X"][0, w.n_tokens - 1] = 0
    batch["Q"][0, 1] = 0
    batch["Q"][1, 1:] = 0
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch)
    sq, _, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    sq, sf = _cpu(sq), _cpu(sf)
    assert np.isfinite(sq).all() and np.isfinite(sf).all()
    assert sq[0, 3] == 0.0 and sq[0, w.n_tokens - 1] == 0.0
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, U.oracle_params(w))
        U.assert_scores_close(sq[b], ref["s_query"], w.dtype, "%s zero vectors s_query[%d]" % (name, b))
        U.assert_scores_close(sf[b], ref["s_fused"], w.dtype, "%s zero vectors s_fused[%d]" % (name, b))


@pytest.mark.parametrize("name", list(SMALL))
def test_score_without_weights_or_hidden(C, name):
    w = SMALL[name]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch, n_act_layers=0)
    sq, sa, sf = C.score(p, dev["X"], None, dev["Q"], None, None)
    assert sa is None
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, U.oracle_params(w), use_hidden=False, use_wq=False, use_wk=False)
        U.assert_scores_close(_cpu(sq)[b], ref["s_query"], w.dtype, "s_query identity")
        U.assert_scores_close(_cpu(sf)[b], ref["s_fused"], w.dtype, "s_fused identity")


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("lr_mode", [0, 1])
def test_select_matches_oracle(C, name, lr_mode):
    import torch
    w = SMALL[name]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    op = U.oracle_params(w, lr_mode=lr_mode)
    refs = [U.oracle_image(w, batch, b, op) for b in range(w.batch)]
    sf32 = np.stack([O.decision_values(r["s_fused"]) for r in refs])      # oracle scores in, HIP selection out
    p = U.lib_params(C, w, w.batch, lr_mode=lr_mode)
    out = C.select(p, dev["X"], torch.from_numpy(sf32).cuda())
    for b, ref in enumerate(refs):
        np.testing.assert_array_equal(_cpu(out["idx_m"])[b], ref["idx_m"])
        if lr_mode == 0:
            U.assert_scores_close(_cpu(out["c"])[b], ref["c"], w.dtype, "%s c[%d]" % (name, b),
                                  tol=1e-5 if w.dtype == I.FP32 else 1e-4)
        else:
            np.testing.assert_array_equal(_cpu(out["pick_order"])[b], ref["pick_order"])
            U.assert_scores_close(_cpu(out["resid"])[b], ref["resid"], w.dtype, "%s resid[%d]" % (name, b),
                                  tol=1e-5 if w.dtype == I.FP32 else 1e-4)
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"],
                                      err_msg="margin_topk=%r" % ref.get("margin_topk"))


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("modes", [(0, 0), (1, 1)])
def test_reduce_matches_oracle(C, name, modes):
    w = SMALL[name]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch, rel_mode=modes[0], lr_mode=modes[1])
    idx, tok = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    idx2, tok2 = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    assert bool((idx == idx2).all()) and bool((tok.view(dev["X"].dtype) == tok2).all())   # deterministic
    idx, tok = _cpu(idx), tok.view({I.BF16: __import__("torch").int16, I.FP32: __import__("torch").float32}[w.dtype]).cpu().numpy()
    X = batch["X"].view(np.int16) if w.dtype == I.BF16 else batch["X"]
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, U.oracle_params(w, rel_mode=modes[0], lr_mode=modes[1]))
        np.testing.assert_array_equal(idx[b], ref["idx"], err_msg="margins topm=%r topk=%r" % (
            ref["margin_topm"], ref.get("margin_topk")))
        assert len(set(idx[b].tolist())) == w.keep_k and np.all(np.diff(idx[b]) > 0)
        np.testing.assert_array_equal(tok[b], X[b][idx[b]])                  # bit copy of the stored rows


def test_ragged_shapes_on_the_large_tile_gemm_path(C):
    # 16 x 1000 tokens x 2176 wide: the projection takes the 256x256-tile kernel (>= 512 tiles) with a
    # ragged last tile in both directions; the oracle checks three of the sixteen images
    w = I.small_workload(cid=14, name="bigtile", batch=16, n_tokens=1000, d_model=2176, dtype=I.BF16, n_query=40,
                         n_heads=17, keep_k=50, preselect_m=100, rank_r=20, factor_rank=128, n_act_layers=1)
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    for rel in (0, 1):
        p = U.lib_params(C, w, w.batch, rel_mode=rel)
        sq, sa, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        idx, _ = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        for b in (0, 7, 15):
            ref = U.oracle_image(w, batch, b, U.oracle_params(w, rel_mode=rel))
            U.assert_scores_close(_cpu(sq)[b], ref["s_query"], w.dtype, "bigtile s_query rel %d img %d" % (rel, b))
            U.assert_scores_close(_cpu(sf)[b], ref["s_fused"], w.dtype, "bigtile s_fused rel %d img %d" % (rel, b))
            np.testing.assert_array_equal(_cpu(idx)[b], ref["idx"], err_msg="margin %r" % ref["margin_topm"])


def test_keep_everything_is_identity(C):
    w = SMALL["bf16-ragged"]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    for lr in (0, 1, 2, 3):   # full-token drafting, whatever the selector
        p = U.lib_params(C, w, w.batch, lr_mode=lr, keep_k=w.n_tokens, preselect_m=w.n_tokens, rank_r=5)
        idx, _ = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        np.testing.assert_array_equal(_cpu(idx), np.tile(np.arange(w.n_tokens, dtype=np.int32), (w.batch, 1)))


@pytest.mark.parametrize("name", ["fp32-ragged", "bf16-ragged"])
def test_selector_ablations_match_oracle(C, name):
    # the selector ablations of Table II / Sec. III-A.3: score-only top-k and seeded random selection
    import torch
    w = SMALL[name]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    X = batch["X"].view(np.int16) if w.dtype == I.BF16 else batch["X"]
    tdt = {I.BF16: torch.int16, I.FP32: torch.float32}[w.dtype]
    for lr, extra in ((C.LR_SCORE_TOPK, {}), (C.LR_RANDOM, dict(seed=20260502)), (C.LR_RANDOM, dict(seed=7))):
        p = U.lib_params(C, w, w.batch, lr_mode=lr, **extra)
        idx, tok = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        idx, tok = _cpu(idx), tok.view(tdt).cpu().numpy()
        for b in range(w.batch):
            ref = U.oracle_image(w, batch, b, U.oracle_params(w, lr_mode=lr, **extra))
            np.testing.assert_array_equal(idx[b], ref["idx"], err_msg="lr_mode %d %r image %d" % (lr, extra, b))
            np.testing.assert_array_equal(tok[b], X[b][idx[b]])
        if lr == C.LR_RANDOM:
            out = C.select(p, dev["X"], None)                        # needs no scores
            np.testing.assert_array_equal(_cpu(out["idx"]), idx)
            assert not np.array_equal(idx[0], idx[1])                # images draw independently
        else:
            sf32 = np.stack([O.decision_values(U.oracle_image(w, batch, b, U.oracle_params(w))["s_fused"]) for b in range(w.batch)])
            out = C.select(p, dev["X"], torch.from_numpy(sf32).cuda())
            for b in range(w.batch):
                np.testing.assert_array_equal(_cpu(out["idx"])[b], O.top_indices(sf32[b], w.keep_k))
                np.testing.assert_array_equal(_cpu(out["idx_m"])[b], O.top_indices(sf32[b], w.preselect_m))


@pytest.mark.parametrize("rel_mode", [0, 1])
@pytest.mark.parametrize("lam", [0.0, 1.0])
def test_activity_only_and_query_only_fusion(C, lam, rel_mode):
    # covspec_score is asked for all three scores and computes both terms; covspec_reduce asks for none and
    # skips the term whose weight is zero: the fused scores and the kept indices are the oracle's either way
    w = SMALL["bf16-ragged"]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    p = U.lib_params(C, w, w.batch, lam=lam, rel_mode=rel_mode)
    _, _, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    idx, _ = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    for b in range(w.batch):
        ref = U.oracle_image(w, batch, b, U.oracle_params(w, lam=lam, rel_mode=rel_mode))
        U.assert_scores_close(_cpu(sf)[b], ref["s_fused"], w.dtype, "s_fused lambda %g" % lam)
        np.testing.assert_array_equal(_cpu(idx)[b], ref["idx"])


EDGE = {
    # one keyword, one act layer, tiny width; M spans less than one 64-row pair of the eigen-solve
    "tiny-bf16": dict(batch=3, n_tokens=50, d_model=16, dtype=I.BF16, n_query=1, n_heads=1, keep_k=5, preselect_m=20,
                      rank_r=3, factor_rank=8, n_act_layers=1),
    # the most act layers the kernels take, keep everything but one token, rank 1
    "k8-bf16": dict(batch=2, n_tokens=64, d_model=8, dtype=I.BF16, n_query=2, n_heads=2, keep_k=63, preselect_m=64,
                    rank_r=1, factor_rank=4, n_act_layers=8),
    # fp32, width not a multiple of 8, keep a single token
    "one-fp32": dict(batch=2, n_tokens=40, d_model=12, dtype=I.FP32, n_query=3, n_heads=3, keep_k=1, preselect_m=2,
                     rank_r=1, factor_rank=6, n_act_layers=2),
    # M just above two row blocks (padded order 192), rank close to M: full Jacobi on three pairs
    "pad-bf16": dict(batch=2, n_tokens=130, d_model=264, dtype=I.BF16, n_query=9, n_heads=3, keep_k=30, preselect_m=129,
                     rank_r=28, factor_rank=64, n_act_layers=1),
    # no pre-selection (M = N), block iteration with the smallest block
    "m-eq-n": dict(batch=2, n_tokens=200, d_model=96, dtype=I.BF16, n_query=4, n_heads=4, keep_k=100, preselect_m=200,
                   rank_r=40, factor_rank=80, n_act_layers=1),
}


@pytest.mark.parametrize("name", list(EDGE))
def test_edge_shapes_match_oracle(C, name):
    import torch
    w = I.small_workload(cid=20 + list(EDGE).index(name), name=name, **EDGE[name])
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    X = batch["X"].view(np.int16) if w.dtype == I.BF16 else batch["X"]
    tdt = {I.BF16: torch.int16, I.FP32: torch.float32}[w.dtype]
    for modes in ((0, 0), (1, 1)):
        # greedy picks beyond the rank of the features (at most d) are decided by rounding noise: keep k <= d / 2 there
        over = dict(keep_k=min(w.keep_k, w.d_model // 2)) if modes[1] == 1 else {}
        p = U.lib_params(C, w, w.batch, rel_mode=modes[0], lr_mode=modes[1], **over)
        sq, sa, sf = C.score(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        idx, tok = C.reduce(p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
        idx, tok = _cpu(idx), tok.view(tdt).cpu().numpy()
        for b in range(w.batch):
            ref = U.oracle_image(w, batch, b, U.oracle_params(w, rel_mode=modes[0], lr_mode=modes[1], **over))
            U.assert_scores_close(_cpu(sq)[b], ref["s_query"], w.dtype, "%s s_query[%d] modes %r" % (name, b, modes))
            U.assert_scores_close(_cpu(sf)[b], ref["s_fused"], w.dtype, "%s s_fused[%d] modes %r" % (name, b, modes))
            np.testing.assert_array_equal(idx[b], ref["idx"], err_msg="%s image %d modes %r margins %r %r" % (
                name, b, modes, ref.get("margin_topm"), ref.get("margin_topk")))
            np.testing.assert_array_equal(tok[b], X[b][idx[b]])


def test_flat_spectrum_takes_the_full_eigen_solve(C):
    # Features that are mostly white noise: the eigenvalues of the Gram matrix barely decay past the few factor
    # directions, so the block iteration of the low-rank stage cannot converge in its fixed number of steps, its
    # residual check fails and the image is solved by the full Jacobi iteration instead.  Same bars as elsewhere.
    w = I.small_workload(cid=15, name="flat", batch=2, n_tokens=400, d_model=256, dtype=I.BF16, n_query=4, n_heads=2,
                         keep_k=100, preselect_m=320, rank_r=60, factor_rank=16, n_act_layers=1, noise_std=1.0)
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    import torch
    op = U.oracle_params(w)
    refs = [U.oracle_image(w, batch, b, op) for b in range(w.batch)]
    sf32 = np.stack([O.decision_values(r["s_fused"]) for r in refs])
    p = U.lib_params(C, w, w.batch)
    ws = C.alloc_workspace(p)
    out = C.select(p, dev["X"], torch.from_numpy(sf32).cuda(), workspace=ws)
    assert list(_cpu(C.lowrank_path(p, ws))) == [0] * w.batch          # neither pass of the block iteration converged
    for b, ref in enumerate(refs):
        assert ref["sigma_gap"] > 1e-3, "workload has no usable gap at r: %r" % ref["sigma_gap"]
        U.assert_scores_close(_cpu(out["c"])[b], ref["c"], w.dtype, "flat c[%d]" % b, tol=1e-4)
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"], err_msg="margin_topk=%r" % ref["margin_topk"])


@pytest.mark.parametrize("decay,path", [(0.03, 1), (0.00775, 2), (0.001, 0)])
def test_eigen_solve_ladder_by_spectral_decay(C, decay, path):
    """Tokens with singular values exp(-decay i): the block iteration (r = 32, block of 128 of 256) grows the 32nd eigenvector over
    what the block leaves out by T_m(2 x - 1) in a block of m products, x = lambda_32 / lambda_129 = exp(194 decay).  Fast decay
    (x = 340) is there in the first pass; x = 4.5 needs the products of the second; slow decay (x = 1.2) ends in the full solve.
    Whatever the path, energies and kept indices match the oracle."""
    import torch
    n, d, k, r = 256, 384, 64, 32
    sigma = np.exp(-decay * np.arange(n))
    B = 2
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=k, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    paths = _cpu(C.lowrank_path(p, ws))
    assert list(paths) == [path] * B, paths
    op = O.Params(preselect_m=n, rank_r=r, keep_k=k)
    for b in range(B):
        ref = O.select(X[b].astype(np.float64), sf[b], op)
        U.assert_scores_close(_cpu(out["c"])[b], ref["c"], I.FP32, "c[%d] decay %g" % (b, decay), tol=1e-4)
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"], err_msg="margin_topk=%r" % ref.get("margin_topk"))


@pytest.mark.parametrize("k", [37, 100])
def test_greedy_picks_on_a_large_batch_of_small_images(C, k):
    """With more images than workgroups that the greedy kernel wants on the device, every image gets a single
    workgroup (no waiting between workgroups); 100 tokens and k = 37 leave ragged 16-tiles and a partial last block
    of 16 picks, k = 100 picks every token.  Pick order, residuals and kept set against the oracle."""
    import torch
    w = I.small_workload(cid=16, name="manysmall", batch=130, n_tokens=100, d_model=128, dtype=I.FP32, n_query=2, n_heads=1,
                         keep_k=k, preselect_m=100, rank_r=8, factor_rank=120, n_act_layers=0)
    batch = U.gen_batch(w)
    X = torch.from_numpy(batch["X"]).cuda()
    sf = torch.from_numpy(np.random.default_rng(1).random((w.batch, w.n_tokens)).astype(np.float32)).cuda()
    p = U.lib_params(C, w, w.batch, lr_mode=C.LR_GREEDY_RESIDUAL)
    out = C.select(p, X, sf)
    op = U.oracle_params(w, lr_mode=1)
    for b in (0, 1, 64, 129):
        ref = O.select(batch["X"][b].astype(np.float64), _cpu(sf)[b], op)
        np.testing.assert_array_equal(_cpu(out["pick_order"])[b], ref["pick_order"], err_msg="image %d" % b)
        U.assert_scores_close(_cpu(out["resid"])[b], ref["resid"], I.FP32, "resid[%d]" % b, tol=1e-5)
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"])


@pytest.mark.parametrize("B,n,d,k,why", [
    (3, 1100, 320, 150, "two rows per thread, blocks of 16 picks, 32 workgroups per image"),
    (2, 1300, 704, 330, "blocks of 12 picks (16 columns of 1344 rows do not fit LDS)"),
    (1, 1700, 896, 430, "blocks of 8 picks"),
    (1, 2500, 2560, 1260, "four rows per thread, blocks of 4 picks"),
    (2, 1500, 256, 40, "few picks out of many rows: the left-looking kernel on several workgroups"),
], ids=["rows2-block16", "rows2-block12", "rows2-block8", "rows4-block4", "left-looking"])
def test_greedy_picks_on_large_images(C, B, n, d, k, why):
    """Images above 1024 rows: the greedy kernel keeps several rows per thread, shrinks its block of picks to what
    LDS holds, and falls back to the left-looking scheme when the picks are a small part of the rows.  Pick order,
    residuals and kept set against the oracle for every image."""
    import torch
    w = I.small_workload(cid=17, name="greedy-large", batch=B, n_tokens=n, d_model=d, dtype=I.FP32, n_query=2, n_heads=1,
                         keep_k=k, preselect_m=n, rank_r=8, factor_rank=min(d, n) - 8, n_act_layers=0)
    batch = U.gen_batch(w)
    X = torch.from_numpy(batch["X"]).cuda()
    sf = torch.from_numpy(np.random.default_rng(2).random((B, n)).astype(np.float32)).cuda()
    p = U.lib_params(C, w, B, lr_mode=C.LR_GREEDY_RESIDUAL)
    out = C.select(p, X, sf)
    op = U.oracle_params(w, lr_mode=1)
    for b in range(B):
        ref = O.select(batch["X"][b].astype(np.float64), _cpu(sf)[b], op)
        np.testing.assert_array_equal(_cpu(out["pick_order"])[b], ref["pick_order"], err_msg="image %d (%s)" % (b, why))
        U.assert_scores_close(_cpu(out["resid"])[b], ref["resid"], I.FP32, "resid[%d]" % b, tol=1e-5)
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"])


def _greedy_inputs(kind, n, d, seed):
    g = np.random.default_rng(seed)
    if kind == "equal":                       # nothing but ties: every pick leaves the others as they were
        return 2.0 * np.eye(n, d)
    X = g.standard_normal((n, d)) * 0.98 ** np.arange(d)
    if kind == "front":                       # the largest rows are neighbours: more of them in one wave than it posts
        X *= np.where(np.arange(n) < 64, 4.0, 1.0)[:, None]
    elif kind == "copies":                    # pairs and triples of equal rows
        X[n // 2:n // 2 + n // 4] = X[:n // 4]
        X[-(n // 8):] = X[:n // 8]
    elif kind == "steep":                     # the largest falls below the others with its first pick
        X *= 0.97 ** np.arange(n)[:, None]
    return X


@pytest.mark.parametrize("n,d,k", [(63, 80, 63), (65, 96, 40), (640, 640, 200), (960, 320, 150), (1024, 512, 200), (1281, 512, 250), (1921, 512, 260),
                                   (2305, 640, 600)], ids=lambda v: str(v))
@pytest.mark.parametrize("kind", ["equal", "front", "copies", "steep"])
def test_greedy_runs_of_picks(C, kind, n, d, k):
    """Picks made in runs among the largest residuals, at the edges of the block sizes: order and residuals against the oracle
    as long as the residuals are above the rounding of the products."""
    import torch
    if kind == "equal" and d < n:
        d = (n + 7) // 8 * 8
    X = _greedy_inputs(kind, n, d, n).astype(np.float32)
    sf = np.random.default_rng(3).random(n).astype(np.float32)
    p = C.Params(batch=1, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, lr_mode=C.LR_GREEDY_RESIDUAL, keep_k=k, preselect_m=n, rank_r=1)
    out = C.select(p, torch.from_numpy(X)[None].cuda(), torch.from_numpy(sf)[None].cuda())
    if kind == "equal":
        np.testing.assert_array_equal(_cpu(out["pick_order"])[0], np.arange(k))
        np.testing.assert_array_equal(_cpu(out["resid"])[0], np.full(k, 4.0, np.float32))
        return
    ref = O.select(X.astype(np.float64), sf, O.Params(lr_mode=1, keep_k=k, preselect_m=n, rank_r=1))
    # residuals carry the rounding of the largest squared length, 1.1e-16 of it per step at most, and are returned in fp32; where that
    # is not far below them the order is noise
    sure = int(np.sum(ref["resid"] > 1e-9 * ref["resid"][0]))
    assert sure >= min(k, n // 4, 200)
    np.testing.assert_array_equal(_cpu(out["pick_order"])[0][:sure], ref["pick_order"][:sure])
    np.testing.assert_allclose(_cpu(out["resid"])[0][:sure].astype(np.float64), ref["resid"][:sure], rtol=1e-6, atol=1.1e-16 * k * ref["resid"][0])
    assert len(set(_cpu(out["idx"])[0].tolist())) == k


@pytest.mark.parametrize("B,n,d", [(1, 40, 64), (2, 65, 128), (3, 700, 192), (7, 1000, 320), (2, 300, 72), (1, 33, 448)],
                         ids=["one-k-tile", "k-halves", "small-tiles", "large-tiles", "width-not-64", "odd-k-tiles"])
def test_greedy_picks_from_bf16_rows(C, B, n, d):
    """The fp64 Gram matrix of bf16 rows, which the residuals show: its tiles, k-tiles of 64 and the general kernel beyond them."""
    import torch
    X = torch.randn(B, n, d, generator=torch.Generator().manual_seed(n)) * 0.97 ** torch.arange(d)
    X = X.to(torch.bfloat16)
    sf = np.random.default_rng(3).random((B, n)).astype(np.float32)
    k = min(n, d) // 2
    m = n - 3                                              # rows that the Gram matrix leaves out
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.BF16, lr_mode=C.LR_GREEDY_RESIDUAL, keep_k=k, preselect_m=m, rank_r=1)
    out = C.select(p, X.cuda(), torch.from_numpy(sf).cuda())
    for b in range(B):
        ref = O.select(X[b].double().numpy(), sf[b], O.Params(lr_mode=1, keep_k=k, preselect_m=m, rank_r=1))
        np.testing.assert_array_equal(_cpu(out["pick_order"])[b], ref["pick_order"])
        # the rounding of the largest squared length once a pick, and of the result to fp32
        np.testing.assert_allclose(_cpu(out["resid"])[b].astype(np.float64), ref["resid"], rtol=1e-6, atol=1.1e-16 * k * ref["resid"][0])


@pytest.mark.parametrize("n", [64, 130, 512, 513, 960])
def test_greedy_picks_among_equal_residuals(C, n):
    """Orthogonal rows of three lengths, so that no pick changes another's residual: the longest first, equal ones by index."""
    import torch
    level = np.random.default_rng(n).integers(1, 4, n)
    d = (n + 7) // 8 * 8
    X = (np.eye(n, d) * level[:, None]).astype(np.float32)
    k = n - 3
    p = C.Params(batch=1, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, lr_mode=C.LR_GREEDY_RESIDUAL, keep_k=k, preselect_m=n, rank_r=1)
    out = C.select(p, torch.from_numpy(X)[None].cuda(), torch.rand(1, n, generator=torch.Generator().manual_seed(n)).cuda())
    order = np.argsort(-level, kind="stable")[:k]
    np.testing.assert_array_equal(_cpu(out["pick_order"])[0], order)
    np.testing.assert_array_equal(_cpu(out["resid"])[0], (level[order] ** 2).astype(np.float32))


def test_greedy_time_does_not_depend_on_ties(C):
    """Blank regions give tokens that are copies of one another.  Equal residuals take as long as distinct ones in the same order, where
    the runs are as long (a run that ended at every tie took five times that)."""
    import torch
    n, took = 512, []
    for step in (0.0, 1e-3):
        X = torch.diag(2.0 - step * torch.arange(n)).float()[None].cuda()
        p = C.Params(batch=1, n_tokens=n, d_model=n, n_query=1, dtype=C.FP32, lr_mode=C.LR_GREEDY_RESIDUAL, keep_k=n // 2, preselect_m=n, rank_r=1)
        ws, sf = C.alloc_workspace(p), torch.rand(1, n).cuda()
        best = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                C.select(p, X, sf, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b))
        took.append(min(best))
    assert took[0] < 2.0 * took[1], took


def test_greedy_picks_with_rows_that_are_not_finite(C):
    """An infinite token is the largest; whatever its column does to the others, the picks stay distinct positions."""
    import torch
    X = torch.randn(1, 300, 64, generator=torch.Generator().manual_seed(5))
    X[0, 77] = float("inf")
    p = C.Params(batch=1, n_tokens=300, d_model=64, n_query=1, dtype=C.FP32, lr_mode=C.LR_GREEDY_RESIDUAL, keep_k=50, preselect_m=300, rank_r=1)
    out = C.select(p, X.cuda(), torch.rand(1, 300, generator=torch.Generator().manual_seed(6)).cuda())
    picks = _cpu(out["pick_order"])[0]
    assert picks[0] == 77 and len(set(picks.tolist())) == 50


def test_select_ties_and_exact_duplicates(C):
    import torch
    # constant fused scores: every cut is a tie -> the first M positions; duplicates tie in the energy ranking
    w = SMALL["bf16-ragged"]
    batch = U.gen_batch(w)
    dev = U.upload(batch, w.dtype)
    sf = torch.zeros(w.batch, w.n_tokens, dtype=torch.float32, device="cuda")
    sf[:, 100:] = -1.0
    p = U.lib_params(C, w, w.batch)
    out = C.select(p, dev["X"], sf)
    np.testing.assert_array_equal(_cpu(out["idx_m"]), np.tile(np.arange(w.preselect_m, dtype=np.int32), (w.batch, 1)))
    for b in range(w.batch):
        ref = O.select(I.as_f64(batch["X"][b], w.dtype), _cpu(sf)[b], U.oracle_params(w))
        np.testing.assert_array_equal(_cpu(out["idx"])[b], ref["idx"])
