"""Parity of covspec_stream_step (frame-by-frame selection with a carried Gram matrix) against oracle/stream_oracle.py."""
import numpy as np
import pytest

import covspec_inputs as I
from oracle import stream_oracle as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2605_02218_amd as C
    C.load_library()
    return C


def _dev(a, dtype):
    import torch
    if dtype == I.BF16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _run(C, B, n_frames, n_frame, d, m, k, r, dtype, cut_every=0, factor_rank=64, seed0=None):
    """Drives B videos through n_frames frames on the GPU and in the oracle; checks every frame."""
    import torch
    seed0 = 10 * B if seed0 is None else seed0
    vids = [I.make_video_stream(n_frames, n_frame, d, dtype=dtype, seed=seed0 + b, cut_every=cut_every,
                                factor_rank=factor_rank) for b in range(B)]
    p = C.StreamParams(batch=B, n_frame=n_frame, d_model=d, frame_m=m, keep_k=k, rank_r=r, dtype=dtype)
    ws = torch.empty(C.stream_workspace_size(p) + 256, dtype=torch.uint8, device="cuda")
    states = [C.stream_alloc_state(p), C.stream_alloc_state(p)]
    ora = [S.empty_state(d) for _ in range(B)]
    n_keep, solved = 0, 0
    tol = 1e-5      # of the largest energy: the rows are given exactly, the Gram matrix and the solve are fp64-grade
    for f in range(n_frames):
        Xf = np.stack([v[0][f] for v in vids])
        sf = np.stack([v[1][f] for v in vids])
        src, dst = states[f & 1], states[(f + 1) & 1]
        nxt, c = C.stream_step(p, n_keep, f * n_frame, _dev(Xf, dtype), torch.from_numpy(sf).cuda(),
                               src if n_keep else None, dst, workspace=ws, want_c=True)
        torch.cuda.synchronize()
        assert nxt == min(k, n_keep + m)
        Z, G, ids = (t.cpu() for t in dst)
        for b in range(B):
            ref = S.stream_step(ora[b], I.as_f64(Xf[b], dtype), sf[b], f * n_frame, m, k, r)
            where = "frame %d video %d" % (f, b)
            if ref["c"] is not None:
                solved += 1
                assert ref["margin_topk"] > 2e-5 and ref["sigma_gap"] > 1e-4, "%s: input has a near-tie: %r" % (where, ref)
                got = c[b].cpu().numpy().astype(np.float64)
                scale = max(np.abs(ref["c"]).max(), 1e-300)
                np.testing.assert_allclose(got / scale, ref["c"] / scale, atol=tol, rtol=0, err_msg=where)
            else:
                assert c is None
            np.testing.assert_array_equal(ids[b, :nxt].numpy(), ref["ids"], err_msg=where)
            rows = Z[b, :nxt].view(torch.int16).numpy() if dtype == I.BF16 else Z[b, :nxt].numpy()
            want = I.store(ora[b].rows.astype(np.float32), dtype)
            np.testing.assert_array_equal(rows, want.view(np.int16) if dtype == I.BF16 else want, err_msg=where)
            # the carried Gram matrix is that of the kept rows: bf16 products are exact and summed in fp32 pieces
            # flushed into fp64 (relative 1e-6 of the row norms); fp32 storage is contracted in fp64
            Gref = ora[b].rows @ ora[b].rows.T
            gs = np.sqrt(np.outer(np.diag(Gref), np.diag(Gref)))
            np.testing.assert_allclose(G[b, :nxt, :nxt].numpy() / gs, Gref / gs, atol=2e-6 if dtype == I.BF16 else 1e-12,
                                       rtol=0, err_msg=where)
        n_keep = nxt
    return solved


def test_stream_matches_oracle_bf16_subspace_iteration(C):
    # k + M_f = 320 candidates, r = 24: block iteration (block of 128); 7 frames: 2 of warm-up, 5 with a decision
    assert _run(C, B=3, n_frames=7, n_frame=200, d=256, m=96, k=224, r=24, dtype=I.BF16) == 15


def test_stream_matches_oracle_fp32_full_solve_and_scene_cuts(C):
    # 150 candidates, r = 60: the full Jacobi solve; a fresh scene every third frame; M_f does not divide k, so the
    # first decision sees fewer candidates than the later ones
    assert _run(C, B=2, n_frames=8, n_frame=130, d=96, m=50, k=100, r=30, dtype=I.FP32, cut_every=3) >= 10


def test_stream_keeps_everything_while_the_memory_is_not_full(C):
    # k is never reached: every frame only appends (no eigen-solve), ids and rows in arrival order
    assert _run(C, B=2, n_frames=3, n_frame=64, d=64, m=16, k=64, r=4, dtype=I.BF16) == 0


def test_stream_frame_m_equals_n_frame_and_single_video(C):
    # no pre-selection inside the frame (M_f = N_f), one video
    assert _run(C, B=1, n_frames=4, n_frame=72, d=128, m=72, k=100, r=10, dtype=I.FP32) == 3


def test_stream_at_the_benchmark_shape(C):
    # the shape bench.py --stream times: 4 videos, frames of 1024 x 1536 bf16, 256 pre-selected, 1024 kept, r = 128;
    # four frames fill the memory, two decide among 1280 candidates (block iteration with a block of 192)
    # (the videos of the benchmark: seeds 0..3)
    assert _run(C, B=4, n_frames=6, n_frame=1024, d=1536, m=256, k=1024, r=128, dtype=I.BF16, seed0=0) == 8


def test_stream_takes_as_many_videos_as_a_grid_dimension(C):
    """65536 tiny videos in one call (11 GB of workspace): as many as the second dimension of a grid holds."""
    import torch
    B, d = 65536, 8
    p = C.StreamParams(batch=B, n_frame=2, d_model=d, frame_m=1, keep_k=2, rank_r=1, dtype=C.FP32)
    ws = torch.empty(C.stream_workspace_size(p) + 256, dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(0)
    Z = torch.randn(B, 2, d, generator=g, device="cuda")
    G = torch.bmm(Z.double(), Z.double().transpose(1, 2).contiguous())
    ids = torch.arange(2, device="cuda", dtype=torch.int32).repeat(B, 1)
    F, s = torch.randn(B, 2, d, generator=g, device="cuda"), torch.rand(B, 2, generator=g, device="cuda")
    dst = C.stream_alloc_state(p)
    n, c = C.stream_step(p, 2, 10, F, s, (Z, G, ids), dst, workspace=ws, want_c=True)
    torch.cuda.synchronize()
    assert n == 2
    for b in (0, 1, 40000, B - 1):
        ref = S.stream_step(S.StreamState(Z[b].double().cpu().numpy(), np.arange(2)), F[b].double().cpu().numpy(), s[b].cpu().numpy(), 10, 1, 2, 1)
        np.testing.assert_allclose(c[b].cpu().numpy(), ref["c"], rtol=0, atol=1e-6 * ref["c"].max())
        np.testing.assert_array_equal(dst[2][b].cpu().numpy(), ref["ids"])


def test_stream_videos_that_need_the_full_solve_beside_others(C):
    """A batch in which the block iteration answers for some videos and the full solve, on its own copy of the Gram matrix, for the others: the
    energies and the carried Gram matrix of each against the oracle."""
    import torch
    B, n_frame, d, m, k, r = 5, 100, 384, 96, 224, 24
    rng = np.random.default_rng(11)
    rows = []
    for b in range(B):
        decay = 0.001 if b % 2 else 0.03                   # 0.001: lambda_24 is 1.2 times what the block leaves out
        sigma = np.exp(-decay * np.arange(k + m))
        rows.append(I.make_spectrum_tokens(k + m, d, sigma, seed=60 + b, dtype=I.FP32))
    Z = np.stack([x[:k] for x in rows])
    F = np.concatenate([np.stack([x[k:] for x in rows]), np.zeros((B, n_frame - m, d), np.float32)], axis=1)
    s = np.concatenate([1.0 + rng.random((B, m)), rng.random((B, n_frame - m))], axis=1).astype(np.float32)     # the first m are pre-selected
    Zd = Z.astype(np.float64)
    G = Zd @ Zd.transpose(0, 2, 1)
    p = C.StreamParams(batch=B, n_frame=n_frame, d_model=d, frame_m=m, keep_k=k, rank_r=r, dtype=I.FP32)
    ws = torch.empty(C.stream_workspace_size(p) + 256, dtype=torch.uint8, device="cuda")
    dst = C.stream_alloc_state(p)
    ids = torch.arange(k, device="cuda", dtype=torch.int32).repeat(B, 1)
    src = (_dev(Z, I.FP32), torch.from_numpy(G).cuda(), ids)
    n, c = C.stream_step(p, k, 1000, _dev(F, I.FP32), torch.from_numpy(s).cuda(), src, dst, workspace=ws, want_c=True)
    # which way the solve of the same matrices takes
    q = C.Params(batch=B, n_tokens=k + m, d_model=d, n_query=1, dtype=C.FP32, keep_k=k, preselect_m=k + m, rank_r=r)
    w2 = C.alloc_workspace(q)
    C.select(q, _dev(np.stack(rows), I.FP32), torch.rand(B, k + m, generator=torch.Generator().manual_seed(0)).cuda(), workspace=w2)
    assert C.lowrank_path(q, w2).tolist() == [1, 0, 1, 0, 1]
    for b in range(B):
        st = S.StreamState(Zd[b], np.arange(k))
        ref = S.stream_step(st, F[b].astype(np.float64), s[b], 1000, m, k, r)
        assert ref["margin_topk"] > 1e-6 and ref["sigma_gap"] > 5e-4, ref
        got = c[b].cpu().numpy().astype(np.float64)
        np.testing.assert_allclose(got, ref["c"], rtol=0, atol=1e-6 * ref["c"].max(), err_msg="video %d" % b)
        np.testing.assert_array_equal(dst[2][b, :n].cpu().numpy(), ref["ids"], err_msg="video %d" % b)
        Gref = st.rows @ st.rows.T
        np.testing.assert_allclose(dst[1][b, :n, :n].cpu().numpy(), Gref, rtol=0, atol=1e-12 * Gref.max(), err_msg="video %d" % b)
