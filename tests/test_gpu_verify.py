"""GPU parity of covspec_verify (paper Sec. II-A: acceptance probability, first rejection, residual draw)
against oracle/verify_oracle.py, element by element on the same seeded logits.

alpha is compared within 1e-5 relative (fp32 exponentials in the streaming pass, fp64 combination);
n_accept and the correction are integers and compared exactly.  Both are decided by a floating-point
comparison, so each case first checks ON THE ORACLE'S VALUES that no decision sits inside the rounding band
(|u - alpha| > 1e-5 alpha; the residual's cumulative sum clears u * total by more than 1e-9 of the total on
both sides of the drawn word): inside that band either answer would be a correct rounding.
"""
import numpy as np
import pytest

import covspec_inputs as I
from oracle import verify_oracle as VO

pytestmark = pytest.mark.gpu

ALPHA_RTOL = 1e-5


def _dev(a, dtype=None):
    import torch
    if dtype == I.BF16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
    if dtype == I.FP16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.float16)
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _run(d, dtype, want_alpha=True):
    import torch
    import paper_2605_02218_amd as C
    S, L, V = d["zt"].shape
    p = C.VerifyParams(n_seq=S, n_draft=L, vocab=V, dtype=dtype)
    n_acc, corr, alpha = C.verify(p, _dev(d["zt"], dtype), _dev(d["zd"], dtype), _dev(d["tok"]), _dev(d["u_acc"]),
                                  _dev(d["u_res"]), want_alpha=want_alpha)
    torch.cuda.synchronize()
    return n_acc.cpu().numpy(), corr.cpu().numpy(), None if alpha is None else alpha.cpu().numpy()


def _check(d, dtype, n_acc, corr, alpha, seqs=None):
    S, L, V = d["zt"].shape
    for s in (range(S) if seqs is None else seqs):
        zt, zd = I.as_f64(d["zt"][s], dtype), I.as_f64(d["zd"][s], dtype)
        o = VO.verify(zt, zd, d["tok"][s], d["u_acc"][s], d["u_res"][s])
        a = o["alpha"]
        # decisions outside the rounding band (a property of the seeded inputs, checked on the oracle)
        assert np.all(np.abs(d["u_acc"][s].astype(np.float64) - a)[: min(o["n_acc"] + 1, L)] > ALPHA_RTOL * a[: min(o["n_acc"] + 1, L)]), s
        if alpha is not None:
            np.testing.assert_allclose(alpha[s], a, rtol=ALPHA_RTOL, atol=0, err_msg="alpha, sequence %d" % s)
        assert n_acc[s] == o["n_acc"], (s, n_acc[s], o["n_acc"])
        if o["n_acc"] < L and o.get("residual_mass", 0.0) > 0.0:
            c = np.cumsum(o["weights"])
            target = float(d["u_res"][s]) * c[-1]
            w = o["corr"]
            lower = c[w - 1] if w > 0 else 0.0
            band = 1e-9 * c[-1]
            assert c[w] - target > band and (target - lower > band or target == 0.0), s
        assert corr[s] == o["corr"], (s, corr[s], o["corr"])


@pytest.mark.parametrize("dtype,V", [(I.BF16, 4392), (I.FP32, 4100), (I.BF16, 8), (I.FP32, 4), (I.BF16, 2048 * 3), (I.FP16, 4392),
                                     (I.FP16, 8)])
def test_verify_matches_oracle_small(dtype, V):
    """Several chunks with a ragged last one (4392 = 2 * 2048 + 296), exact multiples, and the smallest widths."""
    d = I.make_verify_batch(6, 4, V, dtype, seed=V, copy_rows=1)
    n_acc, corr, alpha = _run(d, dtype)
    assert n_acc[0] == 4 and corr[0] == -1 and np.all(alpha[0] == 1.0)    # draft == target: always accepted
    _check(d, dtype, n_acc, corr, alpha)


@pytest.mark.parametrize("S,L,V,dtype", [(1, 64, 32000, I.BF16), (1, 25, 2048 * 40 - 8, I.BF16), (40, 60, 2048, I.BF16), (3, 63, 9 * 1024 + 4, I.FP32),
                                         (64, 1, 32768 - 8, I.BF16), (64, 1, 65536 - 8, I.FP16), (128, 1, 4096, I.BF16), (300, 2, 264, I.FP32)],
                         ids=["sixteen-chunks", "forty-chunks", "one-chunk", "ragged-chunks", "draw-from-1024", "draw-from-2048", "draw-from-256", "short-chunk"])
def test_verify_positions_and_chunks(S, L, V, dtype):
    """The acceptance kernel's groups of lanes (1 to 64 chunks a row, up to 64 positions, several turns of a wave) and the words a
    thread of the residual passes owns (1, 2, 8)."""
    d = I.make_verify_batch(S, L, V, dtype, seed=S + 7 * L + V, disagreement=0.3 if L > 8 else 0.9)
    d["u_acc"][::2, :-1] *= 0.05                           # half of the sequences accept most positions
    d["u_acc"][:, -1] = 0.9                                # and many of them draw a correction at the last
    n, c, a = _run(d, dtype)
    _check(d, dtype, n, c, a)


def test_verify_time_does_not_grow_with_the_positions():
    """The same logits as 16 sequences of 64 positions of 1024 words and of 8 positions of 8192 words: with a wave per position the
    former took about twice the time, now about the same.  A ratio of two medians of one process."""
    import torch
    import paper_2605_02218_amd as C
    z = torch.randn(2, 1 << 20, device="cuda", generator=torch.Generator(device="cuda").manual_seed(0)).bfloat16()
    took = []
    for L in (8, 64):
        V = (1 << 16) // L
        zt, zd = z.view(2, 16, L, V)
        p = C.VerifyParams(n_seq=16, n_draft=L, vocab=V, dtype=C.BF16)
        args = (torch.zeros(16, L, dtype=torch.int32, device="cuda"), torch.zeros(16, L, device="cuda"), torch.zeros(16, device="cuda"))
        ws = torch.empty(C.verify_workspace_size(p) + 256, dtype=torch.uint8, device="cuda")
        C.verify(p, zt, zd, *args, workspace=ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()                     # replayed: the launches from Python would hide the kernels
        with torch.cuda.graph(graph):
            for _ in range(20):
                C.verify(p, zt, zd, *args, workspace=ws)
        times = []
        for _ in range(15):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        took.append(sorted(times)[7])
    assert took[1] < 1.4 * took[0], took


@pytest.mark.parametrize("S,L,V,dtype", [(8, 5, 32768 - 8, I.BF16), (9, 5, 32768 - 8, I.BF16), (3, 64, 4096, I.FP32), (2, 3, 2048 * 64, I.FP16), (5, 1, 8, I.BF16)],
                         ids=["most-workgroups", "one-more", "many-positions", "vectors-per-thread", "smallest"])
def test_verify_few_sequences(S, L, V, dtype):
    """Few sequences, where one launch may take acceptance, masses and draw together; a second call gives the same.  (The edges of that
    launch's range and a workspace used again: test_verify_on_a_used_workspace.)"""
    d = I.make_verify_batch(S, L, V, dtype, seed=3 * S + V, disagreement=0.8)
    n_acc, corr, alpha = _run(d, dtype)
    _check(d, dtype, n_acc, corr, alpha)
    n2, c2, a2 = _run(d, dtype)
    assert np.array_equal(n2, n_acc) and np.array_equal(c2, corr) and np.array_equal(a2, alpha)


@pytest.mark.parametrize("S,L,V", [(3, 5, 16384), (4, 5, 16384), (32, 3, 2048), (33, 3, 2048), (512, 2, 256), (513, 2, 256), (16, 1, 8192), (17, 1, 8192)],
                         ids=["long-rows", "long-rows-one-more", "eight-chunks", "eight-chunks-one-more", "one-chunk", "one-chunk-one-more", "one-position", "one-position-one-more"])
def test_verify_on_a_used_workspace(S, L, V):
    """Both sides of the lines between one launch behind the statistics and three, twice on one workspace that holds other data: with other
    uniforms other sequences reject, so that a count left over from the first call would show."""
    import torch
    import paper_2605_02218_amd as C
    d = I.make_verify_batch(S, L, V, I.BF16, seed=S + V, disagreement=0.8)
    p = C.VerifyParams(n_seq=S, n_draft=L, vocab=V, dtype=I.BF16)
    ws = torch.full((C.verify_workspace_size(p) + 256,), 255, dtype=torch.uint8, device="cuda")
    zt, zd, tok = _dev(d["zt"], I.BF16), _dev(d["zd"], I.BF16), _dev(d["tok"])
    seen = []
    for u in (d["u_acc"], np.float32(1.0) - d["u_acc"]):
        d["u_acc"] = np.clip(u, 1e-3, 0.999).astype(np.float32)
        out = C.verify(p, zt, zd, tok, _dev(d["u_acc"]), _dev(d["u_res"]), workspace=ws)
        n, c, a = (t.cpu().numpy() for t in out)
        _check(d, I.BF16, n, c, a, seqs=range(S) if S <= 40 else range(0, S, 16))
        seen.append(n)
    assert np.any(seen[0] != seen[1])


def test_verify_time_does_not_fall_with_another_sequence():
    """Eight sequences of 16384 words against nine: one launch for all that follows the statistics, taken for eight, cost a fifth of the
    call.  A ratio of two medians of one process."""
    import torch
    import paper_2605_02218_amd as C
    took = []
    for S in (8, 9):
        g = torch.Generator(device="cuda").manual_seed(1)
        zt = 2.0 * torch.randn(S, 8, 16384, generator=g, device="cuda")
        zd = zt + 0.6 * torch.randn(S, 8, 16384, generator=g, device="cuda")
        p = C.VerifyParams(n_seq=S, n_draft=8, vocab=16384, dtype=C.BF16)
        args = (zt.bfloat16(), zd.bfloat16(), zd.argmax(2).to(torch.int32), torch.rand(S, 8, generator=g, device="cuda"), torch.rand(S, generator=g, device="cuda"))
        ws = torch.empty(C.verify_workspace_size(p) + 256, dtype=torch.uint8, device="cuda")
        C.verify(p, *args, workspace=ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()                     # replayed: the launches from Python would hide the kernels
        with torch.cuda.graph(graph):
            for _ in range(20):
                C.verify(p, *args, workspace=ws)
        times = []
        for _ in range(25):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        took.append(sorted(times)[12])
    assert took[0] < 1.1 * took[1], took


@pytest.mark.parametrize("S,L", [(1, 1), (1, 8), (37, 3), (300, 1)])
def test_verify_batch_shapes(S, L):
    """One row (64 chunks of the row), many sequences (one chunk per row), odd counts."""
    d = I.make_verify_batch(S, L, 8200, I.BF16, seed=100 * S + L, disagreement=0.9)
    n_acc, corr, alpha = _run(d, I.BF16)
    _check(d, I.BF16, n_acc, corr, alpha)
    n2, c2, none = _run(d, I.BF16, want_alpha=False)      # alpha_out is optional
    assert none is None and np.array_equal(n2, n_acc) and np.array_equal(c2, corr)


def test_verify_edge_uniforms_and_tokens():
    """u_res at 0 and just below 1 (first / last word with residual mass), drafted tokens at both ends of the
    vocabulary, and a first-position rejection."""
    dtype, V = I.FP32, 5000
    d = I.make_verify_batch(8, 4, V, dtype, seed=77, disagreement=1.2)
    d["tok"][0, :] = 0
    d["tok"][1, :] = V - 1
    d["u_acc"][2, 0] = np.float32(0.99999994)          # rejected at once unless alpha == 1
    d["u_acc"][3, :] = 0.0                              # every position accepted (alpha > 0)
    d["u_res"][2] = 0.0
    d["u_res"][4] = np.float32(0.99999994)
    d["u_acc"][4, 1] = np.float32(0.99999994)
    d["u_res"][5] = 0.0
    d["u_acc"][5, 2] = np.float32(0.99999994)
    n_acc, corr, alpha = _run(d, dtype)
    assert n_acc[3] == 4 and corr[3] == -1
    for s in (2, 4, 5):
        zt, zd = I.as_f64(d["zt"][s], dtype), I.as_f64(d["zd"][s], dtype)
        o = VO.verify(zt, zd, d["tok"][s], d["u_acc"][s], d["u_res"][s])
        assert n_acc[s] == o["n_acc"] and corr[s] == o["corr"], s
        nz = np.nonzero(o["weights"])[0]
        if d["u_res"][s] == 0.0:
            assert corr[s] == nz[0]
    _check(d, dtype, n_acc, corr, alpha, seqs=(0, 1, 3, 6, 7))


def test_verify_masked_words_and_large_logits():
    """A padded vocabulary (-inf logits on the tail and on a whole leading chunk) and logits far from zero:
    the shifted exponentials must neither overflow nor produce NaN."""
    dtype, V = I.BF16, 6144
    d = I.make_verify_batch(5, 3, V, dtype, seed=5, disagreement=0.8)
    zt, zd = I.as_f32(d["zt"], dtype), I.as_f32(d["zd"], dtype)
    zt[:, :, V - 300:] = -np.inf
    zd[:, :, V - 300:] = -np.inf
    zt[1, :, :2048] = -np.inf                         # a whole chunk masked
    zd[1, :, :2048] = -np.inf
    zt[2] = zt[2] * 20.0 + 300.0                      # large offset and spread
    zd[2] = zd[2] * 20.0 - 250.0
    d["zt"], d["zd"] = I.store(zt, dtype), I.store(zd, dtype)
    g = np.random.default_rng(9).gumbel(size=zd.shape)
    d["tok"] = np.argmax(I.as_f64(d["zd"], dtype) + g, axis=2).astype(np.int32)   # drafted words are unmasked
    n_acc, corr, alpha = _run(d, dtype)
    assert np.all(np.isfinite(alpha))
    assert np.all((corr < V - 300) & ((corr >= 0) | (n_acc == 3)))
    _check(d, dtype, n_acc, corr, alpha)


def test_verify_rejection_with_empty_residual_takes_the_argmax():
    """u = 1 lies outside the contract [0, 1) but forces a rejection where p_t == p_d: the residual has no mass
    and the correction is the target's most likely word (lowest index on ties)."""
    dtype, V = I.BF16, 4104
    d = I.make_verify_batch(3, 2, V, dtype, seed=11, copy_rows=3)
    d["u_acc"][:, 0] = 1.0
    n_acc, corr, alpha = _run(d, dtype)
    assert np.all(n_acc == 0) and np.all(alpha == 1.0)
    for s in range(3):
        z = I.as_f64(d["zt"][s, 0], dtype)
        assert corr[s] == int(np.argmax(z))
        o = VO.verify(I.as_f64(d["zt"][s], dtype), I.as_f64(d["zd"][s], dtype), d["tok"][s], d["u_acc"][s], d["u_res"][s])
        assert o["corr"] == corr[s] and o["n_acc"] == 0


def test_verify_full_vocabulary_batch():
    """The benchmark's shape: 64 sequences of 8 drafted positions over 151,936 words, bf16, every sequence
    against the oracle."""
    dtype = I.BF16
    S, L, V = 64, 8, I.VERIFY_VOCAB
    d = I.make_verify_batch(S, L, V, dtype, seed=2024, copy_rows=2)
    n_acc, corr, alpha = _run(d, dtype)
    assert 0 < (n_acc == L).sum() < S                   # the workload has both outcomes
    _check(d, dtype, n_acc, corr, alpha)
