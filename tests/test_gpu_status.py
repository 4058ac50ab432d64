"""covspec_image_status: the per-image word that says whether the multi-workgroup kernels of the low-rank stage
ran to the end or gave up waiting for one another.  The give-up path is driven from the host by shortening the
wait limit to one microsecond: every kernel still exits normally (each wait is bounded and a failed wait only
ends the image's work early), nothing faults or hangs."""
import numpy as np
import pytest

import covspec_inputs as I
from tests import util as U

pytestmark = pytest.mark.gpu

W = I.small_workload(cid=17, name="status", batch=4, n_tokens=1300, d_model=256, dtype=I.BF16, n_query=6, n_heads=2,
                     keep_k=200, preselect_m=640, rank_r=64, factor_rank=200, n_act_layers=1)


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


@pytest.mark.parametrize("lr_mode", [0, 1], ids=["energy", "greedy"])
def test_status_is_zero_after_a_normal_call_and_one_after_a_starved_wait(C, lr_mode):
    import torch
    batch = U.gen_batch(W)
    dev = U.upload(batch, W.dtype)
    p = U.lib_params(C, W, W.batch, rel_mode=0, lr_mode=lr_mode)
    ws = C.alloc_workspace(p)
    args = (p, dev["X"], dev["hidden"], dev["Q"], dev["Wq"], dev["Wk"])
    idx0, tok0 = C.reduce(*args, workspace=ws)
    st0 = C.image_status(p, ws)
    torch.cuda.synchronize()
    assert st0.cpu().numpy().tolist() == [0] * W.batch
    ref = U.oracle_image(W, batch, 0, U.oracle_params(W, rel_mode=0, lr_mode=lr_mode))
    np.testing.assert_array_equal(idx0[0].cpu().numpy(), ref["idx"])

    print("shortening the wait limit to 1 us (lr_mode %d)" % lr_mode, flush=True)
    C.set_wait_limit_us(1)
    try:
        idx1, tok1 = C.reduce(*args, workspace=ws)
        st1 = C.image_status(p, ws)
        torch.cuda.synchronize()
    finally:
        C.set_wait_limit_us(0)
    st1 = st1.cpu().numpy()
    idx1 = idx1.cpu().numpy()
    print("images that gave up:", st1.tolist(), flush=True)
    assert set(st1.tolist()) <= {0, 1}
    assert st1.sum() >= 1, "no image gave up although no workgroup waits longer than a microsecond"
    # whatever happened, the indices are valid positions (never out of range), ascending and unique
    assert idx1.min() >= 0 and idx1.max() < W.n_tokens and np.all(np.diff(idx1, axis=1) > 0)
    for b in range(W.batch):
        if st1[b] == 0:           # an image that did not give up has the normal result
            np.testing.assert_array_equal(idx1[b], idx0[b].cpu().numpy())

    # with the default limit restored the same workspace gives the normal result and a clear status again
    idx2, _ = C.reduce(*args, workspace=ws)
    st2 = C.image_status(p, ws)
    torch.cuda.synchronize()
    assert st2.cpu().numpy().tolist() == [0] * W.batch
    assert torch.equal(idx2, idx0)


@pytest.mark.parametrize("n,r", [(60, 20), (300, 40)], ids=["direct-split", "block-iteration"])
def test_status_one_means_no_result_and_zero_a_valid_one(C, n, r):
    """An image whose split or block iteration gave up goes on to the full solve.  Of 60 tokens that is one workgroup, which waits for nobody:
    the result is valid and the status 0.  Of 300 it gives up as well: status 1 and no energy that could pass for one."""
    import torch
    B, d = 4, 320
    X = np.stack([I.make_spectrum_tokens(n, d, np.exp(-0.05 * np.arange(n)), seed=b, dtype=I.FP32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    args = (p, torch.from_numpy(X).cuda(), torch.rand(B, n, generator=torch.Generator().manual_seed(1)).cuda())
    ws = C.alloc_workspace(p)
    c0 = C.select(*args, workspace=ws)["c"].clone()
    assert C.image_status(p, ws).tolist() == [0] * B
    print("shortening the wait limit to 1 us (%d tokens)" % n, flush=True)
    C.set_wait_limit_us(1)
    try:
        out = C.select(*args, workspace=ws)
        st = C.image_status(p, ws)
        torch.cuda.synchronize()
    finally:
        C.set_wait_limit_us(0)
    st = st.tolist()
    assert sum(st) == (0 if n <= 64 else B), st
    for b in range(B):
        idx = out["idx"][b].tolist()
        assert idx == sorted(set(idx)) and 0 <= idx[0] and idx[-1] < n
        if st[b]:
            assert torch.isnan(out["c"][b]).all()
        else:
            assert (out["c"][b] - c0[b]).abs().max() < 1e-6 * c0[b].max()
