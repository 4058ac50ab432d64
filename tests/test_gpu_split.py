"""The spectral split behind the energies (split.hip): energies against the fp64 oracle at the edges of its ranges."""
import numpy as np
import pytest

import covspec_inputs as I
from oracle import covspec_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    import paper_2605_02218_amd as C
    C.load_library()
    return C


# batch, tokens, width, rank, decay of the singular values per index, the way the solve has to take (lowrank_path: 1 block
# iteration, 3 direct split, 0 full solve; a split that declines or gives up would show as 0 with the same energies); what is at
# its edge
CASES = {
    "smallest": (1, 2, 16, 1, 0.3, 3),
    "one-tile": (3, 64, 96, 63, 0.05, 3),            # direct, every row but one wanted
    "direct-padded": (2, 65, 96, 20, 0.05, 3),       # direct on a padded order of 128
    "direct-largest": (1, 128, 160, 127, 0.05, 3),
    "direct-rank1": (2, 128, 160, 1, 0.05, 3),
    "full-solve": (1, 129, 160, 64, 0.05, 0),        # too large for a direct split, block would be most of the matrix
    "smallest-block": (1, 171, 192, 3, 0.05, 1),     # block of 128 of 171: the whole block is the window
    "many-rows": (4, 900, 960, 40, 0.05, 1),         # products on 64 x 32 tiles
    "few-images": (6, 700, 720, 130, 0.02, 1),       # on 32 x 32 tiles
    "one-round": (12, 640, 660, 60, 0.05, 1),        # on 64 x 64 tiles
    "steep": (2, 400, 420, 180, 0.04, 0),            # the block's last rows drown in rounding: no split passes the check
    "seven-blocks": (1, 700, 720, 330, 0.01, 1),     # block of 448: the substitution goes through memory
    "five-blocks": (1, 500, 520, 230, 0.015, 1),
    "window-inside": (2, 400, 420, 180, 0.02, 1),    # block of 256, window in its middle
    "leading-rows": (1, 600, 640, 250, 0.02, 1),     # leading rows that no longer couple are left out of the iteration
    "eleven-images": (11, 171, 192, 40, 0.05, 1),
    "wide-tiles": (110, 128, 160, 30, 0.05, 3),      # more tiles than the device holds workgroups
}


@pytest.mark.parametrize("name", list(CASES))
def test_energies_match_the_oracle(C, name):
    import torch
    B, n, d, r, decay, path = CASES[name]
    sigma = np.exp(-decay * np.arange(min(n, d)))
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    k = max(1, n // 3)
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=k, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    assert C.lowrank_path(p, ws).tolist() == [path] * B
    c, idx = out["c"].cpu().numpy().astype(np.float64), out["idx"].cpu().numpy()
    op = O.Params(preselect_m=n, rank_r=r, keep_k=k)
    for b in range(B) if B <= 16 else (0, 7, 8, 63, B - 1):
        ref = O.select(X[b].astype(np.float64), sf[b], op)
        # c is rounded to fp32 (6e-8); a residual of 1e-9 enters an energy at most as 1e-9 / relative gap (>= 0.0198 here),
        # twice; energies far below the largest carry its rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 2e-7, "%s image %d: %g" % (name, b, err.max())
        np.testing.assert_array_equal(idx[b], ref["idx"])


# Full solves: images, tokens, width, rank, decay.  Each workgroup adds up 64 columns, a wave an eighth of the rows: one column beyond two
# workgroups' columns and a column short, rows that eight do not divide, several images of which one has no tokens of any length.
FULL = {"129": (1, 129, 160, 64, 0.05), "191": (2, 191, 224, 100, 0.02), "192": (3, 192, 224, 100, 0.02), "577": (2, 577, 608, 420, 0.005)}


@pytest.mark.parametrize("name", list(FULL))
def test_energies_of_a_full_solve(C, name):
    import torch
    B, n, d, r, decay = FULL[name]
    sigma = np.exp(-decay * np.arange(n))
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    if B > 2:
        X[1] = 0.0
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    assert C.lowrank_path(p, ws).tolist() == [0] * B and C.image_status(p, ws).tolist() == [0] * B
    c = out["c"].cpu().numpy().astype(np.float64)
    for b in range(B):
        if not X[b].any():
            assert not c[b].any()
            continue
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))["c"]
        # c is rounded to fp32 (6e-8); a converged sweep leaves 1e-10 of a row in the others, over the relative gap
        err = np.abs(c[b] - ref) / np.maximum(ref, 1e-6 * ref.max())
        assert err.max() < 6e-8 + 2e-10 / (np.exp(2 * decay) - 1) + 2e-8, "%s image %d: %g" % (name, b, err.max())


# The sign iteration of small matrices without meetings (split.hip) at its edges, and the one with meetings beyond: batch, tokens,
# width, rank, decay, way.  Order 64, 128, 192 and 256, each with as many images as it takes and one more (order 64: while a compute unit gets
# one of the 32 x 32 tiles of the other form).
SMALL_SIGN = {
    "order-64": (40, 64, 96, 20, 0.05, 3),
    "order-64-most": (85, 64, 96, 20, 0.05, 3),
    "order-64-over": (86, 64, 96, 20, 0.05, 3),
    "order-128-most": (23, 110, 128, 40, 0.05, 3),
    "order-128-over": (24, 110, 128, 40, 0.05, 3),
    "order-192-most": (7, 300, 320, 100, 0.02, 1),
    "order-192-over": (8, 300, 320, 100, 0.02, 1),
    "order-256-most": (3, 400, 420, 180, 0.02, 1),
    "order-256-over": (4, 400, 420, 180, 0.02, 1),
    "leading-rows-left-out": (2, 600, 640, 190, 0.02, 1),
}


@pytest.mark.parametrize("name", list(SMALL_SIGN))
def test_small_sign_iteration(C, name):
    import torch
    B, n, d, r, decay, path = SMALL_SIGN[name]
    sigma = np.exp(-decay * np.arange(min(n, d)))
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    Xd, sd = torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda()
    out = C.select(p, Xd, sd, workspace=ws)
    assert C.lowrank_path(p, ws).tolist() == [path] * B
    c = out["c"].cpu().numpy().astype(np.float64)
    for _ in range(3):                    # whatever order the workgroups ran in, and whatever the buffers held before
        assert torch.equal(C.select(p, Xd, sd, workspace=ws)["c"], out["c"])
    for b in (0, B // 2, B - 1):
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # c is rounded to fp32 (6e-8); a residual of 1e-9 enters an energy at most as 1e-9 over the relative gap (>= 0.039 here), twice;
        # energies far below the largest carry its rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 2e-9 / (np.exp(2 * decay) - 1) + 2e-8, "%s image %d: %g" % (name, b, err.max())


# The cut by counting (split.hip) at its edges, and by a tridiagonal form beyond: images, tokens, width, rank, decay, way.
CUT = {
    "rank-4": (1, 400, 420, 4, 0.05, 1),                  # too near the window's end for a first interval from the diagonal
    "rank-5": (1, 400, 420, 5, 0.05, 1),
    "window-inside": (1, 900, 960, 240, 0.015, 1),
    "four-images": (4, 300, 320, 100, 0.02, 1),           # the most
    "one-image-more": (5, 300, 320, 100, 0.02, 1),
    "direct-64": (4, 64, 96, 63, 0.05, 3),
    "direct-64-five": (5, 50, 96, 1, 0.05, 3),
    "direct-128": (8, 127, 160, 126, 0.05, 3),
    "direct-128-more": (9, 127, 160, 126, 0.05, 3),
    "direct-128-steep": (2, 100, 128, 40, 0.2, 3),        # the cut far below the largest eigenvalue: points in a geometric sequence
}


@pytest.mark.parametrize("name", list(CUT))
def test_cut_of_few_images(C, name):
    import torch
    B, n, d, r, decay, path = CUT[name]
    sigma = np.exp(-decay * np.arange(min(n, d)))
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    if B > 3:
        X[1] = 0.0                        # nothing to cut: the others must not wait for it
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    Xd, sd = torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda()
    out = C.select(p, Xd, sd, workspace=ws)
    live = [b for b in range(B) if X[b].any()]
    assert [C.lowrank_path(p, ws).tolist()[b] for b in live] == [path] * len(live)
    for _ in range(3):
        assert torch.equal(C.select(p, Xd, sd, workspace=ws)["c"], out["c"])
    c = out["c"].cpu().numpy().astype(np.float64)
    assert not c[[b for b in range(B) if b not in live]].any()
    for b in live[:2] + live[-1:]:
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # as above: fp32 rounding, a residual of 1e-9 over the relative gap twice, the largest energy's rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 2e-9 / (np.exp(2 * decay) - 1) + 2e-8, "%s image %d: %g" % (name, b, err.max())


# Batches whose products go on each width of tile of the fp64 kernel (gemm64.hip): images, tokens, rank; the last tile of 96, 48 and (in one of
# the two) 80 columns is a partial one.  test_gemm64_tiles.py holds the names against the rule.
TILE_WIDTHS = {"64x80": (7, 950, 100), "64x80-partial": (4, 1638, 120), "64x48": (10, 500, 60), "64x96": (12, 1270, 300), "64x64": (4, 1270, 120),
               "64x32": (2, 1000, 180), "32x32": (4, 1000, 240),
               # a 16 x 16 tile per compute unit: 128 x 256 of two images, 192 x 320 of one; and beyond
               "16x16-most": (2, 250, 60), "16x16": (1, 310, 100), "16x16-over": (2, 310, 100)}


@pytest.mark.parametrize("name", list(TILE_WIDTHS))
def test_products_on_every_width_of_tile(C, name):
    import torch
    B, n, r = TILE_WIDTHS[name]
    d, decay = (n + 29) // 4 * 4, 3.0 / r                 # sigma_r is a twentieth of sigma_1
    sigma = np.exp(-decay * np.arange(n))
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) if b in (0, B - 1) else np.zeros((n, d), np.float32) for b in range(B)])
    for b in range(1, B - 1):
        X[b] = X[0][::-1] if b % 2 else X[B - 1]
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    assert set(C.lowrank_path(p, ws).tolist()) <= {1, 2}
    c = out["c"].cpu().numpy().astype(np.float64)
    for b in (0, B - 1):
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))["c"]
        err = np.abs(c[b] - ref) / np.maximum(ref, 1e-6 * ref.max())
        assert err.max() < 6e-8 + 2e-9 / (np.exp(2 * decay) - 1) + 2e-8, "%s image %d: %g" % (name, b, err.max())
    for b in range(1, B - 1):                             # the same tokens, in another place of the batch
        same = c[0][::-1] if b % 2 else c[B - 1]
        assert np.abs(c[b] - same).max() < 2e-7 * same.max()


# tokens, rank, decay of the singular values per index, factor on the four largest of them, the way the solve has to take; what
# the block iteration's schedule has to cope with
SCHEDULES = {
    "slow": (256, 32, 0.006, 1.0, 2),                 # lambda_r 3.2 times what the block leaves out: every block at its longest
    "one-block": (300, 72, 0.03, 1.0, 1),             # there after the first two factorisations but for one product
    "outliers": (300, 72, 0.02, 30.0, 1),             # first row 2e6 above the last: short blocks, rows of very different length
    "far-outliers": (300, 72, 0.02, 100.0, 1),        # 2e7
    "few-wanted": (256, 2, 0.02, 1.0, 1),
    "wanted-to-the-edge": (256, 64, 0.02, 1.0, 1),    # the block ends 64 rows beyond the cut
}


@pytest.mark.parametrize("name", list(SCHEDULES))
def test_schedules_of_the_block_iteration(C, name):
    import torch
    n, r, decay, factor, path = SCHEDULES[name]
    sigma = np.exp(-decay * np.arange(n))
    sigma[:4] *= factor
    B, d = 3, n + 20
    X = np.stack([I.make_spectrum_tokens(n, d, sigma, seed=b, dtype=I.FP32) for b in range(B)])
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    assert C.lowrank_path(p, ws).tolist() == [path] * B
    c = out["c"].cpu().numpy().astype(np.float64)
    for b in range(B):
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # fp32 rounding of c, and the admitted residual over the relative gap exp(2 decay) - 1, twice; energies far below the
        # largest carry its rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 2e-9 / (np.exp(2 * decay) - 1), "%s image %d: %g" % (name, b, err.max())


# tokens, rank, eigenvalues of the Gram matrix by index, the ways the solve may take: spectra so steep that a block stands two or three
# products, and one that is there after the first block but for what its first estimate is off
STEEP = {
    "cubic": (512, 64, lambda i, r: (i + 1.0) ** -3, (1, 2)),
    "cubic-short": (256, 64, lambda i, r: (i + 1.0) ** -3, (1, 2)),
    "power-2.5": (256, 100, lambda i, r: (i + 1.0) ** -2.5, (1, 2)),
    "power-4": (384, 128, lambda i, r: (i + 10.0) ** -4, (1, 2)),
    "outliers": (256, 64, lambda i, r: np.exp(-0.02 * i) * np.where(i < 3, 1e4, 1.0), (1, 2)),
    "outliers-slow": (512, 160, lambda i, r: np.exp(-0.015 * i) * np.where(i < 3, 1e4, 1.0), (1, 2)),
    "outliers-power": (256, 100, lambda i, r: (i + 1.0) ** -2 * np.where(i < 3, 100.0, 1.0), (1, 2)),
    "first-estimate": (200, 8, lambda i, r: (i + 10.0) ** -4, (1,)),
}


@pytest.mark.parametrize("name", list(STEEP))
def test_steep_spectra_stay_on_the_block_iteration(C, name):
    """A few large tokens above the others, or a fast decay: the block iteration has to finish these (a full solve takes ten
    times as long)."""
    import torch
    n, r, spectrum, paths = STEEP[name]
    lam = spectrum(np.arange(n), r)
    B, d = 6, n + 24
    X = np.stack([I.make_spectrum_tokens(n, d, np.sqrt(lam / lam.max()), seed=20 + b, dtype=I.FP32) for b in range(B)])
    sf = np.stack([np.random.default_rng(b).random(n).astype(np.float32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    path = C.lowrank_path(p, ws).tolist()
    c = out["c"].cpu().numpy().astype(np.float64)
    for b in range(B):
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # fp32 rounding of c, and the admitted residual over the relative gap at the cut, twice; energies far below the
        # largest carry its rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 2e-9 / (lam[r - 1] / lam[r] - 1), "%s image %d: %g" % (name, b, err.max())
    assert set(path) <= set(paths), path


# eigenvalues by index of the images of one batch, 256 tokens, rank 32: there at different orthonormalisations, in different buffers,
# in the first or the second pass or by the full solve
MIXED = [lambda i: np.exp(-0.06 * i), lambda i: np.exp(-0.012 * i), lambda i: np.exp(-0.002 * i),
         lambda i: np.exp(-0.04 * i) * np.where(i < 4, 900.0, 1.0), lambda i: (i + 1.0) ** -3, lambda i: np.exp(-0.02 * i) * np.where(i < 3, 1e4, 1.0),
         lambda i: (i + 1.0) ** -1.5, lambda i: np.exp(-0.15 * i)]


def test_images_of_one_batch_do_not_touch_one_another(C):
    """Each image of a mixed batch gives to the bit what it gives in a batch of copies of itself (of the same size, so on the same tiles), by the
    same way; all ways occur, and the energies are the oracle's."""
    import torch
    n, r, B, d = 256, 32, len(MIXED), 280
    i = np.arange(n)
    lam = [f(i) / f(i).max() for f in MIXED]
    X = np.stack([I.make_spectrum_tokens(n, d, np.sqrt(v), seed=80 + b, dtype=I.FP32) for b, v in enumerate(lam)])
    sf = np.random.default_rng(0).random(n).astype(np.float32)
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)

    def solve(x):
        out = C.select(p, torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(sf).repeat(B, 1).cuda(), workspace=ws)
        return out["c"].cpu().numpy(), C.lowrank_path(p, ws).tolist()
    c, path = solve(X)
    assert set(path) == {0, 1, 2}, path
    for b in range(B):
        cb, pb = solve(np.repeat(X[b:b + 1], B, axis=0))
        assert pb == [path[b]] * B, (b, pb, path)
        assert np.array_equal(cb, np.repeat(c[b:b + 1], B, axis=0)), b
        ref = O.select(X[b].astype(np.float64), sf, O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # fp32 rounding of c, and the admitted residual over the relative gap at the cut, twice; energies far below the
        # largest carry its rounding
        err = np.abs(c[b].astype(np.float64) - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 2e-9 / (lam[b][r - 1] / lam[b][r] - 1), (b, err.max())


def test_an_image_that_fails_the_check_goes_on_from_its_last_product(C):
    """Eight eigenvalues falling over 300 to 1 above a flat tail: the estimates are hardest to make there, and one of these three images
    ends the first pass with a residual of 3.4e-9 (the kernels' and that of an fp64 model of the schedule), which the check refuses; the
    second pass takes it on from the product that the check was made with.  The others are there at 1e-12."""
    import torch
    n, r, d = 200, 8, 224
    i = np.arange(n)
    lam = np.where(i < r, 300.0 ** (1.0 - i / r), 0.1 * np.exp(-0.003 * i))
    X = np.stack([I.make_spectrum_tokens(n, d, np.sqrt(lam / lam.max()), seed=s, dtype=I.FP32) for s in (40, 41, 124)])
    sf = np.random.default_rng(0).random((3, n)).astype(np.float32)
    p = C.Params(batch=3, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    out = C.select(p, torch.from_numpy(X).cuda(), torch.from_numpy(sf).cuda(), workspace=ws)
    assert C.lowrank_path(p, ws).tolist() == [1, 1, 2]
    c = out["c"].cpu().numpy().astype(np.float64)
    for b in range(3):
        ref = O.select(X[b].astype(np.float64), sf[b], O.Params(preselect_m=n, rank_r=r, keep_k=n // 3))
        # fp32 rounding of c; the gap at the cut is wide, and energies far below the largest carry its rounding
        err = np.abs(c[b] - ref["c"]) / np.maximum(ref["c"], 1e-6 * ref["c"].max())
        assert err.max() < 6e-8 + 4e-9, (b, err.max())


def test_equal_eigenvalues_at_the_cut_still_give_a_result(C):
    """Orthogonal tokens of equal length: no rank-r subspace is better than another, the split has no gap to use and the
    full solve answers.  Every energy lies between 0 and the squared length, and they sum to r of it."""
    import torch
    for n, d in ((96, 128), (256, 256)):
        X = torch.zeros(1, n, d)
        X[0, torch.arange(n), torch.arange(n)] = 2.0
        p = C.Params(batch=1, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=10, preselect_m=n, rank_r=20)
        ws = C.alloc_workspace(p)
        out = C.select(p, X.cuda(), torch.rand(1, n, generator=torch.Generator().manual_seed(0)).cuda(), workspace=ws)
        assert C.lowrank_path(p, ws).tolist() == [0]
        c = out["c"].cpu().double()
        assert c.min() > -1e-6 and c.max() < 4.0 + 1e-5 and abs(c.sum() - 80.0) < 1e-4, (n, c.sum())
        assert len(set(out["idx"][0].tolist())) == 10


@pytest.mark.parametrize("B,N,d,T", [(1, 33, 64, 1), (1, 65, 320, 5), (2, 128, 192, 33), (1, 1100, 1024, 16), (1, 40, 72, 3), (3, 700, 1024, 8)],
                         ids=["one-k-step", "remainders", "batch", "row-norms-of-few-tiles", "width-not-64", "row-norms-of-many-tiles"])
def test_fp32_scores_on_few_tiles_match_the_oracle(C, B, N, d, T):
    """The fp32 path's products on 32 x 32 tiles and, beyond their range (many tiles, a width that is no multiple of 64),
    on the 64 x 64 ones; X starts at an odd element, so that no row is aligned to more than four bytes."""
    import torch
    g = torch.Generator().manual_seed(N)
    X0 = torch.randn(B * N * d + 1, generator=g).cuda()
    X = X0[1:].view(B, N, d)
    Q = torch.randn(B, T, d, generator=g).cuda()
    Wq, Wk = (torch.randn(2, d, d, generator=g) / d ** 0.5).cuda()
    p = C.Params(batch=B, n_tokens=N, d_model=d, n_query=T, dtype=C.FP32, keep_k=4, preselect_m=8, rank_r=2)
    sq, _, _ = C.score(p, X, None, Q, Wq, Wk)
    v, q = X.double().cpu() @ Wk.double().cpu(), Q.double().cpu() @ Wq.double().cpu()
    ref = torch.nn.functional.normalize(v, dim=-1) @ torch.nn.functional.normalize(q, dim=-1).transpose(1, 2)
    # a maximum over T cosines of N(0, 1/d); everything but the result's rounding to fp32 (6e-8 of 1) is fp64
    assert (sq.double().cpu() - ref.amax(2)).abs().max() < 1e-7
