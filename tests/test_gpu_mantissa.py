"""What the workgroups of the low-rank stage hand one another through the workspace are fp64 values in full: no place of their mantissa is taken
for anything else."""
import numpy as np
import pytest

import covspec_inputs as I

pytestmark = pytest.mark.gpu


def windows_without_a_lowest_bit(words, size=64):
    """Runs of `size` doubles that use every place of the mantissa's lower end evenly but the lowest, which is the same in all of them: 2^-63 by
    chance.  (Differences of nearly equal numbers have zeros in all of the last places.)"""
    w = words[:len(words) // size * size].reshape(-1, size)
    top = (w >> np.uint64(52)) & np.uint64(0x7FF)
    real = ((top > 1023 - 60) & (top < 1023 + 60)).all(axis=1)           # neither zeros, integers, floats in pairs nor unused memory
    for bit in range(1, 9):
        ones = ((w >> np.uint64(bit)) & np.uint64(1)).sum(axis=1)
        real &= (ones >= size // 4) & (ones <= size - size // 4)
    lowest = (w & np.uint64(1)).sum(axis=1)
    return int(real.sum()), int((real & ((lowest == 0) | (lowest == size))).sum())


# images, tokens, width, rank; what is handed on
CASES = {
    "block-rows": (2, 700, 720, 200),     # the inverted diagonal blocks of the factorisation (a sign iteration with meetings)
    "sign-direct": (1, 100, 128, 40),     # the iterates of the sign iteration without meetings
    "sign-block": (2, 300, 320, 100),
}


@pytest.mark.parametrize("name", list(CASES))
def test_no_place_of_the_mantissa_is_lost(name):
    import torch
    import paper_2605_02218_amd as C
    C.load_library()
    B, n, d, r = CASES[name]
    X = np.stack([I.make_spectrum_tokens(n, d, np.exp(-0.02 * np.arange(n)), seed=b, dtype=I.FP32) for b in range(B)])
    p = C.Params(batch=B, n_tokens=n, d_model=d, n_query=1, dtype=C.FP32, keep_k=n // 3, preselect_m=n, rank_r=r)
    ws = C.alloc_workspace(p)
    ws.zero_()
    C.select(p, torch.from_numpy(X).cuda(), torch.rand(B, n, generator=torch.Generator().manual_seed(1)).cuda(), workspace=ws)
    assert 0 not in C.lowrank_path(p, ws).tolist()
    words = ws.cpu().numpy()
    words = words[(-ws.data_ptr()) % 256:]
    words = words[:len(words) // 8 * 8].view(np.uint64)
    real, lost = windows_without_a_lowest_bit(words)
    assert real > 100 and lost == 0, (real, lost)
