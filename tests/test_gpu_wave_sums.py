"""The sum over a wave (norms, vector products of a few rows), bit for bit in its order: lanes 32, 16, 8, 4, 2, 1 apart.  The outputs of a
model in bf16 hang on it: another order changes the last bit of a sum, and a cache entry near the middle between two bf16 numbers
then goes the other way.  wave_sums, which finishes the products of other vector kernels, has the same order."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_order_of_the_additions():
    import torch
    from paper_2501_19324_amd import binding as R
    dbg = ctypes.CDLL(os.path.join(os.path.dirname(R.LIB_PATH), "librsd_debug.so"))
    rng = np.random.default_rng(3)
    n = 64 << 12
    v = (rng.standard_normal(n) * np.exp2(rng.integers(-12, 13, n))).astype(np.float32)
    d = torch.from_numpy(v).cuda()
    far, vec, near = (torch.full_like(d, float("nan")) for _ in range(3))
    torch.cuda.synchronize()
    assert dbg.rsd_debug_wave_sum(*(ctypes.c_void_p(t.data_ptr()) for t in (d, far, vec, near)), n) == 0

    def in_order(steps):
        x = v.reshape(-1, 64).copy()
        for step in steps:
            x = x + x[:, np.arange(64) ^ step]
        return x.reshape(-1).view(np.uint32)

    want = in_order((32, 16, 8, 4, 2, 1))
    assert (far.cpu().numpy().view(np.uint32) == want).all()
    assert (vec.cpu().numpy().view(np.uint32) == want).all()
    # neighbours first (the mirrors at 8 and 16 lanes bring equal sums together: as good as 4 and 8 apart)
    assert (near.cpu().numpy().view(np.uint32) == in_order((1, 2, 4, 8, 16, 32))).all()
