"""The order in which the product without K slices (2 to 128 rows; gate/up projection, output head) adds the K parts of its waves: ascending
for every value, whichever wave adds it.  Four numbers, one in each K part, whose sum hangs on the order: ((2^24 + 1) - 2^24) + 1 = 1 in
fp32, since 2^24 + 1 is 2^24; with the third part first it is 2, with the last one first 0.  Through the whole path: a hidden state of
ones (all layers add zero, no epsilon), so that a logit is the sum of a row of the head."""
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

D, F = 128, 64


def _shape(vocab, head):
    return SimpleNamespace(n_layers=1, d_model=D, n_heads=1, n_kv_heads=1, d_ffn=F, vocab=vocab, dtype="bf16", head_kind=head, rope_theta=1.0e4,
                           rms_eps=0.0)


# vocabularies of the three block widths (64, 96, 160 rows of the head), one of them not a multiple; rows at the edges of the row tiles
@pytest.mark.parametrize("vocab", [16384, 20001, 40960])
@pytest.mark.parametrize("rows", [2, 32, 33, 64, 65, 128])
def test_parts_are_added_in_order(vocab, rows):
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2501_19324_amd import binding as R

    layer = D + 4 * D * D + D + 3 * D * F                    # norm, q k v o, norm, gate up down
    blob = torch.zeros(vocab * D + layer + D + vocab * D, dtype=torch.bfloat16, device="cuda")
    blob[:vocab * D] = 1
    blob[vocab * D + layer:vocab * D + layer + D] = 1        # final norm
    head = blob[vocab * D + layer + D:].view(vocab, D)
    for k, v in ((0, 2.0 ** 24), (16, 1.0), (32, -(2.0 ** 24)), (48, 1.0)):
        head[:, k] = v
    small = torch.zeros(vocab * D + layer + D + D + 8, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    ctx = R.rsd_init([_shape(vocab, "lm"), _shape(vocab, "lm"), _shape(vocab, "reward")], [blob, blob, small], batch=rows, delta=0.5,
                     sep_id=vocab - 1, step_cap=1, max_steps=1, max_ctx=16)
    out = R.rsd_forward(ctx, R.RSD_DRAFT, np.zeros((rows, 1), np.int32), np.ones(rows, np.int32), 1)
    assert out.shape == (rows, 1, vocab) and bool((out == 1.0).all())
    R.rsd_destroy(ctx)
