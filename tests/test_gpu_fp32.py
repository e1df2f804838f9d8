"""The fp32 path at the edges of its kernels: chunked passes around the 32x32 and 64x64 tiles, products with fewer and with
more 64x64 tiles than compute units, an odd vocabulary, decode rows of every template size, and contexts that fit 8 pages
(one block walks them) or just do not (splits that are merged).

Tolerance: as for the tiny configuration.  Both sides differ by fp32 rounding of sums of at most 320 terms only, 320 x 2^-24
of logits of order 1, a few 1e-5; a wrong row, column or page is off by the logits' own size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.mark.parametrize("batch,rows,chunk,vocab,heads", [
    (1, 9, 64, 1001, 6), (1, 32, 64, 1001, 6), (3, 33, 8192, 97, 6), (2, 65, 8192, 1001, 1), (1, 70, 8192, 16385, 6),
    (1, 128, 1, 97, 6), (2, 129, 1, 1001, 6), (3, 40, 1, 1001, 1), (8, 12, 1, 97, 6), (9, 12, 1, 97, 6)])
def test_fp32_edges(batch, rows, chunk, vocab, heads):
    import torch
    from oracle import rsd_oracle as O
    from paper_2501_19324_amd import binding as R
    from rsd_inputs import ModelShape, model_blob_torch, model_weights_np
    shape = ModelShape(2, 192, 6, 3, 320, vocab, dtype="f32") if heads == 6 else ModelShape(1, 128, 1, 1, 320, vocab, dtype="f32")
    stub = ModelShape(1, 64, 2, 2, 64, vocab, dtype="f32")
    shapes = [shape, stub, ModelShape(1, 64, 2, 2, 64, vocab, dtype="f32", head_kind="reward")]
    blobs = [model_blob_torch(7, i, s, torch.device("cuda")) for i, s in enumerate(shapes)]
    torch.cuda.synchronize()
    ctx = R.rsd_init(shapes, blobs, batch=batch, delta=0.5, sep_id=vocab - 1, step_cap=1, max_steps=1, max_ctx=rows)
    rng = np.random.default_rng(rows)
    lens = np.array([max(1, rows - 5 * b) for b in range(batch)], np.int32)
    toks = rng.integers(0, vocab, size=(batch, rows)).astype(np.int32)
    out = R.rsd_forward(ctx, 0, toks, lens, chunk).cpu().numpy()
    m = O.OracleModel(shape, model_weights_np(7, 0, shape))
    for b in range(batch):
        ref = O.lm_logits(m, O.forward_full(m, [int(t) for t in toks[b, :lens[b]]]))
        assert np.max(np.abs(out[b, :lens[b]] - ref)) < TOL, b
    R.rsd_destroy(ctx)
