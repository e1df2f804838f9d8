"""The many-row GEMM (chunked passes of more than 64 rows) at the edges of its tiles: row counts around multiples of 128
and 256, matrices whose sides are no multiple of any tile, an odd vocabulary, K sliced and not.

Small model: against the fp64 checker.  Full widths: against the same model evaluated in passes of 64 rows, which other
kernels serve.  Both sides keep 16 bits of every activation, so they differ by the flips of single bf16 cache entries only:
a flip moves one key or value by 2^-8 of itself, which the softmax average and the projections spread to less than the
2e-2 the bf16 tests allow; a wrong row or column of a tile is off by the logits' own size (0.5 rms and more)."""
import functools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 2e-2


def build(shape, vocab, max_ctx, batch=1):
    import torch
    from dataclasses import replace
    from rsd_inputs import ModelShape, model_blob_torch
    from paper_2501_19324_amd import binding as R
    stub = ModelShape(1, 128, 1, 1, 64, vocab)
    shapes = [shape, stub, replace(stub, head_kind="reward")]
    blobs = [model_blob_torch(7, i, s, torch.device("cuda")) for i, s in enumerate(shapes)]
    torch.cuda.synchronize()
    ctx = R.rsd_init(shapes, blobs, batch=batch, delta=0.5, sep_id=vocab - 1, step_cap=1, max_steps=1, max_ctx=max_ctx)
    return R, ctx


@pytest.mark.parametrize("rows", [65, 128, 129, 255, 257, 390])
def test_small_model_against_the_checker(rows):
    from oracle import rsd_oracle as O
    from rsd_inputs import ModelShape, model_weights_np
    shape = ModelShape(2, 640, 5, 5, 448, 1001)          # N = 1920, 640, 896, 1001; K = 640, 448
    R, ctx = build(shape, 1001, 400)
    toks = np.random.default_rng(rows).integers(0, 1001, size=(1, rows)).astype(np.int32)
    out = R.rsd_forward(ctx, 0, toks, np.array([rows], np.int32), 8192).cpu().numpy()[0]
    m = O.OracleModel(shape, model_weights_np(7, 0, shape))
    ref = O.lm_logits(m, O.forward_full(m, [int(t) for t in toks[0]], "bf16"))
    assert np.max(np.abs(out - ref)) < TOL
    R.rsd_destroy(ctx)


@pytest.mark.parametrize("width,rows", [("7B", 129), ("7B", 700), ("7B", 2049), ("1.5B", 257), ("1.5B", 1100)])
def test_full_width_against_few_row_passes(width, rows):
    from rsd_inputs import ModelShape
    dims = {"7B": (3584, 28, 4, 18944), "1.5B": (1536, 12, 2, 8960)}[width]
    R, ctx = build(ModelShape(1, *dims, 4097), 4097, rows)
    toks = np.random.default_rng(rows).integers(0, 4097, size=(1, rows)).astype(np.int32)
    lens = np.array([rows], np.int32)
    whole = R.rsd_forward(ctx, 0, toks, lens, 8192)
    pieces = R.rsd_forward(ctx, 0, toks, lens, 64)
    assert float((whole - pieces).abs().max()) < TOL
    R.rsd_destroy(ctx)


@pytest.mark.parametrize("chunk", [2, 5, 16, 17, 33, 200])
def test_chunked_attention_at_the_edges_of_its_work_items(chunk):
    """Pieces that end inside a work item of 16 rows, a wave's four rows, a page and a two-page step; 8 query heads per KV
    head; contexts split over several blocks (short passes over more than 8 pages) and not."""
    from oracle import rsd_oracle as O
    from rsd_inputs import ModelShape, model_weights_np
    shape = ModelShape(1, 1024, 8, 1, 64, 501)
    lens = np.array([200, 37, 1], np.int32)
    R, ctx = build(shape, 501, 201, batch=3)
    toks = np.random.default_rng(chunk).integers(0, 501, size=(3, 200)).astype(np.int32)
    out = R.rsd_forward(ctx, 0, toks, lens, chunk).cpu().numpy()
    m = O.OracleModel(shape, model_weights_np(7, 0, shape))
    for b in range(3):
        ref = O.lm_logits(m, O.forward_full(m, [int(t) for t in toks[b, :lens[b]]], "bf16"))
        assert np.max(np.abs(out[b, :lens[b]] - ref)) < TOL, b
    R.rsd_destroy(ctx)


def test_large_scores_survive_the_merge_of_splits():
    """Scores of 33400 (in units of log2) that differ little, so that every split of the context has weight: 16 rows over 400 tokens
    in eight splits against the same rows in one (nine copies of the sequence: more rows than are split).  All weights are
    zero but for one column per output, so both sides compute the same q, k, v and scores bit for bit, whatever their
    kernels' order of summation; what differs is the merge.  The output is 64 x the weighted mean of values +1 and -1:
    probabilities and output are kept as two bf16 halves (2^-17 each, on either side), 4 x 64 x 2^-17 = 2e-3.  Maxima rounded on their
    way to the merge move a split's weight by up to 2^-24 x 33400 = 2e-3 each way and the output by up to 0.1 (0.033 here)."""
    import torch
    from dataclasses import replace
    from rsd_inputs import ModelShape, blob_layout, model_blob_torch
    from paper_2501_19324_amd import binding as R
    n, vocab = 400, 16
    shape = ModelShape(1, 1024, 8, 1, 64, vocab)
    layout, total = blob_layout(shape)
    blob = torch.zeros(total, dtype=torch.bfloat16, device="cuda")
    t = {name: blob[off:off + r * c].view(r, c) for name, r, c, off in layout}
    for name in t:
        if "norm" in name:
            t[name].fill_(1.0)
    t["embed"].fill_(1.0)
    t["embed"][1::2, 1] = -1.0                              # odd tokens: value -1
    for h in range(8):
        t["l0.wq"][h * 128 + 63, 0] = 512.0                 # the slowest rotary pair: cos(1.15e-4 x distance)
    t["l0.wk"][63, 0] = 512.0
    t["l0.wv"][0, 1] = 1.0
    t["l0.wo"][2, 0] = 64.0
    t["lm_head"][0, 2] = 1.0
    stub = ModelShape(1, 128, 1, 1, 64, vocab)
    shapes = [shape, stub, replace(stub, head_kind="reward")]
    stubs = [model_blob_torch(7, i, shapes[i], torch.device("cuda")) for i in (1, 2)]
    torch.cuda.synchronize()
    toks = np.repeat(np.random.default_rng(1).integers(0, vocab, 25), 16)[None, :].astype(np.int32)      # runs of equal values
    out = []
    for batch in (1, 9):
        ctx = R.rsd_init(shapes, [blob] + stubs, batch=batch, delta=0.5, sep_id=vocab - 1, step_cap=1, max_steps=1, max_ctx=n + 1)
        out.append(R.rsd_forward(ctx, 0, np.repeat(toks, batch, 0), np.full(batch, n, np.int32), 16)[0, :, 0])
        R.rsd_destroy(ctx)
    assert float(out[1].abs().max()) > 5.0                   # (the values are there)
    err = float((out[0] - out[1]).abs().max())
    assert err < 2e-3, err


@pytest.mark.parametrize("rows", [2, 31, 33, 64, 65, 127, 128])
@pytest.mark.parametrize("ffn", [5248, 8320, 12864])
def test_unsliced_gate_up_and_head(rows, ffn):
    """The kernel without K slices (2..128 rows, matrices of 160..256 row blocks): gate/up pairs that its blocks of 32, 48 and
    80 units cut evenly and not, a head of an odd vocabulary, row counts around its tiles of 32, 64 and 128."""
    from oracle import rsd_oracle as O
    from rsd_inputs import ModelShape, model_weights_np
    shape = ModelShape(1, 128, 1, 1, ffn, 10241)
    R, ctx = build(shape, 10241, 129)
    toks = np.random.default_rng(rows).integers(0, 10241, size=(1, rows)).astype(np.int32)
    out = R.rsd_forward(ctx, 0, toks, np.array([rows], np.int32), 128).cpu().numpy()[0]
    m = O.OracleModel(shape, model_weights_np(7, 0, shape))
    ref = O.lm_logits(m, O.forward_full(m, [int(t) for t in toks[0]], "bf16"))
    assert np.max(np.abs(out - ref)) < TOL / 4           # (logits of rms 0.2)
    R.rsd_destroy(ctx)


@functools.lru_cache(maxsize=1)
def stream_model(ffn, vocab):
    from oracle import rsd_oracle as O
    from rsd_inputs import ModelShape, model_weights_np
    shape = ModelShape(1, 896, 7, 7, ffn, vocab)
    return shape, O.OracleModel(shape, model_weights_np(7, 0, shape, threads=8))


@pytest.mark.parametrize("ffn,vocab", [(5248, 10241), (8320, 16449), (12864, 25601)])
@pytest.mark.parametrize("rows", [17, 33, 65, 128])
def test_unsliced_kernel_around_its_ring(ffn, vocab, rows):
    """The same kernel with K = 896, 14 K blocks: its ring of three to six stages wraps several times and ends in another stage
    than it began; gate/up pair and head of every block width (64, 96, 160), one, two and four row tiles.  (With K = 128, as
    above, no stage is ever used twice.)"""
    from oracle import rsd_oracle as O
    shape, m = stream_model(ffn, vocab)
    R, ctx = build(shape, vocab, 129)
    toks = np.random.default_rng(rows).integers(0, vocab, size=(1, rows)).astype(np.int32)
    out = R.rsd_forward(ctx, 0, toks, np.array([rows], np.int32), 128).cpu().numpy()[0]
    ref = O.lm_logits(m, O.forward_full(m, [int(t) for t in toks[0]], "bf16"))
    assert np.max(np.abs(out - ref)) < TOL / 4           # (logits of rms 0.6; a stage read too early or late is off by that)
    R.rsd_destroy(ctx)


def test_rows_wider_than_a_block():
    """d_model beyond what a block of 1024 threads covers in two rounds (16896 = 4.1 rounds: the gather with its norm and the
    splits walk on beyond what a block keeps in registers): few-row passes against single-row ones, which gather and normalise
    in other kernels."""
    from rsd_inputs import ModelShape
    R, ctx = build(ModelShape(1, 16896, 132, 22, 128, 97), 97, 40)
    toks = np.random.default_rng(3).integers(0, 97, size=(1, 40)).astype(np.int32)
    lens = np.array([40], np.int32)
    one = R.rsd_forward(ctx, 0, toks, lens, 1)
    for chunk in (2, 40):
        assert float((R.rsd_forward(ctx, 0, toks, lens, chunk) - one).abs().max()) < TOL
    R.rsd_destroy(ctx)


def test_silu_keeps_fp32_accuracy():
    """The activation of the matrix kernels' epilogues (the debug build exposes it) against 64 bits.  Bound: the exponential is good
    to one ulp (2^-23) and enters weighted with e / (1 + e) <= 1; the sum, the quotient and the product round once each (2^-24):
    5 x 2^-24 = 3.0e-7, whatever |g| is.  Where exp(-g) overflows the result is 0, and -inf and NaN
    give NaN, as in the plain formula (+inf may give either: its halves, inf and inf - inf, are no number anyway)."""
    import ctypes
    import os
    import torch
    from paper_2501_19324_amd import binding as R
    dbg = ctypes.CDLL(os.path.join(os.path.dirname(R.LIB_PATH), "librsd_debug.so"))
    n = 1 << 20

    def run(g, u):
        g, u = (torch.from_numpy(a).cuda() for a in (g, u))
        x = torch.empty_like(g)
        torch.cuda.synchronize()
        assert dbg.rsd_debug_silu(ctypes.c_void_p(g.data_ptr()), ctypes.c_void_p(u.data_ptr()), ctypes.c_void_p(x.data_ptr()), g.numel()) == 0
        return x.cpu().numpy()

    rng = np.random.default_rng(0)
    for lo, hi in ((-88.7, 90.0), (-20.0, 20.0), (-1.0, 1.0), (-88.7, -87.0)):
        g = rng.uniform(lo, hi, n).astype(np.float32)
        u = rng.uniform(0.5, 2.0, n).astype(np.float32)
        want = g.astype(np.float64) / (1.0 + np.exp(-g.astype(np.float64))) * u
        err = np.abs(run(g, u) - want) / np.abs(want)
        assert err.max() < 5 * 2.0 ** -24, (lo, hi, err.max())
    g = np.zeros(512, np.float32)
    g[:9] = [np.inf, -np.inf, np.nan, -100.0, -3e38, 3e38, 1e-40, -0.0, 105.0]
    x = run(g, np.ones(512, np.float32))
    assert not np.isfinite(x[0]) and np.isnan(x[1]) and np.isnan(x[2]) and x[3] == 0 and x[4] == 0 and x[5] == np.float32(3e38)
    assert abs(x[6] - 5e-41) < 1e-44 and x[7] == 0 and x[8] == 105.0 and not x[9:].any()


@pytest.mark.parametrize("vocab", [1001, 4096])
@pytest.mark.parametrize("chunk", [2, 7, 40])
def test_short_pieces_share_the_head(vocab, chunk):
    """Chunked evaluation of several ragged sequences, whose pieces go through the output head together, against the same
    sequences one at a time; with and without pieces of a single row; nothing is written behind the end of a sequence."""
    from rsd_inputs import ModelShape
    shape = ModelShape(2, 640, 5, 5, 448, vocab)
    toks = np.random.default_rng(vocab + chunk).integers(0, vocab, (3, 41)).astype(np.int32)
    R, ctx = build(shape, vocab, 64, batch=3)
    R1, one = build(shape, vocab, 64)
    for lens in ([41, 40, 41], [41, 22, 9], [36, 1, 29]):
        out = R.rsd_forward(ctx, 0, toks, np.array(lens, np.int32), chunk).cpu().numpy()
        for b, n in enumerate(lens):
            ref = R1.rsd_forward(one, 0, toks[b:b + 1], np.array([n], np.int32), chunk).cpu().numpy()[0]
            assert np.max(np.abs(out[b, :n] - ref[:n])) < TOL / 4, (lens, b)       # (logits of rms 0.5)
            assert np.isnan(out[b, n:]).all()
    R.rsd_destroy(ctx)
    R1.rsd_destroy(one)


def test_a_piece_of_one_row_leaves_the_others_their_shared_head():
    """32 sequences in chunks of 5, a head of 65536 x 1536 (200 MB): where one of them ends on a single row the others still share
    the head.  That row costs the head's weights once more (by bytes 35 us; a pass over 160 rows takes several times as
    long); one product per sequence made the pass four times as long.  Shortest of ten calls each."""
    import time
    from rsd_inputs import ModelShape
    R, ctx = build(ModelShape(1, 1536, 12, 2, 8960, 65536), 65536, 16, batch=32)
    toks = np.random.default_rng(0).integers(0, 65536, (32, 10)).astype(np.int32)

    def seconds(lens):
        best = 1e9
        for _ in range(11):
            t0 = time.perf_counter()
            R.rsd_forward(ctx, 0, toks, lens, 5)
            best = min(best, time.perf_counter() - t0)
        return best

    even, odd = np.full(32, 10, np.int32), np.full(32, 10, np.int32)
    odd[13] = 6
    assert seconds(odd) < 1.3 * seconds(even)
    R.rsd_destroy(ctx)


@pytest.mark.parametrize("chunk", [2, 3, 8, 9])
def test_fp32_pieces_of_few_rows_keep_their_head(chunk):
    """fp32 weights: pieces of up to eight rows go through the output head by themselves, in the kernel whose sums are more accurate,
    beside a piece of one row and (chunk 9) longer ones that share theirs.  All layer weights are zero, so that the hidden
    rows are the embeddings bit for bit, and the logits of such a piece do not depend on its neighbours either."""
    import torch
    from dataclasses import replace
    from rsd_inputs import ModelShape, blob_layout
    from paper_2501_19324_amd import binding as R
    vocab, B = 1000, 5
    shape = ModelShape(1, 1536, 12, 2, 64, vocab, "f32")
    layout, total = blob_layout(shape)
    g = torch.Generator(device="cuda").manual_seed(3)
    blob = torch.zeros(total, device="cuda")
    for name, r, c, off in layout:
        if not name.startswith("l0.") or "norm" in name:
            blob[off:off + r * c].normal_(1.0 if "norm" in name else 0.0, 0.02, generator=g)
    stub = ModelShape(1, 128, 1, 1, 64, vocab, "f32")
    shapes = [shape, stub, replace(stub, head_kind="reward")]
    blobs = [blob] + [torch.zeros(blob_layout(s)[1], device="cuda") for s in shapes[1:]]
    torch.cuda.synchronize()
    ctx, one = (R.rsd_init(shapes, blobs, batch=b, delta=0.5, sep_id=vocab - 1, step_cap=1, max_steps=1, max_ctx=40) for b in (B, 1))
    toks = np.random.default_rng(chunk).integers(0, vocab, (B, 2 * chunk)).astype(np.int32)
    lens = np.array([2 * chunk, 2 * chunk - 1, 2 * chunk, chunk + 1, 2 * chunk], np.int32)
    out = R.rsd_forward(ctx, 0, toks, lens, chunk)
    for b, n in enumerate(lens):
        ref = R.rsd_forward(one, 0, toks[b:b + 1, :n].copy(), lens[b:b + 1], chunk)[0]
        for s in range(0, n, chunk):
            e = min(s + chunk, n)
            assert torch.equal(out[b, s:e], ref[s:e]) if e - s <= 8 else float((out[b, s:e] - ref[s:e]).abs().max()) < 1e-5, (b, s)
        assert bool(torch.isnan(out[b, n:]).all())
    R.rsd_destroy(ctx)
    R.rsd_destroy(one)


def tile_product(dbg, w, xh, xl, epi, bm, bn, ks=1, y=None, ldy=0, oh=None, ol=None):
    import ctypes
    import torch
    torch.cuda.synchronize()
    ptr = [ctypes.c_void_p(t.data_ptr() if t is not None else None) for t in (w, xh, xl, y, oh, ol)]
    rc = dbg.rsd_debug_tile(ptr[0], w.shape[0], w.shape[1], ptr[1], ptr[2], xh.shape[0], epi, bm, bn, ks, ptr[3], ldy, ptr[4], ptr[5])
    assert rc == 0


def tile_operands(M, N, K, seed):
    """bf16 W [N][K], and fp32 X [M][K] as hi + lo bf16 halves; the product and the sum of the terms' magnitudes in 64 bits"""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn(N, K, generator=g, device="cuda").bfloat16()
    x = torch.randn(M, K, generator=g, device="cuda")
    xh = x.bfloat16()
    xl = (x - xh.float()).bfloat16()
    x64, w64 = xh.double() + xl.double(), w.double()
    return w, xh, xl, x64 @ w64.T, x64.abs() @ w64.abs().T


TILES = [(256, 256), (256, 192), (128, 256), (128, 192), (128, 128)]
STORE, RESID, SWIGLU = 0, 1, 2


@pytest.mark.parametrize("bm,bn", TILES)
@pytest.mark.parametrize("K", [64, 128, 192, 448])
def test_every_tile_and_epilogue(bm, bn, K):
    """Each instance of the many-row kernel by itself (the debug build launches it), whatever the plan would choose: one, two, three and
    seven K blocks in its ring, rows and columns just below, at and above the tile, N no multiple of four, an output at an odd
    address or row pitch (values are then stored one by one), K in slices, among them an empty one; nothing is written beside
    the output.  Bound of a product: 2 K terms summed in fp32 in any order, 2 K 2^-24 times the sum of their magnitudes, once more
    for the residual; SwiGLU: silu has a slope below 1.1, 5 x 2^-24 of its own, and its result is kept in two halves (2^-17)."""
    import torch
    import ctypes
    import os
    from paper_2501_19324_amd import binding as R
    dbg = ctypes.CDLL(os.path.join(os.path.dirname(R.LIB_PATH), "librsd_debug.so"))
    eps = 2 * K * 2.0 ** -24
    for i, (M, N) in enumerate([(bm - 1, bn + 4), (bm, bn), (bm + 1, bn - 1), (2 * bm + 17, 2 * bn + 30), (1, 1), (3, 2 * bn + 20)]):
        w, xh, xl, want, mag = tile_operands(M, N, K, i)
        for pitch, off in ((N, 0), (N + 3, 1), (N + 4, 0)):
            for epi in (STORE, RESID):
                buf = torch.randn(M * pitch + 64, device="cuda")
                kept = buf.clone()
                rows = torch.arange(M, device="cuda")[:, None] * pitch + torch.arange(N, device="cuda")[None, :] + off
                y0 = kept[rows].double() if epi == RESID else 0.0
                tile_product(dbg, w, xh, xl, epi, bm, bn, y=buf[off:], ldy=pitch)
                bound = eps * mag + (2.0 ** -23 * (want.abs() + y0.abs()) if epi == RESID else 0.0)
                assert bool(((buf[rows].double() - (want + y0)).abs() <= bound).all()), (M, N, pitch, off, epi)
                buf[rows] = kept[rows]
                assert torch.equal(buf, kept), (M, N, pitch, off, epi)
        for ks in (2, 3, 4):
            buf = torch.full((ks * M * N + 64,), 7.0, device="cuda")
            tile_product(dbg, w, xh, xl, STORE, bm, bn, ks=ks, y=buf, ldy=N)
            got = buf[:ks * M * N].view(ks, M, N).double().sum(0)
            assert bool(((got - want).abs() <= eps * mag).all()) and bool((buf[ks * M * N:] == 7.0).all()), (M, N, ks)
    for i, (M, F) in enumerate([(bm - 1, 64), (bm + 1, bn // 2 // 64 * 64 + 64), (2 * bm, 192)]):
        w, xh, xl, want, mag = tile_operands(M, 2 * F, K, 9 + i)
        oh, ol = (torch.full((M * F + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        tile_product(dbg, w, xh, xl, SWIGLU, bm, bn, oh=oh, ol=ol)
        g, u = want[:, :F], want[:, F:]
        silu = g * torch.sigmoid(g)
        got = (oh.double() + ol.double())[:M * F].view(M, F)
        bound = eps * (1.1 * mag[:, :F] * u.abs() + silu.abs() * mag[:, F:] + 1.1 * eps * mag[:, :F] * mag[:, F:]) + (2.0 ** -17 + 5 * 2.0 ** -24) * (silu * u).abs()
        assert bool(((got - silu * u).abs() <= bound + 1e-30).all()), (M, F)
        assert bool((oh[M * F:] == 7.0).all()) and bool((ol[M * F:] == 7.0).all())
