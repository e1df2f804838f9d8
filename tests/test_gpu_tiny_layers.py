"""The two-launch layers of small fp32 models at the edges of their range: one and eight rows (nine take the general path), contexts
that cross 64 positions and reach the last one (128), one to eight heads per KV head, MLPs of one slice up to the most slices whose partial
sums a block adds, vocabularies that end inside a block, fill the 64 blocks of the arg max, and exceed them.  Every greedy token is
compared with rsd_forward in one chunk, which runs the tile kernels: equal, or the two logits closer than 1e-5 (fp32 sums in
different order, logits of order one: 1e-6)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,d,hkv,ffn,vocab,prompt,cap", [
    (1, 128, 1, 64, 1000, 5, 20), (8, 256, 1, 1024, 4096, 63, 65), (8, 128, 4, 2048, 4097, 30, 40), (3, 256, 8, 128, 65, 60, 12),
    (9, 128, 2, 512, 1024, 9, 6), (5, 256, 2, 1024, 1024, 64, 8)])
def test_tokens_against_chunked_evaluation(batch, d, hkv, ffn, vocab, prompt, cap):
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from dataclasses import replace
    from paper_2501_19324_amd import binding as R
    from paper_2501_19324_amd.harness import Session
    from rsd_inputs import workload

    w = workload("cfg0", batch=batch, prompt_len_min=prompt, prompt_len_max=prompt, step_cap=cap, max_steps=1, deltas=(1.01,), sep_logit_bias=0.3)
    shape = replace(w.draft, n_layers=2, d_model=d, n_heads=d // 32, n_kv_heads=hkv, d_ffn=ffn, vocab=vocab)
    w = replace(w, draft=shape, target=replace(shape, n_layers=3), prm=replace(w.prm, vocab=vocab), sep_id=vocab - 1)
    s = Session(w)
    assert w.max_ctx <= 128
    rec = R.rsd_step(s.ctx)
    T = w.max_ctx
    for which, toks, n in ((0, rec["draft_tokens"], rec["draft_len"]), (1, rec["final_tokens"], rec["final_len"])):
        full = np.zeros((batch, T), dtype=np.int32)
        for b in range(batch):
            full[b, :prompt] = s.tokens_host[b, :prompt]
            full[b, prompt:prompt + n[b]] = toks[b, :n[b]]
        out = R.rsd_forward(s.ctx, which, full, (prompt + n).astype(np.int32), T).cpu().numpy()
        out[:, :, vocab - 1] += np.float32(0.3)
        for b in range(batch):
            assert n[b] >= 1
            for j in range(int(n[b])):
                z = out[b, prompt - 1 + j]
                assert z.max() - z[toks[b, j]] <= 1e-5, (which, b, j)
    s.close()
