"""Chunked passes whose output is read at each sequence's last token only: the last layer runs on those rows alone.  A reasoning step
is compared with rsd_forward in chunks, which evaluates every row of every layer, on either side of the sizes at which the short
way is taken (65 rows in bf16, nine in fp32, half of the rows kept), with one, a few and more than 64 rows kept, with one and two layers,
and over two passes of 8192 rows that cut a sequence in two.

Tolerances: both ways have the same precision and sum in different order; in bf16 a cache entry may be rounded the other way.  Rewards
1e-3 (measured against 64 bits: 3e-5 to 2e-4), fp32 1e-5; a greedy token may differ where the two best logits are closer than
2e-2 (logits 3e-3 off at most, either way)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BF16 = [([64], 2), ([65], 2), ([1] * 66, 2), ([2] * 33, 2), ([1, 66], 1), ([3, 1, 90], 2), ([2] * 70, 1), ([1000] * 9, 1)]
FP32 = [([8], 2), ([9], 2), ([1, 1, 1, 5], 1), ([3] * 4, 2), ([3] * 9, 2)]


@pytest.mark.parametrize("cfg,lens,layers", [("cfg1",) + c for c in BF16] + [("cfg0",) + c for c in FP32],
                         ids=lambda v: f"{len(v)}x{max(v)}" if isinstance(v, list) else str(v))
def test_step_against_all_rows(cfg, lens, layers):
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2501_19324_amd import binding as R
    from paper_2501_19324_amd.harness import Session
    from rsd_inputs import workload

    f32 = cfg == "cfg0"
    w = workload(cfg, n_layers=layers, vocab=None if f32 else 4096, batch=len(lens), prompt_len_min=max(lens), prompt_len_max=max(lens),
                 step_cap=4, max_steps=1, temperature=0.0, top_p=1.0, deltas=(1.01,), sep_logit_bias=0.0)
    s = Session(w)
    plen = np.array(lens, dtype=np.int32)
    R.rsd_set_prompts(s.ctx, s.tokens, plen)
    rec = R.rsd_step(s.ctx)
    T = int(max(lens)) + 4
    for which, toks, n in ((0, rec["draft_tokens"], rec["draft_len"]), (1, rec["final_tokens"], rec["final_len"])):
        full = np.zeros((len(lens), T), dtype=np.int32)
        for b, p in enumerate(lens):
            full[b, :p] = s.tokens_host[b, :p]
            full[b, p:p + n[b]] = toks[b, :n[b]]
        out = R.rsd_forward(s.ctx, which, full, plen + n, T)
        for b, p in enumerate(lens):
            for j in range(int(n[b])):
                z = out[b, p - 1 + j]
                best = float(z.max())
                assert best - float(z[int(toks[b, j])]) <= (1e-5 if f32 else 2e-2), (which, b, j)
        if which == 0:
            r = R.rsd_forward(s.ctx, 2, full, plen + n, T).cpu().numpy()
            for b, p in enumerate(lens):
                assert abs(float(rec["reward"][b]) - float(r[b, p + n[b] - 1])) < (1e-5 if f32 else 1e-3), b
    s.close()
