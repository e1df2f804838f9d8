"""Decode stages whose sequences end at different lengths: every 16 iterations the sequences still at work move together into fewer rows
(200 -> 128 -> 64 -> 32, 70 -> 64 -> 32).  The step is fixed by a teacher; every token the models would have chosen themselves is compared
with rsd_forward on the same tokens, evaluated in one chunk.  A token may differ where the two best logits are closer than 2e-2 (both
ways are within 3e-3 of the 64-bit value; a cache entry may be rounded either way)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,cap,alive", [(70, 40, (60, 20)), (200, 70, (190, 120, 50, 3)), (40, 33, (32, 1))])
def test_rows_given_up_by_finished_sequences(batch, cap, alive):
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2501_19324_amd import binding as R
    from paper_2501_19324_amd.harness import Session
    from rsd_inputs import workload

    w = workload("cfg1", n_layers=1, vocab=4096, batch=batch, prompt_len_min=3, prompt_len_max=9, step_cap=cap, max_steps=1, temperature=0.0,
                 top_p=1.0, deltas=(0.5,), sep_logit_bias=0.0)
    s = Session(w)
    rng = np.random.default_rng(batch)

    def forced():
        # alive[i] sequences go on beyond 16 (i + 1) tokens; which ones is drawn
        n = np.zeros(batch, dtype=np.int64)
        order = rng.permutation(batch)
        bounds = (batch,) + alive + (0,)
        for i in range(len(bounds) - 1):
            for b in order[bounds[i + 1]:bounds[i]]:
                n[b] = rng.integers(16 * i + 1, min(cap, 16 * (i + 1)) + 1)
        t = rng.integers(0, 4095, (batch, 1, cap)).astype(np.int32)
        for b in range(batch):
            if n[b] < cap:
                t[b, 0, n[b] - 1] = 4095
        return t, n

    (fd, nd), (ft, nt) = forced(), forced()
    keep = np.zeros((batch, 1), dtype=np.int32)                     # every step is rejected: the target serves all rows
    dev = [torch.from_numpy(a).cuda() for a in (fd, ft, keep)]
    R.rsd_set_teacher(s.ctx, *dev)
    s.reset()
    rec = R.rsd_step(s.ctx)
    assert list(rec["draft_len"]) == list(nd) and list(rec["final_len"]) == list(nt)
    own = R.rsd_export_sampled(s.ctx)
    rows = [R.rsd_iter_rows(s.ctx, m) for m in (0, 1)]
    assert max(rows) < batch * (cap - 1)                            # (rows were given up)
    T = int(s.prompt_len.max()) + cap
    for which, toks, n, mine in ((0, fd, nd, own[0]), (1, ft, nt, own[1])):
        full = np.zeros((batch, T), dtype=np.int32)
        for b, p in enumerate(s.prompt_len):
            full[b, :p] = s.tokens_host[b, :p]
            full[b, p:p + n[b]] = toks[b, 0, :n[b]]
        out = R.rsd_forward(s.ctx, which, full, (s.prompt_len + n).astype(np.int32), T)
        best = out.max(dim=-1).values.cpu().numpy()
        for b, p in enumerate(s.prompt_len):
            idx = torch.from_numpy(np.array(mine[b, 0, :n[b]], dtype=np.int64)).cuda()
            got = out[b, p - 1:p - 1 + n[b]].gather(1, idx[:, None])[:, 0].cpu().numpy()
            assert (best[b, p - 1:p - 1 + n[b]] - got <= 2e-2).all(), (which, b)
    R.rsd_set_teacher(s.ctx, None, None, None)
    s.close()
