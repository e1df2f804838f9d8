"""The timing probes bench.py reports from (rsd_probe_start / rsd_probe_read / rsd_probe_clock): the accounting of
algorithmic flops and bytes is exact, the times are positive, and the shader clock read inside the probed
many-row GEMM is a plausible clock of this part.  No numerics here: the same passes are compared with the
checker in test_gpu_bf16.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PREFILL, DECODE = 1, 0
OP_GATE_UP, OP_DOWN = 2, 3


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2501_19324_amd import binding as R
    from paper_2501_19324_amd.harness import Session
    return dict(R=R, Session=Session)


def small_workload(batch):
    from rsd_inputs import workload
    return workload("cfg1", n_layers=2, vocab=4096, batch=batch, prompt_len_min=20, prompt_len_max=70, step_cap=8,
                    max_steps=3, temperature=0.0, top_p=1.0, deltas=(0.6,))


def test_chunked_pass_probe_counts_flops_and_reads_the_clock(gpu):
    R = gpu["R"]
    w = small_workload(4)
    s = gpu["Session"](w)
    T = 80
    lens = np.full(4, T, dtype=np.int32)
    toks = np.random.default_rng(5).integers(0, w.draft.vocab, size=(4, T)).astype(np.int32)
    prm = 2
    shape = w.shapes[prm]
    R.rsd_probe_start(s.ctx, 0, prm, PREFILL, OP_GATE_UP, 64, 1)
    R.rsd_probe_start(s.ctx, 1, prm, PREFILL, OP_DOWN, 64, 1)
    R.rsd_forward(s.ctx, prm, toks, lens, T)        # one chunked pass of 4 x 80 = 320 rows: the many-row GEMM
    clk = [R.rsd_probe_clock(s.ctx, slot) for slot in (0, 1)]
    rec = [R.rsd_probe_read(s.ctx, slot) for slot in (0, 1)]
    rows, d, F, L = 4 * T, shape.d_model, shape.d_ffn, shape.n_layers
    assert rec[0]["n"] == L and rec[1]["n"] == L
    assert rec[0]["total_flops"] == L * 2 * rows * (2 * F) * d
    assert rec[1]["total_flops"] == L * 2 * rows * d * F
    for r, c in zip(rec, clk):
        assert r["total_ms"] > 0
        assert c["launches"] == r["n"]
        mhz = c["shader_ticks"] / c["ref_ticks"] * 100.0
        print(f"shader clock inside the probed GEMM: {mhz:.0f} MHz over {c['launches']} launches")
        assert 50.0 < mhz < 3000.0          # a clock, not garbage; the value itself is a measurement, not a contract
    # a second arming starts from zero, and a pass of few rows (the weight-streaming kernels) reports no clock
    R.rsd_probe_start(s.ctx, 0, prm, PREFILL, OP_GATE_UP, 64, 1)
    R.rsd_forward(s.ctx, prm, toks[:, :8].copy(), np.full(4, 8, dtype=np.int32), 8)       # 32 rows
    c = R.rsd_probe_clock(s.ctx, 0)
    r = R.rsd_probe_read(s.ctx, 0)
    assert r["n"] == L and c["launches"] == 0 and c["shader_ticks"] == 0
    s.close()


def test_timed_iterations_of_the_tiny_configuration(gpu):
    """A generation with every second iteration timed chooses the same tokens as one that is not timed.  The heads make the order of the
    additions visible: their rows hold pairs v, -v in drawn places, so that a logit is nothing but the rounding errors of its sum.  All
    layers add zero to a state of ones."""
    import torch
    from dataclasses import replace
    from rsd_inputs import workload

    R = gpu["R"]
    w = workload("cfg0", max_steps=2, deltas=(1.01,), sep_logit_bias=-100.0)      # (no separator: steps of step_cap tokens)
    w = replace(w, draft=replace(w.draft, rms_eps=0.0), target=replace(w.target, rms_eps=0.0))
    rng = np.random.default_rng(7)
    weights = []
    for i, s in enumerate(w.shapes):
        d, kv, V = s.d_model, s.n_kv_heads * 32, s.vocab
        layers = s.n_layers * (2 * d + 2 * d * d + 2 * kv * d + 3 * d * s.d_ffn)
        if i == 2:
            weights.append(np.zeros(V * d + layers + d + d + 8, dtype=np.float32))
            continue
        v = rng.standard_normal((V, d // 2))
        head = rng.permuted(np.concatenate([v, -v], axis=1), axis=1)
        weights.append(np.concatenate([np.ones(V * d), np.zeros(layers), np.ones(d), head.reshape(-1)]).astype(np.float32))
    weights = [torch.from_numpy(b).cuda() for b in weights]
    torch.cuda.synchronize()

    def generate(model):
        s = gpu["Session"](w, weights=weights)
        ops = (0, 1, 2, 4)
        if model is not None:
            for slot, op in enumerate(ops):
                R.rsd_probe_start(s.ctx, slot, model, DECODE, op, 1024, 2)
        toks = [R.rsd_step(s.ctx) for _ in range(w.max_steps)]
        rec = [R.rsd_probe_read(s.ctx, slot) for slot in range(len(ops))] if model is not None else None
        s.close()
        return np.stack([t["draft_tokens"] for t in toks]), np.stack([t["final_tokens"] for t in toks]), rec

    plain = generate(None)
    assert (plain[0] >= 0).all() and (plain[1] >= 0).all()
    for model in (0, 1):
        timed = generate(model)
        assert (timed[0] == plain[0]).all() and (timed[1] == plain[1]).all(), model
        s, (qkv, out, gate_up, head) = w.shapes[model], timed[2]
        # iterations 0, 2, ... of the decode loops: 15 and 15 of the draft, which begins both steps with a chunked pass, 15 and 16 of the target
        n = -(-(2 * w.step_cap - 2 + model) // 2)
        d, B = s.d_model, w.batch
        assert qkv["n"] == out["n"] == gate_up["n"] == n * s.n_layers and head["n"] == n
        assert qkv["total_flops"] == out["total_flops"] == n * s.n_layers * 2 * B * d * (2 * d + 2 * s.n_kv_heads * 32)
        assert gate_up["total_flops"] == n * s.n_layers * 2 * B * 3 * d * s.d_ffn
        assert head["total_flops"] == n * 2 * B * d * s.vocab
        assert min(r["total_ms"] for r in timed[2]) > 0
