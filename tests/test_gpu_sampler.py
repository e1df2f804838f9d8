"""The sampler at the places where its selection changes path: a few and many rows for the vocabulary (span per block / per
wave), vocabularies
smaller than, and no multiple of, its 64 spans, a deciding bin that overflows the lists of some spans (logits that fall with the
id) or holds too many keys to be listed at all (equal and nearly equal logits), a threshold near the histogram's lower end,
top_p 0 and 1, masked tokens.

A draw is checked against the fp64 distribution: the token's interval of the nucleus's running mass must hold u.  The
kernel forms e = exp(x - max) in fp32 (a few ulp, 2^-22) and sums masses exactly, so interval ends and the nucleus's edge are
known to 1e-6 of the total mass; a token whose probability equals the edge within 2^-20 may be in or out."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def logits_of(kind, n, V, rng):
    if kind == "normal":
        return rng.normal(size=(n, V)) * 2.0
    if kind == "flat":                       # all equal: every token ties at the edge
        return np.zeros((n, V))
    if kind == "steps":                      # few distinct values: thousands of equal keys per bin
        return rng.integers(0, 3, size=(n, V)) * 0.5
    if kind == "near":                       # tens of thousands of different keys in a bin
        return rng.normal(size=(n, V)) * 0.01
    if kind == "ramp":                       # the deciding bin's keys are all in one or two spans
        return np.tile(np.linspace(0.0, -3.0, V), (n, 1))
    if kind == "low":                        # one token, and a tail of masses of a few units
        x = -26.5 + 0.4 * rng.normal(size=(n, V))
        x[:, V // 3] = 0.0
        return x
    if kind == "wide":                       # the tail lies far below 2^-32 of the top
        return np.where(rng.random((n, V)) < 0.01, rng.normal(size=(n, V)), -40.0 + rng.normal(size=(n, V)))
    x = rng.normal(size=(n, V))              # masked
    x[:, rng.random(V) < 0.7] = -np.inf
    x[:, V // 2] = 1.0
    return x


@pytest.mark.parametrize("kind", ["normal", "flat", "steps", "near", "ramp", "low", "wide", "masked"])
@pytest.mark.parametrize("n,V", [(1, 151936), (3, 32011), (4, 32011), (20, 20011), (5, 37), (17, 65)])
@pytest.mark.parametrize("T,top_p", [(0.7, 0.95), (1.0, 1.0), (1.0, 0.0), (0.5, 0.9999999)])
def test_draws_lie_where_the_distribution_puts_them(kind, n, V, T, top_p):
    import torch
    from paper_2501_19324_amd import binding as R
    rng = np.random.default_rng(V + n)
    lg = logits_of(kind, n, V, rng).astype(np.float32)
    u = rng.random(n).astype(np.float32)
    out = R.rsd_sample_static(torch.from_numpy(lg).cuda(), torch.from_numpy(u).cuda(), T, top_p).cpu().numpy()
    x = lg.astype(np.float64) / np.float64(np.float32(T))
    for i in range(n):
        e = np.exp(x[i] - x[i].max())
        e[e < 2.0 ** -40] = 0.0                                    # below the fixed-point unit: no mass
        order = np.sort(e)[::-1]
        reach = np.nonzero(np.cumsum(order) >= float(np.float32(top_p)) * e.sum() * (1 - 1e-7))[0]
        tau = order[reach[0]] if reach.size else order[order > 0][-1]
        t = int(out[i])
        assert 0 <= t < V and e[t] >= tau * (1 - 2.0 ** -20), (i, t, e[t], tau)
        # the edge itself may be one distinct value higher or lower: accept either nucleus
        edges = {tau, max(e[e < tau * (1 - 2.0 ** -20)], default=tau), min(e[e > tau * (1 + 2.0 ** -20)], default=tau)}
        ok = False
        for edge in edges:
            m = np.where(e >= edge * (1 - 2.0 ** -20), e, 0.0)
            c = np.cumsum(m)
            ok |= c[t] - m[t] - 1e-6 * c[-1] <= u[i] * c[-1] <= c[t] + 1e-6 * c[-1]
        assert ok, (kind, i, t)


@pytest.mark.parametrize("kind", ["normal", "flat", "masked"])
@pytest.mark.parametrize("n,V", [(1, 151936), (20, 20011), (5, 37)])
def test_a_uniform_of_one_draws_the_last_member(kind, n, V):
    """u = 1 leaves no span in which the running mass exceeds u times the total: the draw is the nucleus's last token (top_p 1:
    the last one with a mass), the same on every call."""
    import torch
    from paper_2501_19324_amd import binding as R
    lg = logits_of(kind, n, V, np.random.default_rng(V + n)).astype(np.float32)
    want = [np.nonzero(x.astype(np.float64) - x.max() > np.log(2.0 ** -40) + 1e-6)[0][-1] for x in lg]
    dev, u = torch.from_numpy(lg).cuda(), torch.ones(n, device="cuda")
    for _ in range(20):
        assert list(R.rsd_sample_static(dev, u, 1.0, 1.0).cpu().numpy()) == want


@pytest.mark.parametrize("V", [37, 20011])
@pytest.mark.parametrize("T,top_p", [(0.0, 1.0), (1.0, 0.9), (1.0, 1.0)])
def test_rows_without_a_finite_mass_give_ids_of_the_vocabulary(V, T, top_p):
    """All -inf, all NaN, one +inf (its exponential is NaN, all others are 0), all +inf, NaN beside -inf: there is nothing right to
    draw, but an engine looks the id up in the embedding.  A row with finite logits in the same call is drawn as usual."""
    import torch
    from paper_2501_19324_amd import binding as R
    lg = np.full((6, V), -np.inf, np.float32)
    lg[1] = np.nan
    lg[2] = 0.0; lg[2, V - 1] = np.inf
    lg[3] = np.inf
    lg[4, ::2] = np.nan
    lg[5] = -5.0; lg[5, V // 2] = 40.0
    u = torch.full((6,), 0.5, device="cuda")
    out = R.rsd_sample_static(torch.from_numpy(lg).cuda(), u, T, top_p).cpu().numpy()
    assert out.min() >= 0 and out.max() < V and out[5] == V // 2


@pytest.mark.parametrize("n", [1, 64])
@pytest.mark.parametrize("kind", ["flat", "near", "ramp", "steps"])
def test_nearly_equal_logits_cost_little_more(n, kind):
    """Rows whose deciding bin holds thousands of keys: selection over the whole row by one block took 9 to 17 times as long as a
    row of spread-out logits; spread over blocks it takes 1.3 to 1.8 times as long.  Shortest of five batches of calls."""
    import torch
    from paper_2501_19324_amd import binding as R
    u = torch.rand(n, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")

    def ms(k):
        lg = torch.from_numpy(logits_of(k, n, 151936, np.random.default_rng(2)).astype(np.float32)).cuda()
        e0, e1, best = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), 1e9
        for _ in range(5):
            e0.record()
            for _ in range(20):
                R.rsd_sample_static(lg, u, 1.0, 0.95)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    ms("normal")
    assert ms(kind) < 3.0 * ms("normal")


@pytest.mark.parametrize("kind", ["normal", "low", "wide", "masked"])
@pytest.mark.parametrize("n,V", [(19, 151936), (10, 70001)])
@pytest.mark.parametrize("T,top_p", [(0.7, 0.95), (1.0, 0.3), (0.6, 0.999)])
def test_tokens_too_light_for_a_bin(kind, n, V, T, top_p):
    """Spans of more than one batch on many rows, where tokens below the tail are only added up and those above it listed.
    (Not of 151936 nearly equal logits: with top_p 0.3 several of their distinct fp64 masses at the edge are one fp32 key, where the
    check accepts the edge's neighbours only.)"""
    test_draws_lie_where_the_distribution_puts_them(kind, n, V, T, top_p)


@pytest.mark.parametrize("kind", ["normal", "low", "masked"])
@pytest.mark.parametrize("n,V", [(20, 65536), (20, 65537), (20, 81920), (20, 81921), (2, 81920), (2, 81921), (2, 163840), (2, 163841)])
def test_spans_at_the_change_between_plain_and_longer_passes(kind, n, V):
    """Histogram: spans of 1024 tokens (one per wave) and 2560 (one per block) are the last that take the plain pass; selection: 1280."""
    test_draws_lie_where_the_distribution_puts_them(kind, n, V, 0.7, 0.95)


@pytest.mark.parametrize("n,V", [(2, 151936), (20, 151936), (33, 70000)])
def test_draws_do_not_depend_on_the_way_quotients_are_formed(n, V):
    """Logits and temperature times 2^61 have the same quotients, but leave the range of the division by reciprocal.  (Spans of 2374
    and 1094 tokens by waves, whose histogram pass divides that way; by blocks spans of 2374 take the plain pass.)"""
    import torch
    from paper_2501_19324_amd import binding as R
    rng = np.random.default_rng(n)
    lg = torch.from_numpy((rng.normal(size=(n, V)) * 3).astype(np.float32)).cuda()
    lg[:, V // 3] = -torch.inf
    for T in (0.7, 1.3):
        T = float(np.float32(T))
        for i in range(4):
            u = torch.from_numpy(rng.random(n).astype(np.float32)).cuda()
            a = R.rsd_sample_static(lg, u, T, 0.9).cpu().numpy()
            b = R.rsd_sample_static(lg * 2.0 ** 61, u, T * 2.0 ** 61, 0.9).cpu().numpy()
            assert (a == b).all(), (T, i)


def test_arg_max_between_calls_of_other_shapes():
    """The count of finished spans is kept from call to call: rows with a block per span and with four spans a block, and sampled calls
    in between, in turn."""
    import torch
    from paper_2501_19324_amd import binding as R
    rng = np.random.default_rng(5)
    for n, V in [(1, 151936), (64, 1000), (3, 50000), (64, 31), (1, 151936), (17, 32000), (2, 1)] * 3:
        lg = torch.from_numpy(rng.integers(-50, 50, size=(n, V)).astype(np.float32)).cuda()       # ties: the lowest id
        got = R.rsd_sample_static(lg, None, 0.0, 1.0).cpu().numpy()
        assert (got == np.argmax(lg.cpu().numpy(), axis=1)).all(), (n, V)
        R.rsd_sample_static(torch.zeros(n, V, device="cuda"), torch.rand(n, device="cuda"), 1.0, 0.9)


def debug_library():
    import ctypes
    import os
    from paper_2501_19324_amd import binding as R
    return ctypes.CDLL(os.path.join(os.path.dirname(R.LIB_PATH), "librsd_debug.so"))


def test_exponential_is_as_accurate_as_the_library_s():
    """The sampler's exponential (the debug build exposes it) over the differences that carry mass, -28 .. 0, against 64 bits, and
    expf on the same values.  Bound: the argument is exact to 2^-25 of an octave (n is an integer, the rest is at most 1/2 and known to
    2^-26, its sum rounds once more), which is 0.7 x 2^-25 = 2.1e-8 of the value, and the hardware's exponential is good to one ulp of
    a number in [0.7, 1.42), 2^-24 / 0.7 = 8.5e-8 at the worst: 1.1e-7.  An argument with the product's rounding error counted twice
    is up to 1.4e-6 off.  What is below -80, and what is no number, has no mass."""
    import ctypes
    import torch
    dbg = debug_library()

    def run(d):
        d = torch.from_numpy(d).cuda()
        e, lib = torch.empty_like(d), torch.empty_like(d)
        torch.cuda.synchronize()
        assert dbg.rsd_debug_smp_exp(*(ctypes.c_void_p(t.data_ptr()) for t in (d, e, lib)), d.numel()) == 0
        return e.cpu().numpy(), lib.cpu().numpy()

    rng = np.random.default_rng(0)
    for lo, hi in ((-28.0, -16.0), (-16.0, -8.0), (-8.0, -4.0), (-4.0, -1.0), (-1.0, 0.0), (-1e-3, 0.0)):
        d = rng.uniform(lo, hi, 1 << 21).astype(np.float32)
        e, lib = run(d)
        want = np.exp(d.astype(np.float64))
        err, ref = (np.abs(x - want) / want for x in (e, lib))
        assert err.max() < 1.1e-7, (lo, hi, err.max())
        assert err.max() < 1.05 * ref.max() and np.sqrt(np.mean(err ** 2)) < 1.01 * np.sqrt(np.mean(ref ** 2)), (lo, hi)
        assert e.max() <= 1.0
    d = np.float32([0.0, -0.0, -27.0, -81.0, -1e30, -np.inf, np.nan, np.inf - np.inf])
    e, _ = run(d)
    assert e[0] == 1.0 and e[1] == 1.0 and abs(e[2] / np.exp(-27.0) - 1.0) < 1.1e-7
    assert (e[3:] < 2.0 ** -40).all() and (e[3:] > 0.0).all()


@pytest.mark.parametrize("T", [0.7, 1.3, 1.0, 3.0, 1e-3, 2.0 ** -20, 2.0 ** 20, 1.0 - 2.0 ** -24, 1.0 + 2.0 ** -23, 2.0 - 2.0 ** -23, 2.0 ** -7 * (2.0 - 2.0 ** -22),
                               2.0 ** -21, 2.0 ** 21])
def test_quotients_are_correctly_rounded(T):
    """The division of the histogram pass (the debug build exposes it) bit for bit against numpy's, which rounds correctly: mantissas
    at random, all ones, all zeros and next to these, magnitudes from 2^-100 (below, the remainder of a quotient
    leaves the range) to 2^60, where a wave changes to the plain division, and beyond; products of T that lie next to the
    middle between two quotients.  T of 2^-21 and 2^21 take the plain division throughout."""
    import ctypes
    import torch
    T = np.float32(T)
    rng = np.random.default_rng(1)
    n = 1 << 20
    m = rng.integers(0, 1 << 23, n)
    m[: n // 4] = rng.choice([0, 1, 2, (1 << 23) - 1, (1 << 23) - 2, 1 << 22, (1 << 22) - 1], n // 4)
    e = rng.integers(27, 187, n)                                  # 2^-100 .. 2^59
    e[-n // 8:] = rng.integers(185, 190, n // 8)                  # 2^58 .. 2^62: waves of either way
    v = ((rng.integers(0, 2, n) << 31) | (e << 23) | m).astype(np.uint32).view(np.float32)
    mid = rng.integers(1 << 24, 1 << 25, n // 4).astype(np.float64) * 2.0 ** -24      # 25 bits: every other one a middle
    v[n // 4: n // 2] = (mid * np.float64(T)).astype(np.float32)
    v[-8:] = [np.inf, -np.inf, 0.0, -0.0, 3e38, -3e38, 1.0, -1.0]
    with np.errstate(over="ignore"):
        want = v / T
    d = torch.from_numpy(v).cuda()
    q = torch.empty_like(d)
    torch.cuda.synchronize()
    assert debug_library().rsd_debug_smp_divide(ctypes.c_void_p(d.data_ptr()), ctypes.c_float(T), ctypes.c_void_p(q.data_ptr()), n) == 0
    bad = np.nonzero(q.cpu().numpy().view(np.uint32) != want.view(np.uint32))[0]
    assert bad.size == 0, (bad.size, [(float(v[i]), float(q[i]), float(want[i])) for i in bad[:4]])
