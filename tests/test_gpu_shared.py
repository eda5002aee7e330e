"""Jobs with shared spectra (several key chunks and several output windows: each
chunk and seed slice is transformed once, the windows are summed from the
stored spectra), through the C ABI on MI355X.  The reference is the direct GF(2)
product of the whole output, which uses no transform and is tested against the
CPU oracle; both are also compared with the oracle on sampled outputs."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

L = 1 << 21          # chunks and windows of B = 2^20
B = L // 2


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


@pytest.fixture(scope="module")
def ctx(pa):
    c = pa.pa_create(0, 0, None)
    yield c
    pa.pa_destroy(c)


def _job(rng, n, m):
    from gpu_util import to_dev, empty_dev
    p = synth.random_problem(rng, n, m)
    return p, to_dev(p.seed), to_dev(p.key), empty_dev(synth.words_for(m) + 4)


def _check(pa, ctx, p, s, k, y, rng):
    from gpu_util import empty_dev, from_dev, describe
    import torch
    words = synth.words_for(p.m)
    assert np.all(y[words:] == np.uint64(0xFFFFFFFFFFFFFFFF))      # nothing past the output
    d = empty_dev(words)
    assert pa.pa_hash(ctx, s, p.n, p.m, k, d, pa.PA_PREC_DIRECT) == pa.PA_OK
    torch.cuda.synchronize()
    ref = from_dev(d)
    assert np.array_equal(y[:words], ref), describe(y[:words], ref, p.m)
    edges = [i for w in range(0, p.m + B, B) for i in range(w - 40, w + 40) if 0 <= i < p.m]
    idx = np.unique(np.concatenate([edges, rng.integers(0, p.m, 200), [0, p.m - 1]])).astype(np.uint64)
    assert np.array_equal(synth.bits_to_array(y, p.m)[idx.astype(np.int64)], oracle.hash_select(p.seed, p.n, p.m, p.key, idx))


# windows 2, 3, 4 (sums in the row pass), 5, 6 and 9 (sums of 8 and 8 + 2 stored
# windows at a time), chunk counts odd and even, last chunks and windows short, full
# and ragged
SHAPES = [(9 * B + 3, 2 * B - 1), (12 * B, 2 * B), (20 * B + 5, 3 * B - 17), (7 * B + 7, 4 * B), (4 * B, 4 * B + 64), (6 * B + 7, 5 * B + 5),
          (3 * B + 12345, 8 * B + 999_001)]


@pytest.mark.parametrize("n,m", SHAPES)
def test_shared_spectra_exact(pa, ctx, n, m, monkeypatch):
    from gpu_util import from_dev
    import torch
    rng = np.random.default_rng(n % 1009 + m % 997)
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    plan = pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG)
    assert plan["chunk_bits"] == plan["window_bits"] == B and plan["windows"] == -(-m // B) > 1, plan
    p, s, k, o = _job(rng, n, m)
    print(f"shared n={n} m={m} {plan['chunks']}x{plan['windows']}", flush=True)
    for _ in range(2):
        assert pa.pa_hash(ctx, s, n, m, k, o, pa.PA_PREC_FP32_SEG) == pa.PA_OK
    torch.cuda.synchronize()
    st = pa.pa_last_stats(ctx)
    assert st["tiles"] == plan["chunks"] * plan["windows"] and st["fallback_tiles"] == 0, st
    assert st["max_residual"] <= st["bound"], st
    _check(pa, ctx, p, s, k, from_dev(o), rng)


@pytest.mark.parametrize("budget_mib", [700, 400, 60])
def test_shared_spectra_small_budget(pa, budget_mib, monkeypatch):
    """A budget that holds a few packs at a time (chunk groups, XOR-ed windows),
    and one too small for that (plain tiles)."""
    from gpu_util import from_dev
    import torch
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    rng = np.random.default_rng(budget_mib)
    n, m = 20 * B + 5, 3 * B - 17
    c = pa.pa_create(0, budget_mib << 20, None)
    try:
        p, s, k, o = _job(rng, n, m)
        assert pa.pa_hash(c, s, n, m, k, o, pa.PA_PREC_FP32_SEG) == pa.PA_OK
        torch.cuda.synchronize()
        _check(pa, c, p, s, k, from_dev(o), rng)
    finally:
        pa.pa_destroy(c)


@pytest.mark.parametrize("budget_mib", [0, 1200])
def test_shared_spectra_fallback(pa, budget_mib, monkeypatch):
    """All-ones key and seed: every window value is the key length, above what
    the FP32 certificate accepts, so every window is redone in FP64 (also where
    it is the XOR of several chunk groups).  Closed form: every output is n mod
    2.  A random job in the same batch keeps its FP32 result, and without the
    fallback the job reports PA_EPRECISION."""
    from gpu_util import to_dev, empty_dev, from_dev
    import torch
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    rng = np.random.default_rng(5)
    n, m = 31 * B + 1, 4 * B - 100
    c = pa.pa_create(0, budget_mib << 20, None)
    try:
        ones = (to_dev(synth.pattern_bits("ones", n + m - 1)), to_dev(synth.pattern_bits("ones", n)),
                empty_dev(synth.words_for(m)), n, m)
        p, s, k, o = _job(rng, 6 * B + 7, 5 * B + 5)
        small, s2, k2, o2 = _job(rng, 300_000, 400_000)
        st, per = pa.pa_hash_batch(c, [(s, k, o, p.n, p.m), ones, (s2, k2, o2, small.n, small.m)], pa.PA_PREC_FP32_SEG)
        torch.cuda.synchronize()
        assert st == pa.PA_OK and per == [pa.PA_OK] * 3
        assert pa.pa_last_stats(c)["fallback_tiles"] >= 32 * 4
        assert np.array_equal(synth.bits_to_array(from_dev(ones[2]), m), np.full(m, n & 1, np.uint8))
        _check(pa, c, p, s, k, from_dev(o), rng)
        assert np.array_equal(from_dev(o2)[:synth.words_for(small.m)], oracle.hash_words(small.seed, small.n, small.m, small.key))
        assert pa.pa_hash(c, *ones[:1], n, m, *ones[1:3], pa.PA_PREC_FP32_SEG | pa.PA_NO_FALLBACK) == pa.PA_EPRECISION
    finally:
        pa.pa_destroy(c)
