"""FP64 fallback of FP32 jobs whose chunks make several summed groups, through the
C ABI on MI355X.  A failed group is replaced in place: its FP32 run is repeated, so
that its bits cancel out of the window, and its chunks are added in FP64.  That
asks for a repeat that rounds exactly as the first run did, whatever else was in
the first run's launch."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


@pytest.fixture(scope="module")
def ctx(pa):
    c = pa.pa_create(0, 0, None)
    yield c
    pa.pa_destroy(c)


def _groups(chunks):
    """Chunk groups and chunks of a (full) group: at most 64 to a group."""
    groups = -(-chunks // 64)
    return groups, -(-chunks // groups)


def _set_bits(words, lo, hi):
    """The words with bits [lo, hi) set."""
    nbits = words.size * 64
    bits = np.unpackbits(words.view(np.uint8), bitorder="little", count=nbits)
    bits[lo:hi] = 1
    return np.packbits(bits, bitorder="little").view(np.uint64).copy()


# groups of 2, 3 and 7: the first run's launch takes other row kernels than a
# launch of one group would (512 row units per group at 2^19, the device's waves
# taken by 1, 2 and 8 of them)
@pytest.mark.parametrize("n,m", [(39_017_031, 77_303), (60_000_000, 60_000), (190_000_001, 40_000)])
def test_every_group_fails(pa, ctx, n, m, monkeypatch):
    """All-ones key and seed: every value of a group is its weight, above what
    the FP32 certificate accepts (2^20) and, above 2^24, beyond what its residual
    can tell.  Closed form: every output is n mod 2."""
    from gpu_util import gpu_hash
    monkeypatch.setenv("PA_ONLY_LEN", str(1 << 19))
    plan = pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG)
    groups, _ = _groups(plan["chunks"])
    assert plan["windows"] == 1 and groups > 1, plan
    print(f"n={n} m={m} chunks {plan['chunks']} groups {groups}", flush=True)
    st, y = gpu_hash(pa, ctx, synth.pattern_bits("ones", n + m - 1), n, m, synth.pattern_bits("ones", n),
                     pa.PA_PREC_FP32_SEG)
    assert st == pa.PA_OK, pa.pa_strerror(st)
    s = pa.pa_last_stats(ctx)
    assert np.array_equal(synth.bits_to_array(y, m), np.full(m, n & 1, np.uint8)), s
    # replaced in place: the first run, the repeats, the FP64 chunks
    assert s["fallback_tiles"] == plan["chunks"] and s["tiles"] == 3 * plan["chunks"], s


@pytest.mark.parametrize("beside", [False, True])
@pytest.mark.parametrize("L", [1 << 15, 1 << 17, 1 << 19, 5 << 18, 1 << 21])
def test_one_group_fails(pa, ctx, L, beside, monkeypatch):
    """Random seed and key, but ones where the first chunk group lies: that group
    alone fails and is replaced, the others keep their FP32 bits (also with
    another job in the launch).  The reference is the direct GF(2) product, which
    uses no transform."""
    from gpu_util import to_dev, from_dev, empty_dev, describe
    import torch
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    rng = np.random.default_rng(L % 1013)
    m = min(L // 32 + 3, 60_001)
    n = 70 * (L - m + 1) - 12345                     # 70 chunks: two groups of 35
    plan = pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG)
    groups, per = _groups(plan["chunks"])
    assert plan["fft_len"] == L and plan["windows"] == 1 and groups == 2, plan
    ones = per * plan["chunk_bits"]                  # the top key bits meet the first seed bits
    p = synth.random_problem(rng, n, m)
    assert ones > 1 << 20                            # the group's weight, and the certificate's limit
    s, k = to_dev(_set_bits(p.seed, 0, ones + m)), to_dev(_set_bits(p.key, n - ones, n))
    o = empty_dev(synth.words_for(m))
    jobs = [(s, k, o, n, m)]
    if beside:
        q = synth.random_problem(rng, 9 * L + 77, m + 1)
        jobs.append((to_dev(q.seed), to_dev(q.key), empty_dev(synth.words_for(q.m)), q.n, q.m))
    print(f"L={L} n={n} m={m} chunks {plan['chunks']} beside={beside}", flush=True)
    st, each = pa.pa_hash_batch(ctx, jobs, pa.PA_PREC_FP32_SEG)
    torch.cuda.synchronize()
    assert st == pa.PA_OK and each == [pa.PA_OK] * len(jobs)
    stats = pa.pa_last_stats(ctx)
    for js, jk, jo, jn, jm in jobs:
        ref = empty_dev(synth.words_for(jm))
        assert pa.pa_hash(ctx, js, jn, jm, jk, ref, pa.PA_PREC_DIRECT) == pa.PA_OK
        torch.cuda.synchronize()
        a, b = from_dev(jo)[:synth.words_for(jm)], from_dev(ref)[:synth.words_for(jm)]
        assert np.array_equal(a, b), describe(a, b, jm)
    assert stats["fallback_tiles"] == per, stats     # the first group's chunks alone
