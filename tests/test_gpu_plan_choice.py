"""The class that the planner picks against the fastest of all, by the clock on MI355X
(the median of several calls; the limits leave room for the noise of a shared box)."""
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


def _words(gen, bits):
    import torch
    top = (1 << 63) - 1
    return torch.randint(-top - 1, top, (synth.words_for(bits) + 512,), dtype=torch.int64, device="cuda:0", generator=gen)


def _median_us(call, reps=15):
    for _ in range(3):
        call()
    took = []
    for _ in range(reps):
        t = time.perf_counter()
        call()
        took.append(time.perf_counter() - t)
    return float(np.median(took)) * 1e6


def _choice(pa, jobs, n, m, flags, monkeypatch):
    """(us of the planned class, its length, [(us, length)] of the classes beside it)."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n % 1009)
    seed, key = _words(gen, n + m - 1), _words(gen, n)
    ow = synth.words_for(m)
    out = torch.zeros(jobs * ow, dtype=torch.int64, device="cuda:0")
    torch.cuda.synchronize()
    ctx = pa.pa_create(0, 32 << 30, None)
    try:
        if jobs == 1:
            def call():
                assert pa.pa_hash(ctx, seed, n, m, key, out, flags) == pa.PA_OK
        else:
            batch = pa.JobBatch([(seed[q:], key[q:], out[q * ow:(q + 1) * ow], n, m) for q in range(jobs)])

            def call():
                assert pa.pa_hash_batch(ctx, batch, flags)[0] == pa.PA_OK
        monkeypatch.delenv("PA_ONLY_LEN", raising=False)
        planned = _median_us(call)
        length = pa.pa_last_stats(ctx)["fft_len"]
        beside = []
        for L in sorted(p << k for p in (1, 3, 5, 7) for k in range(14, 25) if 1 << 17 <= p << k <= 1 << 24):
            if not length // 16 <= L <= 16 * length:
                continue
            monkeypatch.setenv("PA_ONLY_LEN", str(L))
            beside.append((_median_us(call, 7), L))
        return planned, length, beside
    finally:
        pa.pa_destroy(ctx)


# keys of many chunks for short outputs: one group, whose chunks follow one another
@pytest.mark.parametrize("n,m", [(13_485_586, 383_518), (21_163_809, 340_151), (33_076_724, 393_302), (7_522_386, 373_524),
                                 (4_219_838, 240_643)])
def test_single_keys(pa, n, m, monkeypatch):
    planned, length, beside = _choice(pa, 1, n, m, pa.PA_PREC_FP32_SEG, monkeypatch)
    print(f"n={n} m={m} planned {length}: {planned:.1f} us, fastest {min(beside)}", flush=True)
    assert planned <= 1.16 * min(beside)[0] + 2.0, (planned, length, sorted(beside)[:4])


# batches of equal jobs: what is cheapest for one of them is not for all together
@pytest.mark.parametrize("jobs,n,m,prec", [(64, 1_221_990, 640_930, "fp32"), (128, 919_382, 541_430, "fp32"),
                                           (64, 777_751, 765_368, "fp32"), (256, 856_335, 537_706, "fp32"),
                                           (64, 296_412, 16_745, "fp64"), (256, 310_750, 36_624, "fp64")])
def test_batches(pa, jobs, n, m, prec, monkeypatch):
    flags = pa.PA_PREC_FP32_SEG if prec == "fp32" else pa.PA_PREC_FP64
    planned, length, beside = _choice(pa, jobs, n, m, flags, monkeypatch)
    print(f"{jobs} x n={n} m={m} planned {length}: {planned:.1f} us, fastest {min(beside)}", flush=True)
    assert planned <= 1.2 * min(beside)[0] + 2.0, (planned, length, sorted(beside)[:4])


def test_ntt_of_many_chunks_beside_a_short_job(pa):
    """The NTT sums no chunks: a long key does not follow a short job to its class, at
    a tile for each of 51 chunks.  Both together take little more than the long one."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(7)
    (n, m), (n2, m2) = (2_002_554, 25_360), (32_520, 21_266)
    seed, key = _words(gen, n + m - 1), _words(gen, n)
    outs = [torch.zeros(synth.words_for(x), dtype=torch.int64, device="cuda:0") for x in (m, m2)]
    torch.cuda.synchronize()
    ctx = pa.pa_create(0, 0, None)
    try:
        alone = _median_us(lambda: pa.pa_hash(ctx, seed, n, m, key, outs[0], pa.PA_PREC_NTT))
        batch = pa.JobBatch([(seed, key, outs[0], n, m), (seed, key, outs[1], n2, m2)])
        both = _median_us(lambda: pa.pa_hash_batch(ctx, batch, pa.PA_PREC_NTT))
        print(f"alone {alone:.1f} us, both {both:.1f} us", flush=True)
        assert both <= 1.2 * alone + 30.0, (alone, both)
    finally:
        pa.pa_destroy(ctx)
