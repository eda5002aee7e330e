"""Pass 1 on whole columns (FP32 2^20 and 2^21), through the C ABI on MI355X, against
the direct GF(2) product, which uses no transform."""
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


# rows are 4096 points: slices that end in the first row, at a row, one bit to either
# side of it, within the last row and at the tile's end; one to several chunks, two
# windows
def _shapes(L):
    return [(1, 1), (1000, 97), (4000, 97), (4000, 98), (3 * 4096, 4096), (L // 2, L // 2 + 1), (L // 2, L // 2 - 4094),
            (L - 63, 64), (77, L - 76), (L // 3, L // 5), (3 * L // 2 + 7, L // 3), (2 * L + 1, L // 7), (L // 9, 5 * L // 4)]


@pytest.mark.parametrize("L", [1 << 20, 1 << 21])
def test_whole_columns(pa, ctx, L, monkeypatch):
    """Each shape alone, then all of them as tiles of one launch."""
    from gpu_util import to_dev, from_dev, empty_dev, describe
    import torch
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    rng = np.random.default_rng(L % 997)
    jobs, refs = [], []
    for n, m in _shapes(L):
        p = synth.random_problem(rng, n, m)
        s, k, ref = to_dev(p.seed), to_dev(p.key), empty_dev(synth.words_for(m))
        assert pa.pa_hash(ctx, s, n, m, k, ref, pa.PA_PREC_DIRECT) == pa.PA_OK
        jobs.append((s, k, empty_dev(synth.words_for(m)), n, m))
        torch.cuda.synchronize()
        refs.append(from_dev(ref)[:synth.words_for(m)])
    for (s, k, o, n, m), ref in zip(jobs, refs):
        print(f"L={L} n={n} m={m}", flush=True)
        assert pa.pa_hash(ctx, s, n, m, k, o, pa.PA_PREC_FP32_SEG) == pa.PA_OK
        torch.cuda.synchronize()
        stats = pa.pa_last_stats(ctx)
        assert stats["fft_len"] == L and stats["fallback_tiles"] == 0, stats
        y = from_dev(o)[:synth.words_for(m)]
        assert np.array_equal(y, ref), (n, m, describe(y, ref, m))
        o.fill_(-1)
    torch.cuda.synchronize()
    st, each = pa.pa_hash_batch(ctx, jobs, pa.PA_PREC_FP32_SEG)
    torch.cuda.synchronize()
    assert st == pa.PA_OK and each == [pa.PA_OK] * len(jobs)
    for (s, k, o, n, m), ref in zip(jobs, refs):
        y = from_dev(o)[:synth.words_for(m)]
        assert np.array_equal(y, ref), (n, m, describe(y, ref, m))
