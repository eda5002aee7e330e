"""Batches and serving at their limits, through the C ABI on MI355X: the grid of the
direct path's shared launch, and HBM budgets around one tile of the planned class."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


def test_direct_batch_beyond_one_grid(pa):
    """1,100 direct jobs of 8,192 workgroups each: together more work-items than
    the 2^32 that a launch may have along one dimension, so the jobs are launched
    one by one (1,000 fit one launch)."""
    from gpu_util import to_dev, from_dev, describe
    import torch
    n, m = 50, 1 << 24
    p = synth.random_problem(np.random.default_rng(3), n, m)
    s, k = to_dev(p.seed), to_dev(p.key)
    ref = oracle.hash_words(p.seed, n, m, p.key)
    dref = to_dev(ref)
    c = pa.pa_create(0, 0, None)
    try:
        for count in (1000, 1100):
            outs = torch.full((count, m // 64), -1, dtype=torch.int64, device="cuda:0")
            torch.cuda.synchronize()
            print(f"{count} jobs", flush=True)
            st, per = pa.pa_hash_batch(c, [(s, k, outs[i], n, m) for i in range(count)], pa.PA_PREC_DIRECT)
            torch.cuda.synchronize()
            assert st == pa.PA_OK and per == [pa.PA_OK] * count, pa.pa_strerror(st)
            assert bool((outs == dref[None, :]).all()), describe(from_dev(outs[count - 1]), ref, m)
            launches = pa.pa_last_stats(c)["launches"]
            assert launches == (1 if count == 1000 else count), launches
            del outs
    finally:
        pa.pa_destroy(c)
