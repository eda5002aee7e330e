"""The power-of-two classes from 2^15 to 2^19 (rows of 512 points, one wave each;
pass 1 gathers its bits from the seed and the key) through the C ABI on MI355X,
against the CPU oracle: slices that begin at every bit of a word, wrap past the
end of the circle, end with the buffers, and groups of several summed chunks."""
import numpy as np
import pytest

import synth
from test_gpu_smooth import _check

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


@pytest.mark.parametrize("logL", [15, 16, 17, 18, 19])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_short_class(pa, ctx, prec, logL, monkeypatch):
    from gpu_util import gpu_hash
    L = 1 << logL
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    flags = pa.PA_PREC_FP32_SEG if prec == "fp32" else pa.PA_PREC_FP64
    rng = np.random.default_rng(logL)
    shapes = [(L // 2, L // 2 + 1), (1, L), (L - 6, 7),          # n + m - 1 = L: nothing of the circle unused
              (L // 3 + 5, L // 2 - 33),                         # one tile, ragged
              (2 * L + 31, L // 2 + 1), (5 * L - 64, L // 3)]    # chunks in one window
    if logL < 18:
        shapes.append((L + 77, 2 * L + 129))                     # chunks and windows
    if logL == 15:
        shapes.append((L // 3, 100 * L))                         # more rows than the device has waves
    for n, m in shapes:
        plan = pa.pa_plan_query(n, m, flags)
        assert plan["fft_len"] == L, plan
        p = synth.random_problem(rng, n, m)
        what = f"{prec} 2^{logL} n={n} m={m} plan {plan['chunks']}x{plan['windows']}"
        print(what, flush=True)
        st, y = gpu_hash(pa, ctx, p.seed, n, m, p.key, flags)
        assert st == pa.PA_OK, pa.pa_strerror(st)
        s = pa.pa_last_stats(ctx)
        assert s["fft_len"] == L and s["n1"] * s["n2"] == L and s["fallback_tiles"] == 0, s
        assert s["max_residual"] < (1e-6 if prec == "fp64" else 0.25), s   # 1/4: the certificate's own limit
        _check(p, y, plan["window_bits"], rng, what)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_budget_below_the_planned_tile(pa, prec):
    """A budget that does not hold one tile of the planned class: the job runs on
    shorter classes."""
    from gpu_util import gpu_hash
    flags = pa.PA_PREC_FP32_SEG if prec == "fp32" else pa.PA_PREC_FP64
    n, m = 400_000, 60_001
    rng = np.random.default_rng(23)
    p = synth.random_problem(rng, n, m)
    tile = pa.pa_plan_query(n, m, flags)["fft_len"] * (8 if prec == "fp32" else 16)
    seen = set()
    for budget in (4 * tile, tile + tile // 8, tile - 4096, tile // 2):
        c = pa.pa_create(0, budget, None)
        st, y = gpu_hash(pa, c, p.seed, n, m, p.key, flags)
        assert st == pa.PA_OK, (budget, pa.pa_strerror(st))
        s = pa.pa_last_stats(c)
        assert s["tiles"] >= 1 and s["fft_len"] * (8 if prec == "fp32" else 16) <= budget, (budget, s)
        seen.add(s["fft_len"])
        _check(p, y, s["window_bits"], rng, f"{prec} budget {budget}")
        pa.pa_destroy(c)
    assert len(seen) > 1, seen
