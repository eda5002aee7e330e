"""The worst-case bound of a summed group (CPU only): the chunks' errors in full
and the rounding of the sum, against the formula written out here."""
import math

import pytest


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


@pytest.mark.parametrize("prec,u", [("PA_PREC_FP64", 2.0 ** -53), ("PA_PREC_FP32_SEG", 2.0 ** -24)])
@pytest.mark.parametrize("logL,chunks", [(16, 1), (16, 2), (16, 64), (19, 35), (20, 90)])
def test_group_bound_covers_the_sum(pa, prec, u, logL, chunks, monkeypatch):
    L = 1 << logL
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    m = L // 8
    n = chunks * (L - m + 1) - 3
    p = pa.pa_plan_query(n, m, getattr(pa, prec))
    assert p["fft_len"] == L and p["chunks"] == chunks and p["windows"] == 1, p
    groups = -(-chunks // 64)                        # at most 64 chunks to a group
    c = -(-chunks // groups)
    # a product of the forward, separation and inverse factors (3 levels of a
    # radix-2 transform per doubling, two for the packing), then c - 1 additions
    lv = 3 * logL + 2
    grow = (1 + u) ** lv * (1 + u * math.sqrt(5)) ** (lv + 1) * (1 + 2 * u) ** lv if u > 1e-10 else None
    g = lv * math.log1p(u) + (lv + 1) * math.log1p(u * math.sqrt(5)) + lv * math.log1p(2 * u)
    if grow is not None:
        assert math.isclose(math.expm1(g), grow - 1, rel_tol=1e-6)
    g += (c - 1) * math.log1p(u)
    norms = (math.sqrt(p["chunk_bits"]) + math.sqrt(p["chunk_bits"] + m - 1)) ** 2
    assert p["rigorous_bound"] >= c * norms * math.expm1(g) * (1 - 1e-9), p
    assert p["rigorous_bound"] <= c * norms * math.expm1(g) * (1 + 1e-9), p
