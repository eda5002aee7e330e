"""The planner's scan of a class's windows (CPU only): it finds what a scan of every
number of windows finds, and takes no longer for it where chunks are summed."""
import json
import os
import time

import pytest


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


def _up(a, b):
    return -(-a // b)


def _costs(table, key, L, sums):
    """The tile and chunk costs of a launch of G groups, from the table beside the
    library: (tile of G groups, further chunk of G groups of c chunks and T tiles)."""
    get = lambda name, default: table.get(key + name, {}).get(str(L), default)
    tile = table[key][str(L)][0]
    few, chunk = get("_few", 0.0), get("_chunk", 0.7 * tile)
    alone = get("_chunk_alone", chunk)
    run = get("_chunk_run", alone)

    def of(groups, c, tiles):
        cached = tiles * L * (16 if key == "fp64" else 8) <= 240e6
        chain = (7 * alone + (c - 8) * run) / (c - 1) if c > 8 else alone
        base = min(alone, run, chunk) if cached else chunk
        further = base + max(chain - base, 0.0) / groups
        return max(tile, 12 * few / max(groups, 12)), further if sums and c > 1 else 0.0
    return of


def _scan(n, m, L, of, sums):
    """(chunks, windows, window bits) by the planner's rule, every number of windows
    tried: cheaper, or fewer tiles within 3%."""
    best = None
    for w in range(max(1, _up(m, L)), max(1, min(_up(m, 64), 1 << 14)) + 1):
        bo = m if w == 1 else _up(_up(m, w), 64) * 64
        if bo > L:
            continue
        outs, chunks = _up(m, bo), _up(n, min(L - bo + 1, n))
        group = _up(chunks, _up(chunks, 64)) if sums else 1
        groups = _up(chunks, group) * outs
        tile, further = of(groups, group, chunks * outs)
        cost = groups * tile + (chunks * outs - groups) * further
        if best is None or cost < (1.03 if chunks * outs < best[0] * best[1] else 1.0) * best[3]:
            best = (chunks, outs, bo, cost)
        if best[:2] == (1, 1):
            break
    return best[:3]


@pytest.mark.parametrize("prec,key", [("PA_PREC_FP64", "fp64"), ("PA_PREC_FP32_SEG", "fp32"), ("PA_PREC_NTT", "ntt")])
@pytest.mark.parametrize("L", [1 << 14, 1 << 15, 3 << 15, 1 << 17, 1 << 19, 3 << 20, 1 << 22])
def test_scan_finds_the_plan_of_a_full_scan(pa, prec, key, L, monkeypatch):
    if key == "fp32" and L > 1 << 17:
        pytest.skip("groups below 64 chunks: by the error model")
    if key == "ntt" and L & (L - 1):
        pytest.skip("no such class")
    monkeypatch.setenv("PA_ONLY_LEN", str(L))
    table = json.load(open(os.path.join(os.path.dirname(pa.__file__), "tune_mi355x.json")))
    sums = key != "ntt" and L >= (1 << 15 if L & (L - 1) == 0 else 1 << 20)
    if str(L) not in table[key]:
        pytest.skip("class not in the table")
    of = _costs(table, key, L, sums)
    for n, m in [(L // 2, L // 2 + 1), (L // 2, L // 2 + 2), (3 * L + 5, 1), (40 * L, 63), (3 * L, 2 * L + 77), (L, L),
                 (17 * L // 3, 9 * L // 2), (70 * L - 9, L // 3), (130 * L, 3 * L), (100, 9 * L), (1, 1), (2 * L, L - 64)]:
        p = pa.pa_plan_query(n, m, getattr(pa, prec))
        assert p["fft_len"] == L
        if key == "fp32" and p["windows"] >= 2 and p["chunk_bits"] == p["window_bits"] == L // 2:
            continue   # shared spectra
        assert (p["chunks"], p["windows"], p["window_bits"]) == _scan(n, m, L, of, sums), (n, m, p)


def test_summed_classes_plan_as_fast(pa):
    """FP32 classes beside NTT ones, which scan as many windows without groups and
    their error model: 2.7 times as long (more classes).  With the model asked at
    every window it was 5 times."""
    def took(prec):
        best = 1e9
        for _ in range(40):
            t = time.perf_counter()
            pa.pa_plan_query(128_000_000, 12_800_000, prec)
            best = min(best, time.perf_counter() - t)
        return best
    ratio = min(took(pa.PA_PREC_FP32_SEG) / took(pa.PA_PREC_NTT) for _ in range(3))
    assert ratio < 3.8, ratio


@pytest.mark.parametrize("n,m", [(142_795_849, 65_530_406), (153_272_179, 97_861_985), (150_254_723, 63_964_138)])
def test_shared_spectra_of_many_windows(pa, n, m):
    """Shared spectra with 16 to 47 windows: 2^22 points take 5.85, 14.4 and 5.93 ms on
    MI355X, 2^23 points 6.14, 15.1 and 6.19."""
    assert pa.pa_plan_query(n, m, pa.PA_PREC_FP32_SEG)["fft_len"] == 1 << 22
