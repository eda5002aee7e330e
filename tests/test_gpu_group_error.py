"""The error model of summed groups against the residuals that the certificate
measures, through the C ABI on MI355X: random inputs, the largest groups that the
planner makes.  A group stays below the model of its plan, and so far below the
certificate's limit that no random input falls back to FP64."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CERTIFICATE = 0.125


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


@pytest.fixture(scope="module")
def ctx(pa):
    c = pa.pa_create(0, 0, None)
    yield c
    pa.pa_destroy(c)


def _chunks(L, count):
    m = L // 8
    return count * (L - m + 1) - 5, m, L


# (n, m, class or 0 for the planner's): groups of 64 chunks at 2^15 .. 2^21, of as
# many as the limit admits above, and shapes whose chunks fill between a half and
# all of the class
SHAPES = [_chunks(1 << 15, 64), _chunks(1 << 17, 64), _chunks(1 << 19, 64), _chunks(1 << 21, 32), _chunks(1 << 21, 64),
          _chunks(1 << 23, 8), _chunks(1 << 23, 16), _chunks(7 << 20, 32), (103_936_051, 1_387_651, 0),
          (60_821_400, 1_014_178, 0), (69_081_378, 905_967, 0), (36_902_325, 1_330_031, 0), (8_587_073, 3_744_043, 0),
          (39_017_031, 77_303, 0)]


@pytest.mark.parametrize("n,m,only", SHAPES)
def test_group_residual_below_the_model(pa, ctx, n, m, only, monkeypatch):
    import torch
    if only:
        monkeypatch.setenv("PA_ONLY_LEN", str(only))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n % 1009)
    top = (1 << 63) - 1

    def words(bits):
        return torch.randint(-top - 1, top, (synth.words_for(bits),), dtype=torch.int64, device="cuda:0", generator=gen)

    out = torch.zeros(synth.words_for(m), dtype=torch.int64, device="cuda:0")
    for _ in range(3):
        seed, key = words(n + m - 1), words(n)
        if n & 63:
            key[-1] &= (1 << (n & 63)) - 1
        torch.cuda.synchronize()
        assert pa.pa_hash(ctx, seed, n, m, key, out, pa.PA_PREC_FP32_SEG) == pa.PA_OK
        s = pa.pa_last_stats(ctx)
        print(f"n={n} m={m} L={s['fft_len']} residual {s['max_residual']:.4f} model {s['bound']:.4f}", flush=True)
        assert s["fallback_tiles"] == 0, s
        assert s["max_residual"] <= s["bound"] and s["max_residual"] < CERTIFICATE, s
