"""Tuning tables that other programs write, or earlier libraries (through the C ABI on
MI355X)."""
import json

import pytest

pytestmark = pytest.mark.gpu

N, M = 300_000, 60_000


@pytest.fixture(scope="module")
def pa():
    from paper_1805_02372_amd import pa as _pa
    return _pa


def _planned(pa, path):
    """The class that a context takes for (N, M) after loading a table."""
    import torch
    c = pa.pa_create(0, 0, None)
    try:
        assert pa.pa_tune_load(c, str(path)) == pa.PA_OK
        z = torch.zeros((N + M + 63) // 64 + 1, dtype=torch.int64, device="cuda:0")
        out = torch.zeros((M + 63) // 64, dtype=torch.int64, device="cuda:0")
        torch.cuda.synchronize()
        assert pa.pa_hash(c, z, N, M, z, out, pa.PA_PREC_FP32_SEG) == pa.PA_OK
        return pa.pa_last_stats(c)["fft_len"]
    finally:
        pa.pa_destroy(c)


@pytest.mark.parametrize("separators", [(",", ":"), (", ", ": "), (" , ", " : ")])
def test_white_space_before_a_section(pa, tmp_path, separators):
    """White space around the colons of the section names."""
    path = tmp_path / "table.json"
    rows = json.dumps({"655360": [1e-9, 0.0]}, separators=(",", ":"))
    path.write_text('{"launch":1e-5' + separators[0] + '"fp32"' + separators[1] + rows + "}")
    assert _planned(pa, path) == 655_360


def test_one_cost_per_tile(pa, tmp_path):
    """A table without the sections for few tiles and for chunks: its costs hold for
    launches of any size, and are not mixed with those that ship with the library."""
    path = tmp_path / "table.json"
    path.write_text(json.dumps({"fp32": {"655360": [5e-6, 0.0], "524288": [7e-6, 0.0]}}))
    assert _planned(pa, path) == 655_360
