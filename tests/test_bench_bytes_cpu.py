"""The bytes that bench.py rates the passes with (CPU only): chunks whose products
are summed share one inverse."""
import bench


def test_summed_chunks_share_the_inverse():
    n, m, L = 12_345_679, 1_234_567, 1 << 23
    st = {"prec": 0x10, "fft_len": L, "chunk_bits": 6_172_840, "window_bits": m}
    p1, p2, p3, rest = bench.launch_bytes(st, n, m)
    array = 8.0 * L
    assert p1 == 2 * array + (2 * n + 2 * m) / 8          # two tiles written; no clearing: one group
    assert p2 == 2 * array + array / 2                    # both read, half a tile written
    assert p3 == array / 2 + m / 8 and rest == 0
    # one chunk: as ever
    one = dict(st, prec=0x20, chunk_bits=n, fft_len=7 << 21)
    assert bench.launch_bytes(one, n, m)[1] == 1.5 * 16 * (7 << 21)
    # a class that does not sum: an inverse per chunk
    short = dict(st, fft_len=3 << 18)
    assert bench.launch_bytes(short, n, m)[1] == 2 * 1.5 * 8 * (3 << 18)
