"""The memory an encoder's freed stream leaves with the library (lfc_free): it
serves streams of about its size, not small ones, and goes back when the
program has moved on to small ones.
"""
import ctypes as C

import numpy as np

from paper_1805_06019_amd import lfc
from test_stream_memory import BIG, encode_raw, noise

LARGE = lfc.Params(3, 3, 1400, 1000, 4, 2, (2,))


def resident():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * 4096


def test_a_small_stream_does_not_hold_a_large_ones_memory():
    lib, large, small = lfc.load(), noise(3, 3, 1400, 1000, 1), noise(3, 3, 256, 200, 2)
    want = lfc.lfc_encode(small, BIG)
    out, n = encode_raw(large, LARGE)
    assert n > 16 * len(want) > 16 << 20
    lib.lfc_free(out)
    s, ns = encode_raw(small, BIG)
    assert not out.value <= s.value < out.value + n
    again, _ = encode_raw(large, LARGE)
    assert again.value == out.value   # (still kept: it serves the next large one)
    lib.lfc_free(again)
    assert C.string_at(s.value, ns) == want
    lib.lfc_free(s)
    before, held = resident(), []
    for _ in range(6):
        held.append(encode_raw(small, BIG)[0])
    assert resident() < before - n // 2   # the large one's memory has gone back
    for h in held:
        assert C.string_at(h.value, ns) == want
        lib.lfc_free(h)
