"""Memory of encoded streams (lfc_encode ... lfc_free): streams held at once
have memory of their own, a freed one may serve the next, and threads may
encode and free together.  Streams of more than 1 MiB, which take the kept
memory, and small ones, which do not.
"""
import ctypes as C
from concurrent.futures import ThreadPoolExecutor

import numpy as np

from paper_1805_06019_amd import lfc


def noise(U, V, W, H, seed):
    return np.random.default_rng(seed).integers(0, 256, (V, U, H, W, 3), dtype=np.uint8)


def encode_raw(rgb, p):
    out, n = C.c_void_p(), C.c_size_t()
    lfc._check(lfc.load().lfc_encode(rgb.ctypes.data, C.byref(p.to_c()), C.byref(out), C.byref(n)))
    return out, n.value


BIG = lfc.Params(3, 3, 256, 200, 4, 2, (2,))
SMALL = lfc.Params(2, 2, 16, 12, 4, 2, (2,))


def test_streams_held_together_and_reused():
    rgbs = [noise(3, 3, 256, 200, k) for k in range(3)]
    want = [lfc.lfc_encode(r, BIG) for r in rgbs]
    assert len(want[0]) > 1 << 20
    held = [encode_raw(r, BIG) for r in rgbs]
    assert len({h.value for h, _ in held}) == 3
    for order in ((1, 0, 2), (2, 1, 0)):
        for k in order:
            assert C.string_at(held[k][0].value, held[k][1]) == want[k]
            lfc.load().lfc_free(held[k][0])
        held = [encode_raw(r, BIG) for r in rgbs]
    for h, _ in held:
        lfc.load().lfc_free(h)
    lfc.load().lfc_free(None)


def test_threads_encode_and_free_together():
    jobs = [(noise(3, 3, 256, 200, k), BIG) if k % 3 else (noise(2, 2, 16, 12, k), SMALL) for k in range(12)]
    want = [lfc.lfc_encode(r, p) for r, p in jobs]
    with ThreadPoolExecutor(6) as ex:
        for _ in range(3):
            assert list(ex.map(lambda j: lfc.lfc_encode(*j), jobs)) == want
