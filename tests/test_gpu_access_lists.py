"""GPU tests of long random-access lists, which are served by bands of blocks:
lists over all blocks, within few blocks (a piece's workgroups then split it by
place), of a length that is no multiple of a piece, with requests out of range;
each exact against the oracle, and the same as in short lists.
"""
import numpy as np
import pytest
import torch

from helpers import blocks_of, make_lf, oracle_encode, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu

LONG, TABLES = 1 << 17, 13 << 20   # where lists and tables count as long


@pytest.mark.parametrize("block,size", [(2, (9, 9, 180, 122)), (4, (11, 9, 301, 203))])
def test_long_lists(gpu, block, size):
    U, V, W, H = size
    say("lists", block, size)
    enc = oracle_encode(make_lf(U, V, W, H, seed=5 + block, sigma=8.0), block=block, levels=3, cluster=(2, 2))
    lf = lfc.lfc_open(enc.stream)
    i = lf.info
    tables = i.stream_bytes + 4 * i.present_blocks + 8 * i.n_groups * ((i.n_srv + 31) // 32)
    assert tables >= TABLES
    want = blocks_of(enc.r0, block)
    nv, nb = U * V, i.n_blocks
    r = np.random.default_rng(block)
    for name, n, lo, hi in [("all", LONG + 259, 0, nb), ("just long", LONG, 0, nb), ("short", LONG - 1, 0, nb),
                            ("few blocks", LONG + 1, 5, 9), ("one block", LONG + 513, nb - 1, nb)]:
        req = np.stack([r.integers(0, nv, n), r.integers(lo, hi, n)], 1).astype(np.int32)
        got = lfc.lfc_decode_blocks(lf, torch.from_numpy(req).cuda(), lfc.LAYOUT_BLOCKS).cpu().numpy()
        assert np.array_equal(got, want[req[:, 0], req[:, 1]]), name
    # sorted, so that bands come and go, and out of range: zeros, and the error is kept
    req = np.stack([r.integers(0, nv, LONG + 77), np.sort(r.integers(0, nb, LONG + 77))], 1).astype(np.int32)
    bad = r.choice(len(req), 300, replace=False)
    req[bad[:100], 0] = -1
    req[bad[100:200], 1] = nb
    req[bad[200:], 1] = -7
    got = lfc.lfc_decode_blocks(lf, torch.from_numpy(req).cuda(), lfc.LAYOUT_BLOCKS).cpu().numpy()
    ok = np.ones(len(req), bool)
    ok[bad] = False
    assert np.array_equal(got[ok], want[req[ok, 0], req[ok, 1]])
    assert not got[bad].any()
    with pytest.raises(lfc.LFCError):
        lfc.lfc_check(lf)
