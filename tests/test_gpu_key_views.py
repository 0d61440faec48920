"""GPU tests of the colour whole-field decoder with more key views than a
workgroup holds in LDS (13 at 8 x 8, 16 at 4 x 4, 32 at 2 x 2): each chunk's are
read with it.  One past the number, several times it, trees of one and two
levels, every view and only those a render reads; exact against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import make_lf, oracle_encode, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu

CASES = [
    # U, V, W, H, block, levels, threshold
    (7, 2, 70, 21, 8, 1, 0),       # 14 key views
    (8, 14, 40, 16, 8, 2, 0),      # 28, every block stored
    (9, 13, 70, 9, 8, 2, 300),     # 35, few stored
    (17, 1, 66, 13, 4, 1, 0),      # 17
    (10, 9, 70, 12, 4, 2, 0),      # 25
    (16, 15, 36, 9, 4, 2, 40),     # 64
    (11, 3, 67, 5, 2, 1, 0),       # 33
    (13, 16, 34, 6, 2, 2, 0),      # 56
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}-B{c[4]}-L{c[5]}" for c in CASES])
def test_many_key_views(gpu, case):
    U, V, W, H, block, levels, thr = case
    say("keys", case)
    enc = oracle_encode(make_lf(U, V, W, H, seed=U + 31 * V, sigma=6.0), block=block, levels=levels,
                        cluster=(2,) * (levels - 1), blk_threshold=thr)
    rgb = oracle.ycocg_inverse(np.ascontiguousarray(np.transpose(enc.r0, (0, 2, 3, 1)))).astype(np.uint32)
    words = (rgb[..., 0] | (rgb[..., 1] << 8) | (rgb[..., 2] << 16)).view(np.int32)
    lf = lfc.lfc_open(enc.stream)
    assert np.array_equal(lfc.lfc_decode_rgb(lf).cpu().numpy(), words)
    # a render by decoded views, whose workgroups skip the chunks of unread views
    v = torch.tensor([(0, 0, 0, 0), (U - 1, V - 1, 0.25, -0.5), ((U - 1) / 2, (V - 1) / 3, 1, 1)],
                     dtype=torch.float32, device="cuda")
    some = lfc.lfc_render_views(lf, v, W, H, cfg=(lfc.RENDER_DECODED, 0, 0))
    assert torch.equal(some, lfc.lfc_render_views(lf, v, W, H, cfg=(lfc.RENDER_TILES, 0, 0)))
    # and the batched decode, beside a light field whose key views are all held
    few = lfc.lfc_open(oracle_encode(make_lf(4, 4, 40, 16, seed=3), block=block, levels=2, cluster=(2,)).stream)
    reqs = [(k % 2, 4 * W, 4 * H, (0.5, 0.25 * k, 0.0, 0.0)) for k in range(6)]
    outs = lfc.Batch().render([lf, few], reqs)
    for (li, w, h, view), o in zip(reqs, outs):
        one = lfc.lfc_render_views([lf, few][li], torch.tensor([view], dtype=torch.float32, device="cuda"), w, h,
                                   cfg=(lfc.RENDER_TILES, 0, 0))
        assert torch.equal(o, one[0])
