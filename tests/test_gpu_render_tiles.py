"""GPU tests of the tile renderer, a lane of which decodes one channel of a
footprint block, and of its choice of tiles: one-pixel outputs, single rows and
columns, strong minification, magnification, wide and high outputs, trees of one
to four levels, with and without a focal shift.  The library's choice gives the
bytes of explicit tiles and of the decoded path, and the oracle's values (1e-5,
as every render test).
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import make_lf, max_abs, oracle_encode, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu

FIELDS = [
    # U, V, W, H, block, levels
    (9, 9, 90, 61, 4, 3),
    (6, 5, 203, 120, 4, 1),
    (8, 8, 120, 90, 4, 4),
    (7, 6, 97, 101, 2, 3),
    (5, 5, 150, 130, 8, 2),
]
SIZES = [(1, 1), (1, 40), (75, 1), (3, 2), (12, 9), (65, 17), (130, 33), (40, 100)]


@pytest.mark.parametrize("disparity", [0.0, 1.25])
@pytest.mark.parametrize("field", FIELDS, ids=[f"{f[0]}x{f[1]}x{f[2]}x{f[3]}-B{f[4]}-L{f[5]}" for f in FIELDS])
def test_chosen_tiles(gpu, field, disparity):
    U, V, W, H, block, levels = field
    say("tiles", field, disparity)
    enc = oracle_encode(make_lf(U, V, W, H, seed=W + levels), block=block, levels=levels, cluster=(2,) * (levels - 1),
                        blk_threshold=block * block, quant_bits=1)
    lf = lfc.lfc_open(enc.stream)
    views = np.array([[0.3 * U, 0.6 * V, 1.5, -2.0], [U - 1, 0, -W, H]], dtype=np.float32)
    v = torch.from_numpy(views).cuda()
    for w, h in SIZES:
        try:
            got = lfc.lfc_render_views(lf, v, w, h, cfg=(lfc.RENDER_AUTO, 0, 0, disparity))
        except lfc.LFCError:   # too strongly minified for any tile: as with 8 x 2 tiles
            with pytest.raises(lfc.LFCError):
                lfc.lfc_render_views(lf, v, w, h, cfg=(lfc.RENDER_TILES, 8, 2, disparity))
            continue
        assert torch.equal(got, lfc.lfc_render_views(lf, v, w, h, cfg=(lfc.RENDER_DECODED, 0, 0, disparity))), (w, h)
        for tile in ((8, 2), (5, 7)):
            try:
                t = lfc.lfc_render_views(lf, v, w, h, cfg=(lfc.RENDER_TILES, *tile, disparity))
            except lfc.LFCError:
                continue
            assert torch.equal(got, t), (w, h, tile)
        if disparity == 0.0:
            assert max_abs(got.cpu().numpy(), oracle.render(enc.r0, U, V, W, H, views, w, h)) <= 1e-5
