"""GPU test of the whole-field decode with tiles of 8 x 8 blocks on both sides of
64 and 128 KB, up to the largest that the workgroup's LDS holds, where its
gather tables are smaller: sparse (many runs a chunk) and dense fields, exact
against the oracle.
"""
import numpy as np
import pytest

from helpers import make_lf, oracle_encode, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threshold", [64, 4000])
@pytest.mark.parametrize("grid,levels", [(17, 3), (12, 4)])
def test_largest_tiles(gpu, grid, levels, threshold):
    enc = oracle_encode(make_lf(grid, grid, 72, 16, seed=grid + threshold), block=8, levels=levels,
                        cluster=(2,) * (levels - 1), blk_threshold=threshold, quant_bits=2)
    for tile in (512, 520, 1024, 1032, 1104, 1232 if levels == 3 else 1200):
        say("tile", grid, levels, threshold, tile)
        lf = lfc.lfc_open(enc.stream, tile_blocks=tile)
        for cap in (0, -1):
            got = lfc.lfc_decode_blocks(lf, None, lfc.LAYOUT_IMAGES, stage_cap_words=cap).cpu().numpy()
            assert np.array_equal(got, enc.r0), (tile, cap)
        lf.close()
