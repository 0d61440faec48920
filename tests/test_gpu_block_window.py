"""GPU tests of the whole-field decoders' block windows: 2 x 2 and 4 x 4 blocks
of every kind and width of low bits, from those of one bit to the plain ones too
wide for a window, at every quantisation, with and without staging, for chunks
of one, two and more blocks per lane; exact against the oracle.
"""
import numpy as np
import pytest

import oracle
from helpers import oracle_encode, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu

WIDE = 0xE00   # plain blocks of 10 to 12 bits, which a mask of one kind needs beside it
KINDS = dict(all=0, plain=0xFFF, trit=0x7F000 | WIDE, quint=0x3F80000 | WIDE)


def ramp_lf(U, V, W, H, seed):
    """Views that differ by noise whose amplitude grows from left to right."""
    rng = np.random.default_rng(seed)
    amp = 127.0 * (np.arange(W) / max(W - 1, 1)) ** 2
    x = 128 + rng.uniform(-1, 1, (V, U, H, W, 3)) * amp[None, None, None, :, None]
    return np.clip(np.rint(x), 0, 255).astype(np.uint8)


@pytest.mark.parametrize("q", range(5))
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("block", [2, 4])
def test_block_windows(gpu, block, kind, q):
    say("windows", block, kind, q)
    enc = oracle_encode(ramp_lf(5, 6, 131, 6, seed=17 * block + q), block=block, levels=3, cluster=(2, 2),
                        quant_bits=q, range_mask=KINDS[kind])
    rgb = oracle.ycocg_inverse(np.ascontiguousarray(np.transpose(enc.r0, (0, 2, 3, 1)))).astype(np.uint32)
    words = (rgb[..., 0] | (rgb[..., 1] << 8) | (rgb[..., 2] << 16)).view(np.int32)
    for tile in (0, 512 // block, 2048):   # default; chunks of a few runs; up to four blocks a lane
        lf = lfc.lfc_open(enc.stream, tile_blocks=tile)
        for cap in (None, 0, -1, 600):
            got = lfc.lfc_decode_blocks(lf, None, lfc.LAYOUT_IMAGES, stage_cap_words=cap).cpu().numpy()
            assert np.array_equal(got, enc.r0), (tile, cap)
        assert np.array_equal(lfc.lfc_decode_rgb(lf).cpu().numpy(), words), tile
