"""GPU tests of the interpolation, which renders several output rows per
thread: its shared source rows and partial waves, against the tile renderer
(the same bytes) and the oracle (1e-5, as every render test).
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import make_lf, max_abs, oracle_encode, say
from paper_1805_06019_amd import lfc, synth

pytestmark = pytest.mark.gpu

# U, V, W, H, block, out_w, out_h, views: rows repeated (magnified), one after
# the other (equal scale), skipped (minified); one or two lanes in a row's last
# wave; a row count one past a multiple; images one pixel wide or high
CASES = [
    (4, 3, 40, 32, 4, 40, 32, 300),
    (4, 3, 40, 32, 4, 65, 97, 60),
    (4, 3, 40, 32, 4, 66, 9, 400),
    (3, 3, 90, 70, 4, 63, 13, 600),
    (5, 2, 37, 23, 8, 129, 23, 150),
    (3, 3, 30, 1, 2, 64, 5, 1100),
    (3, 3, 1, 30, 2, 3, 33, 300),
    (2, 2, 20, 18, 2, 1, 1, 2100),
    (1, 1, 24, 20, 4, 48, 41, 200),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[2]}x{c[3]}-to-{c[5]}x{c[6]}x{c[7]}" for c in CASES])
def test_rows_per_thread(gpu, case):
    U, V, W, H, B, wo, ho, n = case
    say("interp rows", case)
    levels = 1 if U * V == 1 else 2
    enc = oracle_encode(make_lf(U, V, W, H, seed=W + ho), block=B, levels=levels, cluster=() if levels == 1 else (2,),
                        blk_threshold=2)
    views = synth.novel_views(n, U, V, seed=wo + ho, pan=2.5)
    views[0], views[1] = (0, 0, 0, 0), (U - 1, V - 1, 0.25, -0.5)
    views[2:5, 3] = (-H, 0.5, H)                  # panned off the top and the bottom: one source row throughout
    lf = lfc.lfc_open(enc.stream)
    v = torch.from_numpy(views).cuda()
    out = torch.full((n, 3, ho, wo), float("nan"), device="cuda")
    lfc.lfc_render_views(lf, v, wo, ho, out=out, cfg=(lfc.RENDER_DECODED, 0, 0))
    tiles = lfc.lfc_render_views(lf, v, wo, ho, cfg=(lfc.RENDER_TILES, 0, 0))
    assert torch.equal(out, tiles)
    few = slice(0, 8)
    assert max_abs(out[few].cpu().numpy(), oracle.render(enc.r0, U, V, W, H, views[few], wo, ho)) <= 1e-5


def test_rows_per_thread_in_a_batch_of_sizes(gpu):
    """Requests of several sizes and light fields share the launch; each has
    the bytes of its own render."""
    lfs, sizes = [], [(64, 48), (130, 37), (1, 1), (66, 50), (33, 2)]
    for k, (U, V, W, H, B) in enumerate([(4, 3, 40, 32, 4), (3, 3, 50, 28, 4), (2, 2, 32, 24, 8)]):
        lfs.append(lfc.lfc_open(oracle_encode(make_lf(U, V, W, H, seed=70 + k), block=B, levels=2, cluster=(2,),
                                              blk_threshold=2).stream))
    r = np.random.default_rng(5)
    reqs = []
    for i in range(260):
        li, (w, h) = i % 3, sizes[(i // 3) % len(sizes)]
        p = lfs[li].params
        reqs.append((li, w, h, (r.uniform(0, p.grid_u - 1), r.uniform(0, p.grid_v - 1), r.uniform(-2, 2), r.uniform(-2, 2))))
    outs = lfc.Batch().render(lfs, reqs)
    for (li, w, h, view), o in zip(reqs, outs):
        one = lfc.lfc_render_views(lfs[li], torch.tensor([view], dtype=torch.float32, device="cuda"), w, h,
                                   cfg=(lfc.RENDER_TILES, 0, 0))
        assert torch.equal(o, one[0])
