"""GPU encoder at the edges of its kernels' tiles: plane widths for 2, 4 and 8
samples a thread, more nodes than one 64-node chunk of a group, groups whose
last chunk or word is full or partial, clusters cut at the grid's edge, block
counts around a workgroup, and every range code.  The stream and the
statistics equal the host encoder's.
"""
import numpy as np
import pytest
import torch

from helpers import make_lf, say
from paper_1805_06019_amd import lfc

pytestmark = pytest.mark.gpu

CASES = [
    # U, V, W, H, parameters
    (8, 8, 6, 6, dict(block=2, levels=2, cluster=(2,))),                       # wp 6: two samples a thread; 64 nodes
    (13, 5, 10, 4, dict(block=2, levels=2, cluster=(3,))),                     # 65 nodes
    (9, 7, 20, 12, dict(block=4, levels=2, cluster=(2,))),                     # 63 nodes; wp 20: four
    (16, 8, 24, 8, dict(block=4, levels=2, cluster=(2,), blk_threshold=10)),   # 128 nodes; wp 24: eight
    (7, 6, 40, 40, dict(block=8, levels=3, cluster=(3, 2), quant_bits=1)),     # clusters cut at both edges
    (3, 3, 128, 128, dict(block=8, levels=2, cluster=(8,))),                   # 256 blocks; one cluster over the grid
    (3, 2, 1028, 4, dict(block=4, levels=2, cluster=(2,))),                    # 257 blocks
    (12, 11, 9, 5, dict(block=2, levels=3, cluster=(2, 2), pix_threshold=3, blk_threshold=4, quant_bits=2)),
    (2, 2, 16, 16, dict(block=4, levels=2, cluster=(2,), blk_threshold=100000)),   # nothing stored
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}x{c[2]}x{c[3]}-B{c[4]['block']}" for c in CASES])
def test_encoder_edges(gpu, case):
    U, V, W, H, kw = case
    say("gpu encode", case)
    rgb = make_lf(U, V, W, H, seed=U * 31 + W, sigma=6.0)
    p = lfc.Params(U, V, W, H, **kw)
    host, hst = lfc.lfc_encode_ex(rgb, p)
    # the pixels at an odd offset of their allocation
    buf = torch.zeros(rgb.size + 5, dtype=torch.uint8, device="cuda")
    buf[5:] = torch.from_numpy(rgb.reshape(-1))
    dev, dst = lfc.lfc_encode_gpu(buf[5:].view(rgb.shape), p)
    assert dev == host and dst == hst


@pytest.mark.parametrize("code", range(26))
@pytest.mark.parametrize("block", [2, 4, 8])
def test_every_range_code_is_packed(gpu, code, block):
    """Only `code` and the widest range allowed, residuals of its size."""
    say("gpu encode code", code, block)
    bound = 2 << code if code < 12 else (3 << (code - 12) if code < 19 else 5 << (code - 19))
    r = np.random.default_rng(code)
    amp = max(1, min(120, bound // 4))
    rgb = np.clip(128 + r.integers(-amp, amp + 1, (4, 5, 17, 22, 3)), 0, 255).astype(np.uint8)
    p = lfc.Params(5, 4, 22, 17, block=block, levels=2, cluster=(2,), range_mask=(1 << code) | (1 << 11))
    host, hst = lfc.lfc_encode_ex(rgb, p)
    dev, dst = lfc.lfc_encode_gpu(rgb, p)
    assert dev == host and dst == hst
