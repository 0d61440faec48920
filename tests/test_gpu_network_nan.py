"""GPU tests of inference where features, weights or a layer's sums are not
finite: the ReLU takes a NaN of either sign, given or made from infinities, to
0, in layer 1 and in layer 2, so a logit is what the same forward pass in numpy
gives.  Tolerance: that of a row with a NaN feature (test_gpu_network.py), 1e-2
of the logits' scale.
"""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from helpers import say
from paper_1805_06019_amd import control, lfc

pytestmark = pytest.mark.gpu

PNAN, NNAN = 0x7FC0, 0xFFC0
W1, B1, W2, B2, W3, B3 = 0, 1024, 1088, 5184, 5248, 7616
FEATURES = {"finite": [], "+nan": [np.nan], "-nan": [np.copysign(np.nan, -1)], "inf": [np.inf], "-inf": [-np.inf],
            "inf, -inf": [np.inf, -np.inf], "nan, inf": [np.nan, np.inf], "-nan, -inf": [np.copysign(np.nan, -1), -np.inf]}
# parameters set to a NaN: (first, step, count)
NANS = {"none": None, "a bias of layer 1": (B1 + 7, 1, 1), "a weight of layer 1": (W1 + 16 * 9 + 3, 1, 1),
        "every bias of layer 1": (B1, 1, 64), "a bias of layer 2": (B2 + 40, 1, 1), "every bias of layer 2": (B2, 1, 64),
        "a column of layer 2": (W2 + 5, 64, 64), "a weight of layer 2": (W2 + 64 * 3 + 20, 1, 1)}


def forward(w, x, bf16):
    p = omlp.unpack(w)
    r = (lambda v: omlp.from_bf16_bits(control.to_bf16_bits(v.astype(np.float32))).astype(np.float64)) if bf16 else (lambda v: v)

    def layer(h, k):
        return (h[:, None, :] * p["W" + k]).sum(-1) + p["b" + k]

    with np.errstate(all="ignore"):
        h1 = r(np.fmax(layer(r(x), "1"), 0.0))
        return layer(r(np.fmax(layer(h1, "2"), 0.0)), "3")


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("signs", ["mixed", "negative", "positive"])
def test_relu_takes_every_nan_to_zero(gpu, bf16, signs):
    prec = lfc.MLP_BF16 if bf16 else lfc.MLP_FP32
    rng = np.random.default_rng(41)
    base = control.init_weights(41)
    base[B1:W2] = rng.normal(0, 0.1, 64)
    base[B2:W3] = rng.normal(0, 0.1, 64)
    base[B3:] = rng.normal(0, 0.1, 37)
    if signs != "mixed":   # of layer 2, so that all of its NaNs come from products of one sign
        base[W2:B2] = np.abs(base[W2:B2]) * (1 if signs == "positive" else -1)
    wrong = []
    for where, span in NANS.items():
        for nan in (PNAN, NNAN) if span else (0,):
            bits = control.to_bf16_bits(base)
            if span:
                bits[span[0]:span[0] + span[1] * span[2]:span[1]] = nan
            x = rng.uniform(0, 1, (64, 16)).astype(np.float32)
            for k, v in enumerate(FEATURES.values()):
                for i, f in enumerate(v):
                    x[8 * k + 3, (5 + 7 * i) % 16] = f
            say("nan", bf16, signs, where, hex(nan))
            z = lfc.mlp_infer(torch.from_numpy(bits.view(np.int16)).cuda(), torch.from_numpy(x).cuda(), logits=True,
                              precision=prec)[3].cpu().numpy()
            want = forward(omlp.from_bf16_bits(bits).astype(np.float64), x.astype(np.float64), bf16)
            for row in range(64):
                g, e = z[row], want[row]
                fin = np.isfinite(e)
                with np.errstate(invalid="ignore"):
                    same = np.array_equal(np.isnan(g), np.isnan(e)) and np.array_equal(g[~fin & ~np.isnan(e)], e[~fin & ~np.isnan(e)])
                    close = (np.abs(g - e)[fin] <= 1e-2 * max(1.0, np.abs(e[fin]).max(initial=0.0))).all()
                if not (same and close):
                    wrong.append((where, hex(nan), row, g[:4].tolist(), e[:4].tolist()))
    assert not wrong, (len(wrong), wrong[:6])
