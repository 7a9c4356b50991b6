"""How exact the floating outputs are, against 64 bits: the activations that a step hands out."""
import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hire():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2402_09360_amd import hire as H
    return H


def log(msg):
    print(msg, flush=True)
@pytest.mark.parametrize("d,N,B,k,kp,kind", [
    (512, 6000, 5, 300, 1500, "int4"),      # 5 to 15 tokens
    (2048, 4096, 15, 205, 820, "int4"),
    (96, 2000, 8, 2000, 2000, "lowrank"),   # every unit selected
    (256, 3001, 9, 7, 300, "lrq"),
    (8224, 300, 2, 20, 60, "int4"),         # few tokens, too long for the route of their own
    (160, 20003, 3, 900, 3000, "int4"),     # ... with more than 16384 units
    (256, 900, 16, 50, 200, "int4"),        # from 16 tokens on: a union of at most 1024 units
    (128, 16390, 24, 80, 800, "int4"),      # ... of more than 16384
    (800, 5003, 33, 251, 1003, "int4"),     # ... of an odd number
])
def test_activations_are_rounded_once_from_64_bits(hire, oracle, d, N, B, k, kp, kind):
    """Half an ulp: products are exact in fp64, a sum of d of them is off by at most d 2^-53 of the sum of their
    magnitudes, which numpy's own sum is as well - together less than 2^-36 of it."""
    log(f"activations d={d} N={N} B={B} k={k} kp={kp} {kind}")
    L = I.ffn_layer(331 + B, d, N) if kind == "int4" else I.lowrank_ffn_layer(332 + B, d, N, 32)
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank", lrq=kind == "lrq")
    x = I.tokens(333 + B, B, d)
    got, _ = T.check_ffn(layer, scorer, L, x, k, kp)
    W, xf = I.bf16_bits_to_f64(L["w1u"]), I.bf16_bits_to_f64(x)
    for b in range(B):
        rows = W[got["topk_idx"][b]]
        h = np.maximum(rows @ xf[b], 0.0)
        slack = 2.0 ** -36 * (np.abs(rows) @ np.abs(xf[b]))
        err = np.abs(got["topk_val"][b].astype(np.float64) - h)
        assert (err <= 2.0 ** -24 * h + slack).all(), (b, (err / np.maximum(h, 1e-30)).max() * 2.0 ** 24)
