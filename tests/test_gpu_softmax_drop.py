"""Long vocabularies, the shortlist cut out of the keys at or above the maxima's bound: classes that come in copies, so that the
key at the cut belongs to several of them and the higher classes go; one token (whose logits are counted in bins between the
smallest and the largest) and batches.  Against the oracle."""
import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 4])
@pytest.mark.parametrize("c,copies,k,kp", [(40000, 3, 16, 301), (40000, 20, 64, 256), (33001, 60, 8, 400), (50000, 1, 1, 777)])
def test_copies_at_the_cut(oracle, B, c, copies, k, kp):
    assert torch.cuda.is_available(), "these tests need the MI355X"
    d = 128
    W = I.classifier(751 + copies, -(-c // copies), d)
    W = np.ascontiguousarray(W[np.random.default_rng(752).permutation(np.arange(c) // copies)])
    layer, scorer = T.make_softmax_layer(W)
    print(f"c={c} in {copies} copies, B={B} k={k} k'={kp}", flush=True)
    x = I.tokens(753, B, d)
    want = oracle.softmax_step(W, scorer, x, k, kp, want_acc=True)
    for got in T.run_softmax(layer, x, k, kp, steps=2):
        T.compare_softmax(got, want)


@pytest.mark.parametrize("B", [1, 4])
@pytest.mark.parametrize("c,k,kp", [(40000, 64, 1024), (33001, 1, 1), (33001, 16, 300)])
def test_logits_that_differ_below_fp32(oracle, B, c, k, kp):
    """A common term of 2^26 beside terms of a few units: all logits round to a handful of fp32 values."""
    d = 256
    W, x = I.classifier(761, c, d).copy(), I.tokens(762, B, d).copy()
    W[:, 0], x[:, 0] = 0x3D00, 0x4F00  # 2^-5, 2^31
    layer, scorer = T.make_softmax_layer(W)
    print(f"close logits, c={c} B={B} k={k} k'={kp}", flush=True)
    want = oracle.softmax_step(W, scorer, x, k, kp, want_acc=True)
    for got in T.run_softmax(layer, x, k, kp, steps=2):
        T.compare_softmax(got, want)
