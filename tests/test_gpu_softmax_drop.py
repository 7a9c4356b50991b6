"""Long vocabularies, the shortlist cut out of the keys at or above the maxima's bound: classes that come in copies, so that the
key at the cut belongs to several of them and the higher classes go; one token (whose logits are counted in bins between the
smallest and the largest) and batches.  Against the oracle; what the steps did shows that the cut was taken from that list."""
import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


def _run(layer, x, k, kp, want, counts):
    from paper_2402_09360_amd import hire
    ws = hire.alloc_workspace(hire.hire_softmax_workspace_bytes(layer, x.shape[0], k, kp))
    for got in T.run_softmax(layer, x, k, kp, steps=2, ws=ws):
        T.compare_softmax(got, want)
    # tokens whose shortlist was taken from the keys instead, narrowed selections, steps that filled key histograms
    assert hire.hire_debug_general_fallbacks(ws) == counts


@pytest.mark.parametrize("B", [1, 4])
@pytest.mark.parametrize("c,copies,k,kp", [(40000, 3, 16, 301), (40000, 20, 64, 256), (33001, 60, 8, 400), (50000, 1, 1, 777),
                                           (40000, 60, 8, 300)])
def test_copies_at_the_cut(oracle, B, c, copies, k, kp):
    assert torch.cuda.is_available(), "these tests need the MI355X"
    d = 128
    W = I.classifier(751 + copies, -(-c // copies), d)
    W = np.ascontiguousarray(W[np.random.default_rng(752).permutation(np.arange(c) // copies)])
    layer, scorer = T.make_softmax_layer(W)
    print(f"c={c} in {copies} copies, B={B} k={k} k'={kp}", flush=True)
    x = I.tokens(753, B, d)
    want = oracle.softmax_step(W, scorer, x, k, kp, want_acc=True)
    # one token and a large k' for its workgroups' slots: the key histograms
    _run(layer, x, k, kp, want, (0, 0, 1 if B == 1 and kp >= 400 else 0))


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
    _run(layer, x, k, kp, want, (0, 0, 0))


@pytest.mark.parametrize("B", [1, 4])
def test_more_copies_at_the_cut_than_the_list_holds(oracle, B):
    """Hundreds of copies of the class at the cut: the shortlist comes from the keys themselves, in every step."""
    from paper_2402_09360_amd import hire
    c, d, k, kp = 40000, 128, 8, 300
    W = I.classifier(771, 100, d)
    W = np.ascontiguousarray(W[np.random.default_rng(772).permutation(np.arange(c) // 400)])
    layer, scorer = T.make_softmax_layer(W)
    print(f"crowded cut, B={B}", flush=True)
    x = I.tokens(773, B, d)
    want = oracle.softmax_step(W, scorer, x, k, kp, want_acc=True)
    ws = hire.alloc_workspace(hire.hire_softmax_workspace_bytes(layer, B, k, kp))
    for got in T.run_softmax(layer, x, k, kp, steps=2, ws=ws):
        T.compare_softmax(got, want)
    assert hire.hire_debug_general_fallbacks(ws)[0] == 2 * B
