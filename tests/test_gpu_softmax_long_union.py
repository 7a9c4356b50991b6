"""The softmax step's filter and refine on unions of more classes than one mask of the refining selection stands for: just
beyond 65536 and as many as the route takes; a token of zeros, whose logits are all equal, so that its whole union goes through
the rounds of one workgroup, span by span.  Against the oracle; on no more workspace than fp64 logits of the union take."""
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


@pytest.mark.parametrize("d,c,B,k,kp", [(64, 66000, 33, 64, 1986), (64, 131072, 64, 128, 1536), (96, 140000, 64, 512, 2048),
                                        (64, 100000, 16, 8, 5000)])
def test_softmax_long_union(hire, oracle, d, c, B, k, kp):
    print(f"softmax d={d} classes={c} B={B} k={k} k'={kp}", flush=True)
    W = I.classifier(1300 + B, c, d)
    W[c // 3:c // 3 + 50] = W[c // 3]
    layer, scorer = T.make_softmax_layer(W)
    x = I.tokens(1301, B, d)
    x[1, :] = 0
    got, _ = T.check_softmax(layer, scorer, W, x, k, kp)
    print(f"union of {len(got['cand'])}", flush=True)
    rows = min(c, B * kp)
    assert hire.hire_softmax_workspace_bytes(layer, B, k, kp) >= 8 * B * rows
