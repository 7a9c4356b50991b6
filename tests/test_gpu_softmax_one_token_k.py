"""One token's softmax step where the k largest logits are more than a wave and than the sixteen-lane rows of a workgroup hold at
once: both sides of 64, the largest k of the short sequence and the first beyond it; classes of equal logits across the line;
both int4 scorers.  Against the oracle."""
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


@pytest.mark.parametrize("k,kp", [(63, 512), (64, 64), (65, 300), (100, 1536), (127, 127), (128, 128), (128, 1536), (129, 700)])
@pytest.mark.parametrize("copies", [1, 100])
def test_softmax_one_token(hire, oracle, k, kp, copies):
    print(f"softmax of one token k={k} k'={kp} copies={copies}", flush=True)
    d, c = 128, 40000
    W = I.classifier(1400 + k, c, d)
    W[c // 3:c // 3 + copies] = W[c // 3]
    x = I.tokens(1401, 1, d)
    if copies > 1:  # the copies among the largest: more equal logits than places
        x[0, :] = W[c // 3]
    layer, scorer = T.make_softmax_layer(W)
    T.check_softmax(layer, scorer, W, x, k, kp)
