"""The softmax step's filter and refine at the edges of its rule and of the maxima that it finds its mark with: three tokens,
tiles that fill one, two, three or four groups of sixteen candidates, k of the largest size, tokens that share their
candidates, equal classes.  Against the oracle."""
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


@pytest.mark.parametrize("d,c,B,k,kp,rho", [
    (64, 4000, 3, 4, 60, 0.0), (64, 4000, 3, 5, 60, 0.0),         # three workgroups: twelve maxima, and the rule's other side
    (96, 33000, 15, 32, 300, 0.99), (128, 33000, 16, 60, 600, 0.9),  # tiles of few candidates: quarters and halves of a group
    (64, 9000, 5, 20, 1800, 0.0), (64, 33000, 15, 256, 1100, 0.0), (64, 33000, 16, 512, 2048, 0.9),
    (64, 20000, 40, 512, 1024, 0.0), (64, 20000, 33, 512, 2000, 0.99), (2048, 3000, 9, 16, 200, 0.9)])
def test_softmax_filter(hire, oracle, d, c, B, k, kp, rho):
    print(f"softmax d={d} classes={c} B={B} k={k} k'={kp} rho={rho}", flush=True)
    W = I.classifier(1200 + B, c, d)
    W[c // 3:c // 3 + 50] = W[c // 3]
    layer, scorer = T.make_softmax_layer(W)
    x = I.correlated_tokens(1201, B, d, rho) if rho else I.tokens(1201, B, d)
    x[1, :] = 0
    T.check_softmax(layer, scorer, W, x, k, kp)
