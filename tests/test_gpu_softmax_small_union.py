"""The softmax step's filter stage on unions of few classes: as many as 256 workgroups of sixteen hold and just beyond, sixteen
tokens and seventeen; a few workgroups, whose maxima are few, and workgroups with fewer than sixteen classes.  Against the
oracle."""
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
    (64, 9000, 16, 16, 256, 0.0), (64, 9000, 16, 16, 257, 0.0), (64, 4096, 3, 20, 2000, 0.9), (64, 4097, 3, 20, 2000, 0.0),
    (96, 5000, 17, 4, 20, 0.0), (96, 5000, 17, 5, 60, 0.99), (2048, 3000, 17, 16, 100, 0.9), (64, 33000, 40, 64, 150, 0.9),
    (128, 33000, 64, 128, 300, 0.99)])
def test_softmax_small_union(hire, oracle, d, c, B, k, kp, rho):
    print(f"softmax d={d} classes={c} B={B} k={k} k'={kp} rho={rho}", flush=True)
    W = I.classifier(1500 + B, c, d)
    W[c // 3:c // 3 + 50] = W[c // 3]
    layer, scorer = T.make_softmax_layer(W)
    x = I.correlated_tokens(1501, B, d, rho) if rho else I.tokens(1501, B, d)
    x[1, :] = 0
    T.check_softmax(layer, scorer, W, x, k, kp)
