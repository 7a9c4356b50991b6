"""One token with the int4 low-rank scorer, both products in one kernel: the smallest and the largest r, waves with more rows
of Z1 than there are and with one, tokens of several passes, units that do not fill a wave's rows; and the two sides of the
rule that chooses it.  Against the oracle."""
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


@pytest.mark.parametrize("d,N,r", [(64, 66, 32), (96, 1001, 96), (512, 2049, 128), (2080, 2083, 160), (2048, 2051, 256),
                                   (2080, 2100, 256), (288, 303, 288), (4096, 4097, 128), (544, 16384, 64)])
def test_lrq_one_token(hire, oracle, d, N, r):
    print(f"ffn_step lrq d={d} N={N} r={r}", flush=True)
    L = I.lowrank_ffn_layer(1300 + d, d, N, r)
    layer, scorer = T.make_ffn_layer(L, lrq=True)
    k, kp = max(1, N // 40), max(2, N // 8)
    T.check_ffn(layer, scorer, L, I.tokens(1301, 1, d), k, kp)
    got, _ = T.check_ffn(layer, scorer, L, np.zeros((1, d), dtype=np.uint16), k, kp)
    assert not got["y"].any()
