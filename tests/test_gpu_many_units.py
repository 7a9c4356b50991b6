"""One to five tokens on more units than the route for few tokens holds, 16385 to 32768: all scorers, one token through the
batch's kernels, unions of at most and of more than 16384 units (fp64 values ranked, or filter and refine), a token of zeros,
equal units.  Against the oracle."""
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


@pytest.mark.parametrize("kind", ["int4", "lowrank", "lrq"])
@pytest.mark.parametrize("d,N,B,k,kp", [(64, 16385, 1, 100, 1000), (96, 32768, 1, 4000, 20000), (64, 20002, 2, 500, 8192),
                                        (64, 20001, 2, 500, 8193), (64, 32767, 4, 700, 6000), (96, 17001, 4, 300, 4096),
                                        (64, 24003, 5, 900, 4001), (64, 32766, 17, 90, 3000)])
def test_many_units(hire, oracle, kind, d, N, B, k, kp):
    print(f"{kind} d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1500 + d, d, N) if kind == "int4" else I.lowrank_ffn_layer(1500 + d, d, N, 32)
    L["w1u"][N // 2:N // 2 + 30] = L["w1u"][N // 2]
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank", lrq=kind == "lrq")
    x = I.tokens(1501 + B, B, d)
    if B > 1:
        x[1] = 0
    T.check_ffn(layer, scorer, L, x, k, kp)
