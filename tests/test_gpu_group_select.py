"""Groups of eight, both selections of the longer sequence: one group, the waves' shares at their ends, the loads of 2048 and
4096 groups, unions shorter than their bound, everything selected, equal groups and groups of zeros.  Against the oracle."""
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


@pytest.mark.parametrize("kind", ["int4", "lowrank"])
@pytest.mark.parametrize("d,N,B,k,kp", [(64, 64, 9, 8, 8), (64, 8 * 513, 17, 8 * 40, 8 * 100), (96, 8 * 511, 33, 8 * 511, 8 * 511),
                                        (64, 8 * 2048, 16, 8 * 100, 8 * 400), (64, 8 * 2049, 10, 8 * 200, 8 * 2049),
                                        (64, 8 * 4096, 64, 8 * 90, 8 * 300), (64, 8 * 4095, 9, 8 * 1000, 8 * 3000),
                                        (64, 8 * 4200, 12, 8 * 50, 8 * 400)])
def test_group_select(hire, oracle, kind, d, N, B, k, kp):
    print(f"{kind} groups d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1600 + d, d, N) if kind == "int4" else I.lowrank_ffn_layer(1600 + d, d, N, 64)
    same = N // 16 * 8
    L["w1u"][same:same + 80] = L["w1u"][same]
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank")
    x = I.correlated_tokens(1601, B, d, 0.9)
    x[1] = 0
    T.check_ffn_group(layer, scorer, L, x, k, kp, 8)


@pytest.mark.parametrize("d,N,B,k,kp", [(288, 8192, 5, 8 * 60, 8 * 204), (288, 8200, 5, 8 * 60, 8 * 204), (256, 8192, 8, 8 * 61, 8 * 203),
                                        (288, 64, 8, 8, 8 * 2), (480, 8 * 1023, 8, 8 * 1023, 8 * 1023)])
def test_five_to_eight_tokens_around_the_line_between_the_routes(hire, oracle, d, N, B, k, kp):
    print(f"groups around the line d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1610 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1611 + B, B, d)
    x[1] = 0
    T.check_ffn_group(layer, scorer, L, x, k, kp, 8)
