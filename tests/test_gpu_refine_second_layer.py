"""The refining selection with the second layer in one kernel (16 tokens and more whose selected rows are few enough) and with its
values rounded from 64 bits, against the oracle: slices of 64 to 512 columns with a remainder, lists that end inside, at and behind a batch of rows, the shared-out list
of the candidates, tokens that the list in LDS does not settle; and infinite second-layer weights."""
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


@pytest.mark.parametrize("d,N,B,k,kp", [
    (32, 1026, 16, 1, 80),         # less than a slice, one entry
    (96, 1090, 16, 128, 300),      # 64 columns: a slice and a half, a batch of rows and no more
    (96, 1090, 17, 129, 300),
    (1056, 2000, 16, 257, 400),    # 128 columns, the last slice of 32
    (544, 3002, 64, 200, 600),     # 256 columns
    (1088, 2048, 64, 513, 700),    # 512 columns
    (64, 16384, 16, 4096, 4096),   # the longest list; all of it selected
    (64, 16382, 33, 700, 1000),    # the last word of the bitmap is not whole
    (8192, 1100, 16, 60, 200),     # the longest token in LDS
    (8224, 1100, 16, 60, 200),     # longer
])
def test_against_the_oracle(hire, oracle, d, N, B, k, kp):
    print(f"ffn_step d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1200 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1201 + B, B, d)
    x[1, :] = 0                                    # threshold among the zeros
    x[3:6, :] = x[2, :]
    T.check_ffn(layer, scorer, L, x, k, kp)


@pytest.mark.parametrize("d,N,B,k,kp", [
    (64, 777, 5, 3, 9),            # a workgroup per token, fewer entries than waves
    (96, 1091, 8, 512, 600),       # a round of workgroups, none left for the candidates' list: all of them share it
    (800, 2003, 16, 250, 400),     # 256 workgroups again
    (2080, 1501, 7, 33, 200),      # rows of more than one request of a wave
    (64, 16390, 6, 300, 1500),     # more units than 16384
    (8224, 1000, 5, 20, 100),      # a token that is not in LDS
    (64, 2001, 33, 372, 800), (64, 2001, 33, 373, 800),  # three rows per wave, and more: the kernel behind the list
])
def test_values_from_64_bits_against_the_oracle(hire, oracle, d, N, B, k, kp):
    print(f"ffn_step d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1220 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1221 + B, B, d)
    x[1, :] = 0
    got, want = T.check_ffn(layer, scorer, L, x, k, kp)
    # one rounding of a 64-bit sum: half an ulp, and the difference between two orders of the sum
    assert (np.abs(got["topk_val"].astype(np.float64) - want["topk_val"]) <= np.abs(want["topk_val"]) * (0.5 + 1e-3) * 2.0 ** -23).all()


def test_infinite_weights_stay_in_their_columns(hire, oracle):
    """Rows that are selected for every token, the first and the last of its list, are infinite in one column each."""
    d, N, B, k, kp = 256, 2050, 16, 100, 300
    L = I.ffn_layer(1210, d, N)
    x = np.repeat(I.tokens(1211, 1, d), B, axis=0)
    L["w1u"][0, :] = L["w1u"][N - 1, :] = x[0, :]    # by far the largest activations
    L["w2u"][0, 5] = 0x7F80
    L["w2u"][N - 1, 200] = 0xFF80
    layer, _ = T.make_ffn_layer(L)
    y = T.run_ffn(layer, x, k, kp)["y"]
    assert (y[:, 5] == np.inf).all() and (y[:, 200] == -np.inf).all()
    assert np.isfinite(np.delete(y, [5, 200], axis=1)).all()
