"""The selection of k' beside the filter stage over all rows (both sides of its line), against the oracle: bit for bit in
every index, with tokens whose shortlists are few rows of all, thresholds among the zeros, and rows that no token may
select although their activation is the largest."""
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
    (32, 64, 9, 3, 9), (96, 777, 16, 20, 60), (64, 5003, 17, 251, 1003), (800, 1001, 33, 50, 200),  # a tile; odd rows
    (64, 12289, 64, 100, 900), (64, 16384, 40, 819, 3276), (64, 16390, 12, 300, 2000), (32, 32767, 48, 100, 2000),  # more
    (1024, 15000, 17, 400, 1500), (1024, 12000, 17, 400, 1500)])  # behind the selection, beside it  # than one round
def test_all_rows(hire, oracle, d, N, B, k, kp):
    print(f"ffn_step d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(970 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(971 + B, B, d)
    x[1, :] = 0                                   # ties among zeros
    x[2:, :] = np.where(np.arange(d) % 3 == 0, x[2, :], x[2:, :])  # shortlists overlap
    T.check_ffn(layer, scorer, L, x, k, kp)


def test_a_unit_outside_the_union_is_never_selected(hire, oracle):
    """The int4 copy of a row is replaced by zeros: its activation is by far the largest, its key none."""
    d, N, B, k, kp = 64, 2000, 20, 30, 200
    L = I.ffn_layer(980, d, N)
    x = I.tokens(981, B, d)
    L["w1u"][37, :] = x[5, :]
    layer, (kind, q, s) = T.make_ffn_layer(L)
    q = q.copy()
    q[37, :] = 0
    packed = layer.q4.view(torch.uint8)[:N * d // 2].view(N, d // 2)
    packed[37] = 0
    got, _ = T.check_ffn(layer, (kind, q, s), L, x, k, kp)
    assert 37 not in got["cand"]


@pytest.mark.parametrize("d,N,r,B,k,kp", [
    (40, 64, 8, 9, 3, 9), (72, 777, 24, 16, 20, 60), (520, 5003, 136, 17, 100, 1003),   # odd rows, ranks and token lengths
    (1032, 1033, 1024, 5, 50, 200), (64, 16384, 16, 33, 819, 3276), (64, 16384, 40, 64, 100, 900),  # beside the filter stage
    (1024, 13000, 24, 6, 400, 700),                                                      # in front of it
    (64, 16390, 16, 12, 300, 2000)])                                                     # rows too long for the fp64 keys
def test_lowrank_keys(hire, oracle, d, N, r, B, k, kp):
    """fp64 keys: the projection's sums over all rows of Z1, the scores of whole rows per wave, their selection."""
    print(f"ffn_step lowrank d={d} N={N} r={r} B={B} k={k} k'={kp}", flush=True)
    L = I.lowrank_ffn_layer(990 + d, d, N, r)
    layer, scorer = T.make_ffn_layer(L, lowrank=True)
    x = I.tokens(991 + B, B, d)
    x[1, :] = 0
    T.check_ffn(layer, scorer, L, x, k, kp)
