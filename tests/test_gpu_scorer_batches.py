"""The int4 scorer for batches at the edges of its tiles and dispatch: rows per workgroup, token tiles of 16, the places where
it quantises the tokens itself and where a kernel in front does, segments of long rows, one or two row tiles per wave on
vocabularies.  Integer sums and index sets bit for bit, against the oracle."""
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


def log(msg):
    print(msg, flush=True)


def _tokens(seed, B, d):
    """Ordinary tokens, one of zeros, one of denormal bf16 values (its scale's reciprocal is not used), one of equal
    values, which are all quantised to the largest code."""
    x = I.tokens(seed, B, d)
    if B > 4:
        x[1, :] = 0
        x[2, :] = np.arange(d) % 7
        x[3, :] = 0x3F80
    return x


@pytest.mark.parametrize("d,N,B", [
    (32, 17, 9), (2048, 1024, 16), (2048, 1025, 32),           # quantised by the scorer, 16 and 32 rows per workgroup
    (2080, 1023, 16), (96, 3001, 33), (4128, 130, 64),         # codes: long tokens, more than 32 tokens, three segments
    (64, 8192, 17), (64, 8193, 31), (160, 16384, 24),          # 32 and 64 rows per workgroup
    (64, 16385, 16), (32, 32768, 64),                          # 128
    (512, 4096, 33), (512, 4097, 64), (544, 4097, 33),         # more than 32 tokens: short ones are quantised here too
    (1024, 20003, 24), (1056, 8193, 7), (2048, 16385, 17),     # the vectors of a token per lane
    (544, 1023, 40), (1024, 4000, 40), (1024, 4097, 40), (800, 8193, 34), (1024, 16385, 40),  # four tokens per wave, two
    (1024, 4097, 41), (1056, 4097, 33)])                       # vectors each: 16, 32, 64, 128 rows; past each limit
def test_ffn_rows(hire, oracle, d, N, B):
    log(f"ffn_step d={d} N={N} B={B}")
    L = I.ffn_layer(900 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    T.check_ffn(layer, scorer, L, _tokens(901 + B, B, d), max(1, N // 40), max(2, N // 8))


@pytest.mark.parametrize("d,N,B", [
    (96, 15, 21), (96, 700, 33), (1056, 2048, 32), (32, 1366, 64),   # sixteen tokens per workgroup: tiles of 16 rows, the last part
    (160, 2049, 21), (64, 2731, 48), (1024, 2100, 49),               # of one token and of sixteen; 32 rows
    (2048, 4097, 21), (544, 5461, 48), (64, 8000, 17),               # 64; (17 tokens take no parts)
    (2048, 8193, 25), (1056, 8192, 49), (32, 10922, 33),             # 128
    (512, 8193, 24), (544, 8193, 24), (544, 8192, 24), (544, 8193, 25),  # long tokens, many rows: from 25 on
    (512, 4097, 28), (1024, 4097, 28), (1056, 4097, 28), (512, 2049, 28), (1056, 2049, 28),  # steps per wave: one, two, four; 32 rows
    (64, 1280, 33), (64, 1281, 33), (544, 2561, 48), (1056, 5120, 40), (1056, 5121, 40), (512, 10240, 47), (512, 10241, 47),  # a round of every die
    (32, 10923, 33), (2080, 1000, 33), (32, 16385, 21)])             # past each limit
def test_parts_of_sixteen_tokens(hire, oracle, d, N, B):
    log(f"ffn_step d={d} N={N} B={B}")
    L = I.ffn_layer(940 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    T.check_ffn(layer, scorer, L, _tokens(941 + B, B, d), max(1, N // 40), max(2, N // 8))


@pytest.mark.parametrize("d,N,r,B", [(576, 1500, 544, 64), (576, 4100, 512, 64), (1536, 1537, 64, 32), (1056, 2090, 1024, 17), (64, 8200, 32, 48),
                                     (96, 20003, 96, 18), (64, 16390, 64, 3)])
def test_ffn_rows_lrq(hire, oracle, d, N, r, B):
    """The intermediate is rounded and quantised by the second product's kernel."""
    log(f"ffn_step lrq d={d} N={N} r={r} B={B}")
    L = I.lowrank_ffn_layer(920 + d, d, N, r)
    layer, scorer = T.make_ffn_layer(L, lrq=True)
    T.check_ffn(layer, scorer, L, _tokens(921, B, d), max(1, N // 40), max(2, N // 8))


@pytest.mark.parametrize("d,c,B", [
    (64, 32769, 16), (32, 32897, 17), (64, 65536, 64), (64, 65537, 48),  # row tiles at their ends; 64 x 65536: two per wave
    (2080, 40000, 33), (96, 131000, 64)])
def test_vocabulary_rows(hire, oracle, d, c, B):
    log(f"softmax_step d={d} c={c} B={B}")
    W = I.classifier(940 + d, c, d)
    layer, scorer = T.make_softmax_layer(W)
    x = _tokens(941, B, d)
    _, want = T.check_softmax(layer, scorer, W, x, 8, 300)
    T.compare_softmax(T.run_softmax(layer, x, 8, 300, debug=False), dict(want, acc=None))  # no sums wanted: their own epilogue


@pytest.mark.parametrize("copies", [3, 300])
def test_vocabulary_rows_adjacent_shortlist(hire, oracle, copies):
    """Every token's largest keys next to each other, in two rounds of a workgroup: 300 are more than a wave's list holds
    (the token is then selected from its keys)."""
    d, c, B = 32, 140000, 33
    log(f"softmax_step d={d} c={c} B={B} copies={copies}")
    W = I.classifier(960, c, d)
    x = _tokens(961, B, d)
    for b in range(B):
        at = 4100 * b + 37
        W[at:at + copies, :] = x[b]
    layer, scorer = T.make_softmax_layer(W)
    T.check_softmax(layer, scorer, W, x, 8, 500)
