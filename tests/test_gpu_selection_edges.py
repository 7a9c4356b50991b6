"""Selections on rows that a program masks or that carry many equal values: the rows of topk_select that are selected from
the maxima of interleaved groups (beyond 32768 entries, k up to 2048; one more takes the histograms), and classes whose
logit is minus infinity.  Indices bit for bit."""
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


def _rows(N, k):
    rng = np.random.default_rng(N + k)
    inf = np.float32(np.inf)
    ordinary = rng.standard_normal(N).astype(np.float32)
    masked = np.where(rng.random(N) < 0.6, -inf, ordinary)
    few = np.full(N, -inf, dtype=np.float32)         # fewer numbers than are asked for (k = 1: none)
    few[rng.choice(N, k // 2, replace=False)] = rng.standard_normal(k // 2)
    above = ordinary.copy()
    above[rng.choice(N, 5, replace=False)] = inf     # the window below them holds nothing else
    equal = rng.integers(-3, 4, N).astype(np.float32)
    spread = (ordinary * np.exp2(rng.uniform(-60, 60, N))).astype(np.float32)
    tail = np.zeros(N, dtype=np.float32)             # all that counts in the last entries; -0 counts as +0
    tail[-3:] = [1.0, 2.0, 1.0]
    tail[:N // 2] = -0.0
    return np.stack([ordinary, masked, np.full(N, -inf, dtype=np.float32), few, above, equal, spread, tail,
                     np.sort(ordinary)])


@pytest.mark.parametrize("N", [32769, 49153, 131071])
@pytest.mark.parametrize("k", [1, 700, 2048, 2049])
def test_topk_select_long_rows(hire, oracle, N, k):
    v = _rows(N, k)
    B = v.shape[0]
    scores = torch.from_numpy(v).cuda()
    for relu in (False, True):
        for rank in (False, True):
            flags = (hire.RELU if relu else 0) | (hire.ORDER_RANK if rank else 0)
            ws = hire.alloc_workspace(hire.hire_topk_workspace_bytes(B, N, k, flags))
            ref = np.maximum(v, 0) if relu else v
            for call in range(2):
                log(f"topk_select N={N} k={k} relu={relu} rank={rank} call {call}")
                idx, val = hire.topk_select(scores, k, relu=relu, rank_order=rank, workspace=ws)
                torch.cuda.synchronize()
                idx, val = idx.cpu().numpy(), val.cpu().numpy()
                for b in range(B):
                    want = oracle.topk_f32(v[b], k, relu=relu, rank_order=rank)
                    assert np.array_equal(idx[b], want), (relu, rank, call, b)
                    assert np.array_equal(val[b], ref[b][want] + np.float32(0.0)), (relu, rank, call, b)


@pytest.mark.parametrize("c,B,k,kp", [(5000, 16, 32, 400), (5000, 40, 300, 700), (40000, 16, 64, 300), (5000, 3, 16, 300),
                                      (40000, 1, 40, 1024)])
def test_softmax_step_with_masked_classes(hire, oracle, c, B, k, kp):
    """A third of the classes has a logit of minus infinity (one weight is, its component of every token is positive): they
    are shortlisted by a scorer that does not know, and come last.  Their norm leaves the filter stage no bound."""
    d, r = 256, 64
    W = I.classifier(351, c, d)
    W[::3, 0] = 0xFF80
    z1, z2 = I.normal_bf16(352, (d, r), d ** -0.5), I.normal_bf16(353, (c, r), 1.0)
    layer, scorer = T.make_softmax_layer(W, lrq=(z1, z2))
    x = I.tokens(354, B, d)
    x[:, 0] = 0x3F80
    log(f"softmax_step with masked classes c={c} B={B} k={k} kp={kp}")
    want = oracle.softmax_step(W, scorer, x, k, kp)
    for got in T.run_softmax(layer, x, k, kp, steps=3):
        assert np.array_equal(got["cand"], want["cand"])
        assert np.array_equal(got["top_idx"], want["top_idx"])
        assert np.isfinite(got["top_logit"]).all() and not (got["top_idx"] % 3 == 0).any()
        T.assert_float_close(got["top_prob"], want["top_prob"], "top_prob")


@pytest.mark.parametrize("d,N,B,k,kp", [
    (64, 5461, 8, 300, 1400),     # the longest rows that eight tokens take the few-token kernels with
    (64, 5462, 8, 300, 1400),     # one unit more: the longer sequence
    (96, 8192, 6, 8192, 8192),    # six tokens, everything selected
    (4096, 640, 8, 40, 160),      # the longest eight tokens
    (4128, 640, 5, 40, 160),      # too long for them
    (160, 65, 7, 5, 20),          # a workgroup with one unit
    (288, 1000, 5, 1, 1),
])
def test_five_to_eight_tokens(hire, oracle, d, N, B, k, kp):
    log(f"five to eight tokens d={d} N={N} B={B} k={k} kp={kp}")
    L = I.ffn_layer(361 + B, d, N)
    L["w1u"][N // 4:N // 4 + 40] = L["w1u"][N // 4]     # equal keys and activations
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(362 + B, B, d)
    x[B // 2] = 0                                       # every key ties at zero
    T.check_ffn(layer, scorer, L, x, k, kp)
