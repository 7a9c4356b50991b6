"""The softmax step's filter and refine where the union may have more classes than one mask of the refining selection stands for:
layouts for just more than 65536 and for as many as the route takes, on no more workspace than the route through fp64 logits, with
a token of zeros, whose logits are all equal; unions that have 65535 to 65537 and 131072 classes.  Against the oracle.
Tokens with more equal logits than the selection has slots, which are settled in rounds, span by span; what such a token
may cost."""
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


@pytest.mark.parametrize("d,c,B,k,kp", [(64, 66000, 33, 64, 1986), (64, 131072, 64, 128, 1536), (96, 140000, 64, 512, 2048),
                                        (64, 100000, 16, 8, 5000)])
def test_softmax_long_union(hire, oracle, d, c, B, k, kp):
    print(f"softmax d={d} classes={c} B={B} k={k} k'={kp}", flush=True)
    W = I.classifier(1300 + B, c, d)
    W[c // 3:c // 3 + 50] = W[c // 3]
    layer, scorer = T.make_softmax_layer(W)
    x = I.tokens(1301, B, d)
    x[1, :] = 0
    T.check_softmax(layer, scorer, W, x, k, kp)
    # (more than 512 logits go through fp64 always)
    assert hire.hire_softmax_workspace_bytes(layer, B, k, kp) <= hire.hire_softmax_workspace_bytes(layer, B, 513, kp)


def _tiling(c, d, seed):
    """Classes and tokens (all but the last one) whose shortlists tile the vocabulary: class j is far the largest in column j mod
    (d - 1), token t is one in column t alone.  The last column is all classes' by chance."""
    W = I.normal_bf16(seed, (c, d), 0.02)
    j = np.arange(c)
    W[j, j % (d - 1)] = I.f32_to_bf16_bits(1.0 + np.random.default_rng(seed).random(c, dtype=np.float32))
    x = np.zeros((d - 1, d), np.uint16)
    x[np.arange(d - 1), np.arange(d - 1)] = 0x3F80
    return W, x


@pytest.mark.parametrize("c", [65535, 65536, 65537, 131072])
@pytest.mark.parametrize("k", [64, 300])
def test_unions_at_the_edges_of_a_span(hire, oracle, c, k):
    """All classes are candidates.  The last token has most of the logits at its k-th place equal: 3000 classes in both halves of
    the row, the lowest of which come first; and a token of zeros."""
    d, kp = 64, -(-c // 63) + 20
    W, x = _tiling(c, d, 1310)
    last = np.zeros((1, d), np.uint16)
    last[0, 63] = 0x3F80
    W[:, 63] = I.f32_to_bf16_bits(np.random.default_rng(1311).random(c, dtype=np.float32) * 0.5)
    at = np.random.default_rng(1312).permutation(c)
    W[at[:k // 2], 63] = 0x4000
    W[at[k // 2:k // 2 + 3000], 63] = 0x3F80
    x = np.concatenate([x, last])
    print(f"union of all {c} classes, k={k} k'={kp}", flush=True)
    layer, scorer = T.make_softmax_layer(W)
    got, _ = T.check_softmax(layer, scorer, W, x, k, kp)
    assert len(got["cand"]) == c
    x[5, :] = 0
    T.check_softmax(layer, scorer, W, x, k, kp)


def _us_per_step(hire, layer, x_bits, k, kp):
    x, ws = T.dev_bf16(x_bits), hire.alloc_workspace(hire.hire_softmax_workspace_bytes(layer, len(x_bits), k, kp))
    out = hire.SoftmaxOutputs(layer, len(x_bits), k, kp)
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(4):
        start.record()
        for _ in range(4):
            hire.hire_softmax_step(layer, x, k, kp, out, ws)
        stop.record()
        stop.synchronize()
        best = min(best, start.elapsed_time(stop) * 250)
    return best


def test_what_one_token_with_equal_logits_costs(hire):
    """A token of zeros, or one with a thousand equal logits at its k-th place, costs some times the ordinary step at most: its
    shortlist is one workgroup's work, its logits are not, and no round ranks all of them against all (139 times the step)."""
    d, c, B, k, kp = 512, 100000, 64, 64, 1100
    W, x = I.classifier(1320, c, d), I.tokens(1321, B, d)
    layer, _ = T.make_softmax_layer(W)
    plain = _us_per_step(hire, layer, x, k, kp)
    x0 = x.copy()
    x0[7, :] = 0
    zero = _us_per_step(hire, layer, x0, k, kp)
    W[::32] = x[9]  # by far the largest of token 9: 1100 of 3125 equal ones are shortlisted, and others' shares of the rest
    layer, _ = T.make_softmax_layer(W)
    equal = _us_per_step(hire, layer, x, k, kp)
    print(f"plain {plain:.1f} us, a token of zeros {zero:.1f}, equal logits {equal:.1f}", flush=True)
    assert zero < 4 * plain and equal < 8 * plain
