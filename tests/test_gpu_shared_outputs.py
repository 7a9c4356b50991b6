"""Groups of eight, few tokens: the workgroups of the second layer's slices write the caller's lists as well, where that
admits slices of half the width (four tokens of d = 2048, eight of d = 1024): lists shorter than the workgroups are many,
ends inside a word, everything selected; rows whose threshold only the range narrowing finds.  Against the oracle; then
without the optional outputs."""
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


@pytest.mark.parametrize("d,N,B,k,kp,m1", [
    (2048, 520, 4, 40, 120, 0), (2048, 8, 4, 8, 8, 33), (1024, 2056, 8, 2056, 2056, 70), (1024, 16384, 8, 640, 3200, 100),
    (2048, 4104, 4, 200, 800, 500)])
def test_shared_outputs(hire, oracle, d, N, B, k, kp, m1):
    print(f"commonpath d={d} N={N} B={B} k={k} k'={kp} m1={m1}", flush=True)
    L = I.ffn_layer(1000 + B, d, N)
    D = I.ffn_layer(1001, d, max(m1, 1))
    layer, scorer = T.make_ffn_layer(L)
    x_bits = I.tokens(1002 + B, B, d)
    dense = (D["w1u"][:m1], D["w2u"][:m1])
    _, want = T.check_ffn_commonpath(layer, scorer, L, dense, x_bits, k, kp, 8)
    dw = [T.dev_bf16(m) if m1 else None for m in dense]
    ws = hire.alloc_workspace(hire.hire_ffn_commonpath_workspace_bytes(layer, m1, B, k, kp, 8))
    out = hire.FFNGroupOutputs(layer, B, k, kp, 8)
    x = T.dev_bf16(x_bits)
    for step in range(2):
        out.y.fill_(float("nan"))
        hire.hire_ffn_commonpath_step(layer, dw[0], dw[1], x, k, kp, 8, out, ws, minimal=True)
        torch.cuda.synchronize()
        T.assert_float_close(out.y.cpu().numpy(), want["y"], "y")


@pytest.mark.parametrize("d,groups,B,k,kp,m1,distinct", [
    (2048, 24, 4, 5, 12, 0, 24), (2048, 1, 4, 1, 1, 0, 1), (2048, 200, 4, 120, 160, 0, 2), (2048, 2048, 4, 300, 900, 40, 3),
    (1024, 70, 8, 30, 66, 40, 1), (1024, 33, 8, 32, 33, 7, 33)])
def test_thresholds_among_zeros_and_equal_groups(hire, oracle, d, groups, B, k, kp, m1, distinct):
    """The first token is zero: its threshold lies among the zeros.  Groups that repeat put more than 64 equal activations
    around the other tokens' thresholds.  Few groups leave most waves without keys: nothing that the narrowing shares
    between the waves may be written again before all of them have read it."""
    print(f"narrowing d={d} groups={groups} B={B} k={k} k'={kp} m1={m1} distinct={distinct}", flush=True)
    L = I.ffn_layer(1010 + distinct, d, 8 * groups)
    rows = (np.arange(groups) % distinct)[:, None] * 8 + np.arange(8)
    L["w1u"] = np.ascontiguousarray(L["w1u"][rows.ravel()])
    D = I.ffn_layer(1011, d, max(m1, 1))
    layer, scorer = T.make_ffn_layer(L)
    x_bits = I.tokens(1012 + B, B, d)
    x_bits[0] = 0
    T.check_ffn_commonpath(layer, scorer, L, (D["w1u"][:m1], D["w2u"][:m1]), x_bits, 8 * k, 8 * kp, 8)
