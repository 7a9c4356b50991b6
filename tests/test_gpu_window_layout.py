"""Steps of one token and of several keep their window histograms in different orders of the slots: on one workspace in
turn, neither may find counts where the other left them, and the selections go by the histograms throughout."""
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N", [(64, 1000), (256, 16384)])
def test_one_and_several_tokens_in_turn(oracle, d, N):
    from paper_2402_09360_amd import hire
    assert torch.cuda.is_available(), "these tests need the MI355X"
    k, kp = N // 20, N // 5
    L = I.ffn_layer(701, d, N)
    layer, scorer = T.make_ffn_layer(L)
    ws = hire.alloc_workspace(max(hire.hire_ffn_workspace_bytes(layer, B, k, kp) for B in (1, 2, 3, 4)))
    T.run_ffn(layer, I.tokens(702, 4, d), k, kp, ws=ws)  # stamps the four regions
    before = hire.hire_debug_fast_fallbacks(ws)
    for turn, B in enumerate((1, 4, 1, 3, 2, 4, 1)):
        print(f"d={d} N={N} turn {turn}: B={B}", flush=True)
        x = I.tokens(703 + turn, B, d)
        want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
        for got in T.run_ffn(layer, x, k, kp, ws=ws, steps=2):
            T.compare_ffn(got, want)
        assert hire.hire_debug_fast_state(ws)[:2] == (1, 0)
    assert hire.hire_debug_fast_fallbacks(ws) == before
