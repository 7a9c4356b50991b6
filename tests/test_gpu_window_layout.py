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


@pytest.mark.parametrize("B,group,distinct", [(2, 1, 3), (4, 1, 1), (4, 1, 40), (3, 8, 2), (8, 8, 1), (8, 8, 30)])
def test_many_units_in_the_threshold_bins(oracle, B, group, distinct):
    """Rows that repeat: whole workgroups' units share the threshold bins of several tokens, up to every unit of all of them,
    and the lower index decides.  The thresholds are found in the windows throughout; the second selection's bins may hold more
    than its list."""
    import numpy as np
    from paper_2402_09360_amd import hire
    assert torch.cuda.is_available(), "these tests need the MI355X"
    d, N, k, kp = 256, 1504, 64, 304
    L = dict(I.ffn_layer(711, d, N))
    rows = np.random.default_rng(712 + distinct).integers(0, distinct, N // group).repeat(group)
    L["w1u"] = np.ascontiguousarray((L["w1u"] & 0x7FFF)[rows])  # keys of one sign
    x = I.tokens(713, B, d) & 0x7FFF
    print(f"{distinct} distinct rows, B={B}, groups of {group}", flush=True)
    layer, scorer = T.make_ffn_layer(L)
    if group == 1:
        want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
        ws = hire.alloc_workspace(hire.hire_ffn_workspace_bytes(layer, B, k, kp))
        for got in T.run_ffn(layer, x, k, kp, steps=3, debug=False, ws=ws):
            T.compare_ffn(got, dict(want, acc=None))
        assert hire.hire_debug_fast_fallbacks(ws)[0] == 0
        return
    want = oracle.ffn_group_step(L["w1u"], L["w2u"], scorer, x, k, kp, group)
    ws = hire.alloc_workspace(hire.hire_ffn_group_workspace_bytes(layer, B, k, kp, group))
    results = T.run_ffn_group(layer, x, k, kp, group, steps=3, debug=False, ws=ws)
    assert hire.hire_debug_fast_fallbacks(ws)[0] == 0
    for got in results:
        assert np.array_equal(got["cand"], want["cand"]) and np.array_equal(got["topk_group"], want["topk_group"])
        T.assert_float_close(got["topk_val"], want["topk_val"], "topk_val")
        T.assert_float_close(got["y"], want["y"], "y")


@pytest.mark.parametrize("d,N,kp,kind", [(96, 1030, 1030, "int4"), (2080, 700, 350, "int4"), (256, 1000, 300, "lowrank"),
                                         (256, 4100, 2050, "lrq")])
def test_one_token_many_rows_per_workgroup(oracle, d, N, kp, kind):
    """One token whose workgroups have up to all of their 64 units to read: one to four rows per wave."""
    assert torch.cuda.is_available(), "these tests need the MI355X"
    k = kp // 3
    L = I.ffn_layer(741, d, N) if kind == "int4" else I.lowrank_ffn_layer(742, d, N, 32)
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank", lrq=kind == "lrq")
    print(f"one token, d={d} N={N} k'={kp} {kind}", flush=True)
    x = I.tokens(743, 1, d)
    want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
    for got in T.run_ffn(layer, x, k, kp, steps=3, debug=False):
        T.compare_ffn(got, dict(want, acc=None))


@pytest.mark.parametrize("d,N,kp,kind", [(96, 1032, 1032, "int4"), (2080, 704, 352, "int4"), (256, 1000, 1000, "lowrank"),
                                         (256, 4104, 2056, "lowrank")])
def test_one_token_many_groups_per_workgroup(oracle, d, N, kp, kind):
    """The same with groups of eight, whose waves have their rows one at a time: up to four trips."""
    assert torch.cuda.is_available(), "these tests need the MI355X"
    L = I.ffn_layer(761, d, N) if kind == "int4" else I.lowrank_ffn_layer(762, d, N, 32)
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank")
    print(f"one token, groups, d={d} N={N} k'={kp} {kind}", flush=True)
    T.check_ffn_group(layer, scorer, L, I.tokens(763, 1, d), kp // 16 * 8, kp, 8)


@pytest.mark.parametrize("B,d", [(1, 64), (4, 2048), (4, 4096)])  # sixteen, eight and four rows per load
def test_few_tokens_rows_per_wave_of_the_second_layer(oracle, B, d):
    """All units selected, all of them one wave's: one to eight loads, whole and not, and more than one trip."""
    assert torch.cuda.is_available(), "these tests need the MI355X"
    for N in (1, 15, 24, 28, 40, 45, 50, 61, 65, 81, 100, 113, 128, 129, 250):
        print(f"B={B} d={d} N={N}", flush=True)
        L = dict(I.ffn_layer(781 + N, d, N))
        L["w1u"] = L["w1u"] & 0x7FFF  # no activation is zero
        layer, scorer = T.make_ffn_layer(L)
        T.check_ffn(layer, scorer, L, I.tokens(782, B, d) & 0x7FFF, N, N)


@pytest.mark.parametrize("m1", [1, 300, 700, 900, 1100, 1500, 1700, 2040, 2100])
def test_one_token_dense_rows_per_wave_of_the_second_layer(oracle, m1):
    """One to eight loads of dense rows per wave, and a second trip."""
    assert torch.cuda.is_available(), "these tests need the MI355X"
    print(f"m1={m1}", flush=True)
    d, N = 64, 512
    L, D = I.ffn_layer(791, d, N), I.ffn_layer(792, d, m1)
    layer, scorer = T.make_ffn_layer(L)
    T.check_ffn_commonpath(layer, scorer, L, (D["w1u"], D["w2u"]), I.tokens(793, 1, d), 64, 128, 8)
