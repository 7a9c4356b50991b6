"""Steps on workspaces and layers that are not as the step before would have left them: a step that the runtime refused
half-way, row-norm bounds and row scales that do not fit the layer.  The window histograms that guide the selections of
one to eight tokens live in the workspace and are placed by bounds of the keys: neither may decide what is selected, only
how fast.  Integers bit for bit, floats to the parity tests' bar."""
import ctypes as C

import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu

ELAUNCH = -4


@pytest.fixture(scope="module")
def hire():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2402_09360_amd import hire as H
    return H


def log(msg):
    print(msg, flush=True)


def _end_after(hire, kernels, step):
    """Runs the step with an event array that makes it end behind its first `kernels` stages: the event that is recorded
    there does not exist, which the runtime refuses on the host.  What was enqueued before runs to its end."""
    from paper_2402_09360_amd.hiprt import Events, hip
    ev = Events(hire.NUM_STAGE_EVENTS)
    holes = (C.c_void_p * hire.NUM_STAGE_EVENTS)()
    for i in range(kernels):
        holes[i] = ev.array[i]
    hire.hire_set_stage_events(holes)
    try:
        with pytest.raises(hire.HireError) as e:
            step()
        assert e.value.code == ELAUNCH
    finally:
        hire.hire_set_stage_events(None)
        hip().hipGetLastError()
    torch.cuda.synchronize()


@pytest.mark.parametrize("route,B", [("int4", 1), ("int4", 3), ("lowrank", 1), ("lowrank", 4), ("lrq", 1), ("lrq", 2),
                                     ("groups", 1), ("groups", 8)])
def test_step_after_one_that_ended_half_way(hire, oracle, route, B):
    """The kernels that ran have counted keys which nobody has cleared: the next step must not take them for its own."""
    d, N, k, kp = 256, 1504, 64, 304
    L = I.ffn_layer(301, d, N) if route in ("int4", "groups") else I.lowrank_ffn_layer(302, d, N, 64)
    layer, scorer = T.make_ffn_layer(L, lowrank=route == "lowrank", lrq=route == "lrq")
    groups = route == "groups"
    ws = hire.alloc_workspace(hire.hire_ffn_group_workspace_bytes(layer, B, k, kp, 8) if groups else
                              hire.hire_ffn_workspace_bytes(layer, B, k, kp))

    def step(x, steps=1):
        if groups:
            return T.run_ffn_group(layer, x, k, kp, 8, ws=ws, steps=steps, debug=False)
        return T.run_ffn(layer, x, k, kp, ws=ws, steps=steps, debug=False)

    step(I.tokens(303, B, d), steps=2)                       # the workspace's steady state
    assert hire.hire_debug_fast_state(ws)[0] == 1
    for kernels in (1, 2):
        log(f"{route} B={B}: ends after {kernels} of its stages")
        _end_after(hire, kernels, lambda: step(I.tokens(304, B, d)))
        assert hire.hire_debug_fast_state(ws)[0] == 0        # no marker: the counts in the workspace are nobody's
        x = I.tokens(305 + kernels, B, d)
        if groups:
            want = oracle.ffn_group_step(L["w1u"], L["w2u"], scorer, x, k, kp, 8)
        else:
            want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
        for got in step(x, steps=3):
            assert np.array_equal(got["cand"], want["cand"])
            name = "topk_group" if groups else "topk_idx"
            assert np.array_equal(got[name], want[name])
            T.assert_float_close(got["topk_val"], want["topk_val"], "topk_val")
            T.assert_float_close(got["y"], want["y"], "y")
        assert hire.hire_debug_fast_state(ws)[:2] == (1, 0)


@pytest.mark.parametrize("kind", ["lowrank", "lrq"])
@pytest.mark.parametrize("B", [1, 3])
def test_row_norm_bounds_only_place_the_histograms(hire, oracle, kind, B):
    """Bounds of another layer: from a little too small, so that a few of the keys lie above the window, to useless."""
    d, N, r, k, kp = 256, 1200, 32, 50, 200
    L = I.lowrank_ffn_layer(311, d, N, r)
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank", lrq=kind == "lrq")
    right = layer.row_norm_bounds.clone()
    x = I.tokens(312, B, d)
    want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
    slow = 0
    for factor in (1.0, 0.5, 0.3, 0.2, 0.1, 2.0 ** -6, 2.0 ** -20, 0.0, 2.0 ** 20):
        layer.row_norm_bounds.copy_(right * factor)
        torch.cuda.synchronize()
        ws = hire.alloc_workspace(hire.hire_ffn_workspace_bytes(layer, B, k, kp))
        for got in T.run_ffn(layer, x, k, kp, steps=3, ws=ws):
            assert np.array_equal(got["cand"], want["cand"]), factor
            assert np.array_equal(got["topk_idx"], want["topk_idx"]), factor
            T.assert_float_close(got["topk_val"], want["topk_val"], "topk_val")
            T.assert_float_close(got["y"], want["y"], "y")
        keys, activations = hire.hire_debug_fast_fallbacks(ws)
        log(f"{kind} B={B} bounds times {factor}: selections without a histogram {keys}, {activations}")
        slow += keys + activations
    assert slow > 0


@pytest.mark.parametrize("B", [1, 4, 8, 20])
def test_row_scales_above_the_packed_maximum(hire, oracle, B):
    """The codes carry the largest row scale, which bounds the keys; row scales that are larger than that put keys above
    the bound.  They are ranked as what they are."""
    d, N, k, kp = 128, 2000, 60, 400
    L = I.ffn_layer(321, d, N)
    layer, (kind, q, s) = T.make_ffn_layer(L)
    factor = np.ones(N, dtype=np.float32)
    factor[5::37] = 8.0
    layer.q4_scale.mul_(torch.from_numpy(factor).cuda())
    torch.cuda.synchronize()
    log(f"row scales above the maximum, B={B}")
    T.check_ffn(layer, (kind, q, s * factor), L, I.tokens(322 + B, B, d), k, kp)


@pytest.mark.parametrize("d,N,B,k,kp", [(512, 16384, 32, 81, 327), (256, 30000, 16, 163, 655), (64, 9000, 64, 3, 18)])
def test_static_scratch_takes_large_batches_with_small_unions(hire, oracle, d, N, B, k, kp):
    """Steps whose buffers are sized by their unions, next to one of few tokens whose state lies where theirs do."""
    L = I.ffn_layer(341, d, N)
    layer, scorer = T.make_ffn_layer(L)
    small = I.ffn_layer(342, 128, 700)
    small_layer, small_scorer = T.make_ffn_layer(small)

    def static(layer, x_bits, k, kp):
        x = T.dev_bf16(x_bits)
        out = hire.FFNOutputs(layer, x.shape[0], k, kp)
        hire.hire_ffn_step_static(layer, x, k, kp, out)
        torch.cuda.synchronize()
        n = int(out.n_cand.item())
        return dict(y=out.y.cpu().numpy(), topk_idx=out.topk_idx.cpu().numpy(), topk_val=out.topk_val.cpu().numpy(),
                    cand=out.cand_idx.cpu().numpy()[:n], n_cand=n, acc=None)

    x, xs = I.tokens(343, B, d), I.tokens(344, 3, 128)
    want = oracle.ffn_step(L["w1u"], L["w2u"], scorer, x, k, kp)
    want_small = oracle.ffn_step(small["w1u"], small["w2u"], small_scorer, xs, 30, 150)
    for turn in range(3):
        log(f"static scratch, turn {turn}: B={B} N={N} k'={kp}, then 3 tokens twice")
        T.compare_ffn(static(layer, x, k, kp), want)
        for _ in range(2):
            T.compare_ffn(static(small_layer, xs, 30, 150), want_small)


@pytest.mark.parametrize("B,stages", [(1, 2), (2, 3)])
def test_long_rows_after_a_step_that_ended_half_way(hire, oracle, B, stages):
    """The general sequence on rows beyond 32768 keeps key histograms in the workspace: counted by the scorer (one token)
    or by a pass of the selection (two), restored by the kernel that resolves the threshold bin, which does not run here."""
    d, c, k, kp = 256, 40000, 16, 400
    W = I.classifier(345, c, d)
    layer, scorer = T.make_softmax_layer(W)
    ws = hire.alloc_workspace(hire.hire_softmax_workspace_bytes(layer, B, k, kp))
    hire.hire_force_generic_path(True)
    try:
        T.run_softmax(layer, I.tokens(346, B, d), k, kp, ws=ws, steps=3)
        assert hire.hire_debug_general_fallbacks(ws) == (0, 0, 1)
        log(f"long rows B={B}: ends after {stages} stages")
        _end_after(hire, stages, lambda: T.run_softmax(layer, I.tokens(347, B, d), k, kp, ws=ws))
        x = I.tokens(348, B, d)
        want = oracle.softmax_step(W, scorer, x, k, kp, want_acc=True)
        for got in T.run_softmax(layer, x, k, kp, ws=ws, steps=3):
            T.compare_softmax(got, want)
        assert hire.hire_debug_general_fallbacks(ws) == (0, 0, 2)     # cleared and stamped once more
    finally:
        hire.hire_force_generic_path(False)
    for got in T.run_softmax(layer, x, k, kp, ws=ws, steps=2):        # the sequence from the scorer's maxima
        T.compare_softmax(got, want)
    hire.hire_force_generic_path(True)
    try:
        for got in T.run_softmax(layer, x, k, kp, ws=ws, steps=2):    # and the histograms behind it
            T.compare_softmax(got, want)
    finally:
        hire.hire_force_generic_path(False)
