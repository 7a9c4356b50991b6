"""The filter stage of long rows, whose workgroups start in different stages of a row where the rows are whole multiples of 4 KB
apart: more workgroups of a die than a row has stages, a last workgroup with few candidates; and rows of other lengths, which
end inside a stage.  |stored - <u, x>| <= err_c |u| |x|, the stage's
proven bound."""
import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rows,B", [(2048, 1100, 16), (2080, 2113, 9), (2176, 8 * 64 * 3, 17), (4104, 700, 32), (2040, 1100, 16),
                                      (2080, 2113, 33), (2048, 8 * 64 * 17 + 50, 9), (2048, 8 * 64 * 17 + 50, 32),
                                      (4096, 2113, 16), (4096, 8 * 64 * 3 + 49, 24)])
def test_stages_in_turn(d, rows, B):
    from paper_2402_09360_amd import hire
    assert torch.cuda.is_available(), "these tests need the MI355X"
    Wb, xb = I.normal_bf16(721 + d, (rows, d)), I.tokens(722 + d, B, d)
    print(f"filter stage d={d} rows={rows} B={B}", flush=True)
    stored, xnorm, wmax, err_c = hire.hire_debug_filter_stage(T.dev_bf16(Wb), T.dev_bf16(xb))
    stored = stored.cpu().numpy().astype(np.float64)
    W, x = I.bf16_bits_to_f64(Wb), I.bf16_bits_to_f64(xb)
    h = x @ W.T
    un, xn = np.sqrt((W * W).sum(axis=1)), np.sqrt((x * x).sum(axis=1))
    delta = err_c * xn[:, None] * un[None, :]
    kept = stored > np.float64(np.float32(1e-45))
    assert (np.abs(stored - h)[kept] <= delta[kept] / 8).all()   # (8: the slack that the shorter rows' test asks for)
    assert (h[~kept] <= delta[~kept] / 8).all()
    assert un.max() <= wmax <= 1.01 * un.max()
    xg = xnorm.cpu().numpy().astype(np.float64)
    assert (xg >= xn).all() and (xg <= 1.01 * xn).all()


@pytest.mark.parametrize("d,rows,B", [(2048, 8 * 64 * 16, 16), (2048, 8 * 64 * 16, 32), (2080, 8 * 64 * 17, 9)])
def test_token_norms_come_from_one_order(d, rows, B):
    """The selection's band goes by the tokens' norms: whatever stage the workgroups start in, they are bit for bit those
    of the first 64 rows by themselves."""
    from paper_2402_09360_amd import hire
    W, x = T.dev_bf16(I.normal_bf16(731 + d, (rows, d))), T.dev_bf16(I.tokens(732 + d, B, d))
    print(f"token norms d={d} rows={rows} B={B}", flush=True)
    alone = hire.hire_debug_filter_stage(W[:64].contiguous(), x)[1]
    for _ in range(8):
        assert torch.equal(hire.hire_debug_filter_stage(W, x)[1], alone)


@pytest.mark.parametrize("kind", ["int4", "lowrank"])
@pytest.mark.parametrize("B", [16, 32])
def test_steps_repeat_bit_for_bit(B, kind):
    d, N, k, kp = 2048, 16384, 819, 3276
    L = I.ffn_layer(741, d, N) if kind == "int4" else I.lowrank_ffn_layer(742, d, N, 32)
    layer, _ = T.make_ffn_layer(L, lowrank=kind == "lowrank")
    print(f"repeated steps B={B} {kind}", flush=True)
    first, *more = T.run_ffn(layer, I.tokens(743, B, d), k, kp, steps=6, debug=False)
    for got in more:
        for name in ("y", "topk_idx", "topk_val", "cand"):
            assert np.array_equal(got[name], first[name]), name


@pytest.mark.parametrize("d,B", [(2048, 16), (2080, 24)])  # the others start in all of the stages; rows that end inside one
def test_first_units_outside_the_union(oracle, d, B):
    """The workgroup that stores the tokens' norms has no candidates."""
    N = 16384
    L = dict(I.ffn_layer(751, d, N))
    L["w1u"] = L["w1u"].copy()
    L["w1u"][:64] = 0x2000  # tiny weights, no token's pick
    layer, scorer = T.make_ffn_layer(L)
    print(f"first units outside the union, d={d} B={B}", flush=True)
    got, _ = T.check_ffn(layer, scorer, L, I.tokens(752, B, d), 819, 3276)
    assert got["cand"].min() >= 64
