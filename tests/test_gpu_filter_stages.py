"""The filter stage of long rows, whose workgroups start in different stages of a row: rows that end inside a stage, more
workgroups than a die has stages, a last workgroup with few candidates.  |stored - <u, x>| <= err_c |u| |x|, the stage's
proven bound."""
import numpy as np
import pytest
import torch

import hire_testlib as T
from paper_2402_09360_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rows,B", [(2048, 1100, 16), (2080, 2113, 9), (2176, 8 * 64 * 3, 17), (4104, 700, 32), (2040, 1100, 16),
                                      (2080, 2113, 33)])
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
