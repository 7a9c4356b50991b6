"""The sharded step's sequence for batches: one and many shards, shards that begin and end inside a word of the union's
bitmap, the widths that a wave's registers are cut for (64, 128, 256 and 1024 units), tiles of sixteen tokens and one more, rows of
the second layer's edges, ties and zeros.  Against the oracle; then without the optional outputs."""
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


@pytest.mark.parametrize("d,N,B,k,kp,s", [
    (64, 1024, 8, 100, 300, 1), (32, 257 * 3, 16, 50, 160, 3), (96, 65 * 7, 17, 35, 140, 7), (128, 63 * 16, 33, 40, 200, 16),
    (64, 300, 64, 100, 150, 300), (256, 129 * 5, 9, 640, 645, 5), (8192, 128 * 4, 8, 51, 160, 4), (2080, 192, 32, 9, 30, 3),
    (32, 1000 * 33, 10, 900, 3000, 33), (512, 1024, 64, 1024, 1024, 4)])
def test_shard_batches(hire, oracle, d, N, B, k, kp, s):
    print(f"shards d={d} N={N} B={B} k={k} k'={kp} s={s}", flush=True)
    L = I.ffn_layer(1100 + B, d, N)
    L["w1u"][N // 4:N // 4 + 20] = L["w1u"][N // 4]  # equal keys and equal activations
    layer, scorer = T.make_ffn_layer(L)
    x_bits = I.tokens(1101 + B, B, d)
    x_bits[B // 2] = 0
    x_bits[B - 1] = x_bits[0]
    got, want = T.check_ffn_shard(layer, scorer, L, x_bits, k, kp, s)
    assert not got["y"][B // 2].any() and np.array_equal(got["y"][0], got["y"][B - 1])
    ws = hire.alloc_workspace(hire.hire_ffn_shard_workspace_bytes(layer, B, k, kp, s))
    out = hire.FFNShardOutputs(layer, B, k, kp, s)
    x = T.dev_bf16(x_bits)
    for step in range(2):
        out.y.fill_(float("nan"))
        hire.hire_ffn_shard_step(layer, x, k, kp, s, out, ws, minimal=True)
        torch.cuda.synchronize()
        T.assert_float_close(out.y.cpu().numpy(), want["y"], "y")
