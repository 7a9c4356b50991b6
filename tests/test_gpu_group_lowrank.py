"""Groups of eight with the low-rank scorers on the three-kernel route: one to four tokens (and five, which take the longer
sequence), rows of one and of four waves per trip, an odd number of groups, units that do not fill a workgroup, everything
selected, dense units beside them, a token of zeros, a workspace that the step before has left.  Against the oracle."""
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


@pytest.mark.parametrize("kind", ["lowrank", "lrq"])
@pytest.mark.parametrize("d,N,B,k,kp,r,m1", [
    (64, 72, 1, 8, 16, 32, 0), (96, 1304, 1, 64, 200, 96, 50), (256, 2056, 2, 2056, 2056, 160, 0), (512, 16384, 1, 640, 3200, 64, 0),
    (2048, 2056, 3, 80, 400, 256, 33), (96, 16376, 4, 800, 3200, 32, 100), (544, 552, 5, 40, 160, 544, 7),
    (320, 3000, 4, 160, 600, 320, 0)])
def test_group_lowrank(hire, oracle, kind, d, N, B, k, kp, r, m1):
    print(f"{kind} groups d={d} N={N} B={B} k={k} k'={kp} r={r} m1={m1}", flush=True)
    L = I.lowrank_ffn_layer(1400 + d, d, N, r)
    D = I.ffn_layer(1401, d, max(m1, 1))
    layer, scorer = T.make_ffn_layer(L, lowrank=kind == "lowrank", lrq=kind == "lrq")
    dense = (D["w1u"][:m1], D["w2u"][:m1])
    x_bits = I.tokens(1402 + B, B, d)
    T.check_ffn_commonpath(layer, scorer, L, dense, x_bits, k, kp, 8)
    x_bits[B - 1] = 0
    T.check_ffn_commonpath(layer, scorer, L, dense, x_bits, k, kp, 8)
