"""The refining selection with the second layer in one kernel (16 tokens and more whose selected rows are few enough) and with its
values rounded from 64 bits, against the oracle: slices of 64 to 512 columns with a remainder, lists that end inside, at and behind a batch of rows, the shared-out list
of the candidates, tokens that the list in LDS does not settle; and infinite second-layer weights."""
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


@pytest.mark.parametrize("d,N,B,k,kp", [
    (32, 1026, 16, 1, 80),         # less than a slice, one entry
    (96, 1090, 16, 128, 300),      # 64 columns: a slice and a half, a batch of rows and no more
    (96, 1090, 17, 129, 300),
    (1056, 2000, 16, 257, 400),    # 128 columns, the last slice of 32
    (544, 3002, 64, 200, 600),     # 256 columns
    (1088, 2048, 64, 513, 700),    # 512 columns
    (64, 16384, 16, 4096, 4096),   # the longest list; all of it selected
    (64, 16382, 33, 700, 1000),    # the last word of the bitmap is not whole
    (8192, 1100, 16, 60, 200),     # the longest token in LDS
    (8224, 1100, 16, 60, 200),     # longer
])
def test_against_the_oracle(hire, oracle, d, N, B, k, kp):
    print(f"ffn_step d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1200 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1201 + B, B, d)
    x[1, :] = 0                                    # threshold among the zeros
    x[3:6, :] = x[2, :]
    T.check_ffn(layer, scorer, L, x, k, kp)


@pytest.mark.parametrize("d,N,B,k,kp", [
    (64, 777, 5, 3, 9),            # a workgroup per token, fewer entries than waves
    (96, 1091, 8, 512, 600),       # a round of workgroups, none left for the candidates' list: all of them share it
    (800, 2003, 16, 250, 400),     # 256 workgroups again
    (2080, 1501, 7, 33, 200),      # rows of more than one request of a wave
    (64, 16390, 6, 300, 1500),     # more units than 16384
    (8224, 1000, 5, 20, 100),      # a token that is not in LDS
    (64, 2001, 33, 336, 800), (64, 2001, 33, 337, 800),  # three rows per wave, and a wave with four: the kernel behind the list
    (64, 2001, 63, 192, 800), (64, 2001, 63, 193, 800),
])
def test_values_from_64_bits_against_the_oracle(hire, oracle, d, N, B, k, kp):
    print(f"ffn_step d={d} N={N} B={B} k={k} k'={kp}", flush=True)
    L = I.ffn_layer(1220 + d, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1221 + B, B, d)
    x[1, :] = 0
    got, want = T.check_ffn(layer, scorer, L, x, k, kp)
    # one rounding of a 64-bit sum: half an ulp, and the difference between two orders of the sum
    assert (np.abs(got["topk_val"].astype(np.float64) - want["topk_val"]) <= np.abs(want["topk_val"]) * (0.5 + 1e-3) * 2.0 ** -23).all()


@pytest.mark.parametrize("d,B,rows", [(256, 16, 128), (1024, 8, 64), (1024, 30, 32), (1024, 64, 16)])  # rows per load of a workgroup
def test_lists_of_every_number_of_loads(hire, oracle, d, B, rows):
    """The second layer by itself, slices of 32 to 256 columns: one, two, four, eight loads per lane, and more; whole and not."""
    N = 1101  # (odd: the values are rounded from 64 bits, by a kernel without the second layer)
    L = I.ffn_layer(1250 + B, d, N)
    layer, scorer = T.make_ffn_layer(L)
    x = I.tokens(1251 + B, B, d)
    for loads in (1, 2, 4, 8):
        for k in (loads * rows - 1, loads * rows, loads * rows + 1):
            print(f"d={d} B={B} k={k}", flush=True)
            T.check_ffn(layer, scorer, L, x, k, N)


def _infinite(y, plus, minus):
    assert (y[:, plus] == np.inf).all() and (y[:, minus] == -np.inf).all()
    assert np.isfinite(np.delete(y, [plus, minus], axis=1)).all()


def _largest_everywhere(seed, d, N, B, at):
    """A layer and B equal tokens whose largest activations are the units `at`; infinite in one column each."""
    L = I.ffn_layer(seed, d, N)
    x = np.repeat(I.tokens(seed + 1, 1, d), B, axis=0)
    L["w1u"][at, :] = x[0, :]
    L["w2u"][at[0], 5] = 0x7F80
    L["w2u"][at[-1], 200] = 0xFF80
    return L, x


# one to eight tokens; the kernel with the second layer in it; the second layer by itself (1024 units; 96 MB of rows)
@pytest.mark.parametrize("N,B,k,kp", [(2050, 16, 100, 300), (2050, 1, 100, 300), (2050, 1, 1, 2), (2050, 4, 100, 300), (2050, 4, 127, 300),
                                      (2050, 8, 33, 300), (1024, 16, 52, 208), (1024, 16, 64, 208), (16384, 64, 3100, 4000)])
@pytest.mark.parametrize("generic", [False, True])
def test_infinite_weights_stay_in_their_columns(hire, oracle, N, B, k, kp, generic):
    """Rows that are selected for every token, the first and the last of its list, are infinite in one column each."""
    print(f"infinite weights N={N} B={B} k={k} k'={kp} generic={generic}", flush=True)
    L, x = _largest_everywhere(1210, 256, N, B, [0, N - 1] if k > 1 else [N - 1])
    if k == 1:
        L["w2u"][0, 5] = L["w2u"][N - 1, 200]
    layer, _ = T.make_ffn_layer(L)
    hire.hire_force_generic_path(generic)
    try:
        for r in T.run_ffn(layer, x, k, kp, steps=2):
            _infinite(r["y"], 5, 200)
    finally:
        hire.hire_force_generic_path(False)


@pytest.mark.parametrize("B", [1, 4, 8, 16])
@pytest.mark.parametrize("k,kp,m1", [(104, 304, 0), (8, 16, 3), (104, 304, 300)])
def test_infinite_weights_of_groups_and_dense_units(hire, oracle, B, k, kp, m1):
    """The same for the last unit of the last selected group, and for the last of the dense units."""
    print(f"infinite weights, groups, B={B} k={k} k'={kp} m1={m1}", flush=True)
    d, N = 256, 2048
    L, x = _largest_everywhere(1220, d, N, B, [N - 8, N - 1])
    layer, _ = T.make_ffn_layer(L)
    dense = None, None
    if m1:
        D = I.ffn_layer(1230, d, m1)
        D["w1u"][m1 - 1, :] = x[0, :]
        D["w2u"][m1 - 1, 5] = 0x7F80
        dense = T.dev_bf16(D["w1u"]), T.dev_bf16(D["w2u"])
    out = hire.FFNGroupOutputs(layer, B, k, kp, 8)
    ws = hire.alloc_workspace(hire.hire_ffn_commonpath_workspace_bytes(layer, m1, B, k, kp, 8))
    for _ in range(2):
        hire.hire_ffn_commonpath_step(layer, *dense, T.dev_bf16(x), k, kp, 8, out, ws)
        _infinite(out.y.cpu().numpy(), 5, 200)


@pytest.mark.parametrize("shards,B,k,kp", [(16, 1, 80, 320), (16, 4, 48, 320), (16, 16, 48, 320), (8, 4, 600, 900), (8, 4, 66, 300)])
def test_infinite_weights_of_shards(hire, oracle, shards, B, k, kp):
    """The same for the first and last units of a layer in shards, whose lists do not come in fours."""
    print(f"infinite weights, shards={shards} B={B} k={k} k'={kp}", flush=True)
    N = 2048
    L, x = _largest_everywhere(1240, 256, N, B, [0, N - 1])
    layer, _ = T.make_ffn_layer(L)
    for r in T.run_ffn_shard(layer, x, k, kp, shards, steps=2):
        _infinite(r["y"], 5, 200)
