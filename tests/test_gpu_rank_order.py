"""Selections in rank order: up to two waves of entries by comparison, more by bins of their keys, or sorted where many are in one
bin.  Sizes at both sides of every round of threads; rows of distinct values, of a few values (long runs of equal keys in one
bin), and with one far outlier (all other keys share the last bins); infinities, NaN and both zeros; what equal values cost."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _order_keys(v):
    """Unsigned keys that rank like the selection: -0 as +0, NaN by its bits."""
    u = np.where(v == 0.0, np.float32(0.0), v).astype(np.float32).view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint32)


@pytest.mark.parametrize("N,k", [(1, 1), (65, 64), (65, 65), (1000, 63), (1000, 512), (1025, 1024), (1025, 1025), (5000, 66),
                                 (9000, 4096), (30001, 2049), (32769, 2048), (40000, 1025), (70001, 64)])
def test_rank_order_of_all_kinds_of_rows(N, k):
    from paper_2402_09360_amd import hire
    assert torch.cuda.is_available(), "these tests need the MI355X"
    rng = np.random.default_rng(977 + N + k)
    v = rng.standard_normal((4, N)).astype(np.float32)
    v[1] = rng.integers(0, 3, N).astype(np.float32)
    v[2, N // 2] = np.float32(1e30)
    for bits in (0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000, 0x80000000, 0x00000001):
        v[3].view(np.uint32)[rng.integers(0, N, max(1, N // 50))] = np.uint32(bits)
    keys = _order_keys(v)
    want = np.lexsort((np.broadcast_to(np.arange(N), v.shape), ~keys), axis=1)[:, :k]
    print(f"rank order N={N} k={k}", flush=True)
    idx, val = hire.topk_select(torch.from_numpy(v).cuda(), k, rank_order=True)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(_order_keys(val.cpu().numpy()), np.take_along_axis(keys, want, axis=1))


@pytest.mark.parametrize("run", [47, 48, 49, 64, 130])
@pytest.mark.parametrize("N,k", [(1000, 128), (1000, 129), (1000, 513), (3000, 2047), (40000, 1500), (40000, 2048)])
def test_runs_of_equal_values(N, k, run):
    """Every value `run` times, at random places; a row of values a unit in the last place apart (all in one bin or two) beside
    an outlier."""
    from paper_2402_09360_amd import hire
    rng = np.random.default_rng(1000 * run + N + k)
    v = rng.permuted(np.tile((np.arange(N) // run).astype(np.float32), (3, 1)), axis=1)
    v[1] = (np.uint32(0x3F800000) + rng.permutation(N).astype(np.uint32)).view(np.float32)
    v[1, N // 3] = np.float32(3e38)
    v[2] = 0.25
    keys = _order_keys(v)
    want = np.lexsort((np.broadcast_to(np.arange(N), v.shape), ~keys), axis=1)[:, :k]
    print(f"runs of {run} N={N} k={k}", flush=True)
    idx, val = hire.topk_select(torch.from_numpy(v).cuda(), k, rank_order=True)
    assert np.array_equal(idx.cpu().numpy(), want)
    assert np.array_equal(_order_keys(val.cpu().numpy()), np.take_along_axis(keys, want, axis=1))


@pytest.mark.parametrize("B,k", [(2, 128), (2, 129), (2, 300), (1, 1000)])
def test_equal_logits(oracle, B, k):
    """The same for logits in 64 bits: a token of zeros, whose logits are all equal, and long runs of equal classes."""
    import hire_testlib as T
    from paper_2402_09360_amd import inputs as I
    W = I.classifier(1600, 40000, 64)
    W[::40] = W[0]
    layer, scorer = T.make_softmax_layer(W)
    x = I.tokens(1601, B, 64)
    x[0, :] = W[0]
    T.check_softmax(layer, scorer, W, x, k, 1200)
    x[-1, :] = 0
    T.check_softmax(layer, scorer, W, x, k, 1200)


@pytest.mark.parametrize("N,k", [(1000, 100), (1000, 256), (1000, 512), (16384, 512)])
def test_what_equal_values_cost(N, k):
    """Ranking equal values takes no more than every entry's comparison with every other: 100 of them were 2.1 times the distinct
    ones' time, 256 3.8 times, 512 4.9 times, of 16384 4.3 times."""
    from paper_2402_09360_amd import hire
    ws = hire.alloc_workspace(max(256, hire.hire_topk_workspace_bytes(16, N, k, hire.ORDER_RANK)))
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def us(v):
        best = float("inf")
        for _ in range(6):
            start.record()
            for _ in range(50):
                hire.topk_select(v, k, rank_order=True, workspace=ws)
            stop.record()
            stop.synchronize()
            best = min(best, start.elapsed_time(stop) * 20)
        return best

    distinct, equal = us(torch.randn((16, N), device="cuda")), us(torch.ones((16, N), device="cuda"))
    print(f"N={N} k={k}: distinct {distinct:.1f} us, equal {equal:.1f}", flush=True)
    assert equal < (1.6 if k < 256 else 2.6) * distinct
