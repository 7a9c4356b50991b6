"""Selections in rank order: up to a wave of entries by comparison, more by bins of their keys.  Sizes at both sides of every
round of threads; rows of distinct values, of a few values (long runs of equal keys in one bin), and with one far outlier (all
other keys share the last bins); infinities, NaN and both zeros."""
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
