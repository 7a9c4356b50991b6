"""The bare selection on long rows, whose lists' lengths lie in the place of the longer sequence's bitmaps.  Values that a
comparison of floats does not order (NaN), equal ones in their hundreds, masks of the lowest value, rows that end inside a
workgroup's part, one row and many; then the longer sequence on the same workspace."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _order_keys(v):
    """Unsigned keys that rank like the selection: -0 as +0, NaN by its bits."""
    u = np.where(v == 0.0, np.float32(0.0), v).astype(np.float32).view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000)).astype(np.uint32)


@pytest.mark.parametrize("B,N,k,relu", [(1, 32769, 1, False), (3, 49157, 2048, False), (3, 49157, 700, True), (64, 33000, 65, False),
                                        (2, 262145, 2000, True)])
def test_long_rows_with_values_of_all_kinds(B, N, k, relu):
    from paper_2402_09360_amd import hire
    assert torch.cuda.is_available(), "these tests need the MI355X"
    rng = np.random.default_rng(731 + N + k)
    v = rng.standard_normal((B, N)).astype(np.float32)
    v[:, rng.integers(0, N, N // 3)] = np.finfo(np.float32).min
    v[:, rng.integers(0, N, 300)] = np.float32(2.5)
    for bits in (0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000, 0x80000000, 0x00000001):
        v.view(np.uint32)[:, rng.integers(0, N, 3)] = np.uint32(bits)
    print(f"long rows B={B} N={N} k={k} relu={relu}", flush=True)
    ranked = np.where(v > 0.0, v, np.float32(0.0)) if relu else v
    keys = _order_keys(ranked)
    order = np.lexsort((np.broadcast_to(np.arange(N), v.shape), ~keys), axis=1)[:, :k]
    scores = torch.from_numpy(v).cuda()
    flags = (hire.RELU if relu else 0) | hire.ORDER_RANK
    ws = hire.alloc_workspace(max(hire.hire_topk_workspace_bytes(B, N, kk, flags) for kk in (k, 2049)))
    long_order = np.lexsort((np.broadcast_to(np.arange(N), v.shape), ~keys), axis=1)[:, :2049]  # (k > 2048: with bitmaps)
    for kk, first in ((k, order), (2049, long_order), (k, order)):
        for rank in (True, False):
            for _ in range(2):
                idx, val = hire.topk_select(scores, kk, relu=relu, rank_order=rank, workspace=ws)
                want = first if rank else np.sort(first, axis=1)
                assert np.array_equal(idx.cpu().numpy(), want)
                assert np.array_equal(_order_keys(val.cpu().numpy()), np.take_along_axis(keys, want, axis=1))
