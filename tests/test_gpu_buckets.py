"""Counting sort of the pairs by block: every number of threads it is launched with, chunks with more pairs than a
thread holds, shares of chunks that do not divide, and the bases from a launch of their own.  Whole numbers: equal to a stable sort."""
import numpy as np
import pytest
import torch

from paper_2312_10365_amd import spt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,N,k", [
    (8192, 4, 2),            # 256 threads, four buckets
    (4097, 33, 3),           # one token in the last chunk
    (2048, 32, 8),           # 512 threads
    (1300, 257, 7),          # as many threads as buckets, rounded up
    (2100, 96, 16),          # 1024 threads, shares of 17 chunks
    (700, 128, 64),          # eight pairs per thread in a full chunk
    (650, 130, 65),          # one more than that
    (300, 1024, 100),        # a thread per bucket, no share
    (2700, 1024, 4),         # bases from their own launch
])
def test_sorted_positions(T, N, k):
    rng = np.random.default_rng(T + N + k)
    idx = np.sort(np.argsort(rng.random((T, N)) - 0.4 * (np.arange(N) % 5 == 1), axis=1)[:, :k], axis=1).astype(np.int32)
    shape = spt.make_shape(T, 64, N, 32, k, spt.ACT_RELU)
    print(f"T {T} N {N} k {k}", flush=True)
    offsets, perm, inv = spt.bucket_tokens(shape, torch.from_numpy(idx).cuda())
    flat = idx.ravel()
    order = np.argsort(flat, kind="stable").astype(np.int32)
    np.testing.assert_array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(flat, minlength=N))]))
    np.testing.assert_array_equal(perm.cpu().numpy(), order)
    back = np.empty_like(order)
    back[order] = np.arange(T * k, dtype=np.int32)
    np.testing.assert_array_equal(inv.cpu().numpy().ravel(), back)
