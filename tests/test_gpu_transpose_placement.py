"""Transpose on both sides of the entries and the runs per bucket of 32 columns that decide how many
waves place a bucket: the stable sort by column."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 640          # 20 buckets


@pytest.mark.parametrize("per_bucket", [511, 512, 513, 1023, 1024, 1025])
@pytest.mark.parametrize("run", [32, 16, 5])
@pytest.mark.parametrize("outside", [False, True])
def test_transpose_is_the_stable_sort(per_bucket, run, outside):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    rng = np.random.default_rng(per_bucket * run)
    rows, left = [], per_bucket * (N // 32)
    while left > 0:          # rows of runs within buckets, then as many entries as are left
        c = np.concatenate([32 * b + int(rng.integers(0, 33 - run)) + np.arange(run) for b in range(N // 32)])[:left]
        if outside and len(rows) < 3:
            c = np.concatenate([c, N + np.arange(min(200, left - len(c)))])      # one long run that is not placed
        rows.append(c)
        left -= len(c)
    ip = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    idx = np.concatenate(rows).astype(np.int32)
    val = rng.normal(size=len(idx)).astype(np.float32)
    T = CSR(torch.from_numpy(ip).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(), N).transpose()
    row = np.repeat(np.arange(len(rows), dtype=np.int32), np.diff(ip))
    order = np.argsort(np.where(idx < N, idx, N), kind="stable")[:int((idx < N).sum())]
    want = np.concatenate([[0], np.cumsum(np.bincount(idx[idx < N], minlength=N))])
    np.testing.assert_array_equal(T.indptr.cpu().numpy(), want)
    np.testing.assert_array_equal(T.indices.cpu().numpy()[:len(order)], row[order])
    np.testing.assert_array_equal(T.values.cpu().numpy()[:len(order)].view(np.int32), val[order].view(np.int32))
