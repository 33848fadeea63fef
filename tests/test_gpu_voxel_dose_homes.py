"""Dose on the voxel rows on both sides of the number of weights per entry that decides whether the
weights are copied to LDS: the same bits, and the FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,mean,start", [(64, 40, 0), (65, 70, 0), (700, 9, 0), (900, 7, 5)])
def test_the_home_of_the_weights_does_not_matter(rows, mean, start):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import VoxelCSR
    rng = np.random.default_rng(rows + mean)
    groups = -(-rows // 64)                                     # workgroups, a copy of the weights each
    lens = rng.poisson(mean, rows)
    lens[0] += -int(lens.sum()) % groups                        # so that the words divide evenly
    ip = start + np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    nnz = int(lens.sum())
    n_w = 3 * nnz // groups                                     # the most that are copied
    assert n_w > 1024                                           # fewer are copied in any case
    idx = rng.integers(0, n_w, start + nnz).astype(np.int32)
    val = rng.normal(size=start + nnz).astype(np.float32)
    w = rng.uniform(-1.0, 1.0, n_w + 1).astype(np.float32)
    dev = [torch.from_numpy(x).cuda() for x in (ip, idx, val)]
    got = [VoxelCSR(*dev, k).dose(torch.from_numpy(w[:k]).cuda()) for k in (n_w, n_w + 1)]
    assert torch.equal(got[0], got[1])
    row = np.repeat(np.arange(rows), lens)
    term = val[start:].astype(np.float64) * w[idx[start:]].astype(np.float64)
    want = np.bincount(row, weights=term, minlength=rows)
    size = np.bincount(row, weights=np.abs(term), minlength=rows)
    # one rounding per product, one per addition (in any order)
    assert np.all(np.abs(got[0].cpu().numpy() - want) <= (lens + 1) * 2.0 ** -24 * size)
