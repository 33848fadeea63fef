"""Dose on the voxel rows: both homes of the weights (LDS, cache), rows at the edges of a step,
arrays whose offsets differ, and more rows than one round of workgroups gives the FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [  # rows, mean entries, beamlets, offsets of the index and value arrays, columns outside the range
    (1, 1, 1, (0, 0), False), (63, 3, 5, (0, 0), False), (65, 31, 40, (1, 1), False), (129, 32, 10240, (2, 2), True),
    (200, 33, 10241, (3, 3), True), (77, 300, 20000, (0, 1), True), (300, 65, 700, (2, 1), False),
    (8191 * 64 + 65, 2, 300, (1, 1), True), (40, 5000, 9000, (3, 3), False), (50, 0, 10, (0, 0), False),
]


@pytest.mark.parametrize("rows,mean,n_w,off,outside", CASES)
def test_voxel_dose_is_the_fp64_sum(rows, mean, n_w, off, outside):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import VoxelCSR
    rng = np.random.default_rng(rows + 13 * mean)
    lens = rng.poisson(mean, rows) if rows > 1 else np.array([mean])
    lens[:5] = np.array([0, 32, 33, 35, 64])[:len(lens[:5])] if mean and rows > 5 else lens[:5]
    ip = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = rng.integers(0, n_w, ip[-1]).astype(np.int32)
    val = rng.normal(size=len(idx)).astype(np.float32)
    if outside:
        bad = rng.uniform(size=len(idx)) < 0.2
        idx[bad] = rng.choice([-1, n_w, n_w + 3, 2 ** 31 - 1], size=int(bad.sum()))
        val[bad] = np.nan                              # skipped, whatever they hold
    w = rng.uniform(-1.0, 1.0, n_w).astype(np.float32)
    ok = (idx >= 0) & (idx < n_w)
    row = np.repeat(np.arange(rows), lens)[ok]
    term = val[ok].astype(np.float64) * w[idx[ok]].astype(np.float64)
    want = np.bincount(row, weights=term, minlength=rows)
    size = np.bincount(row, weights=np.abs(term), minlength=rows)
    many = np.bincount(row, minlength=rows)
    ti = torch.zeros(len(idx) + 4, dtype=torch.int32, device="cuda:0")[off[0]:off[0] + len(idx)]
    tv = torch.zeros(len(idx) + 4, dtype=torch.float32, device="cuda:0")[off[1]:off[1] + len(idx)]
    ti.copy_(torch.from_numpy(idx))
    tv.copy_(torch.from_numpy(val))
    T = VoxelCSR(torch.from_numpy(ip).cuda(), ti, tv, n_w)
    wg = torch.from_numpy(w).cuda()
    got = T.dose(wg)
    # one rounding per product, one per addition (in any order)
    assert np.all(np.abs(got.cpu().numpy() - want) <= (many + 1) * 2.0 ** -24 * size)
    assert torch.equal(T.dose(wg), got)
