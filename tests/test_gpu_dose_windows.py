"""Dose on the beamlet rows: every route of an entry (a wave's window, straight to memory) gives
the FP64 sum, whatever the order of a row's columns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rows(rng, lens, n, order):
    idx = []
    for k in lens:
        lo = int(rng.integers(0, max(1, n - 3 * k)))
        c = lo + np.sort(rng.choice(min(n - lo, max(k, 3 * k)), size=k, replace=False))
        if order == "descending":
            c = c[::-1]
        elif order == "shuffled":
            c = rng.permutation(c)
        elif order == "repeated":
            c = np.sort(rng.choice(c, size=k)) if k else c
        elif order == "outside" and k:
            c = c.copy()
            c[rng.choice(k, size=max(1, k // 5), replace=False)] = rng.choice([-1, -7, n, n + 5, 2 ** 31 - 1])
        elif order == "dense":
            c = np.arange(k) + (n - k) // 2
        idx.append(c.astype(np.int32))
    return np.concatenate(idx) if idx else np.zeros(0, np.int32)


CASES = [  # rows, mean entries, columns, order
    (1, 1, 1, "ascending"), (1, 5000, 5000, "dense"), (31, 300, 2047, "ascending"), (33, 700, 4097, "dense"),
    (32, 2049, 2049, "dense"), (40, 64, 10 ** 5, "ascending"), (511, 200, 3000, "ascending"), (512, 200, 3000, "dense"),
    (513, 900, 9000, "outside"), (70, 4000, 20000, "descending"), (70, 4000, 20000, "shuffled"),
    (70, 4000, 20000, "repeated"), (640, 129, 6000, "outside"), (2100, 17, 10 ** 6, "ascending"),
    (64, 6000, 2 ** 15, "dense"), (9, 2000, 10 ** 6, "outside"),
]


@pytest.mark.parametrize("rows,mean,n,order", CASES)
def test_dose_is_the_fp64_sum(rows, mean, n, order):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    rng = np.random.default_rng(rows * 7 + mean)
    lens = np.minimum(rng.poisson(mean, rows), n) if rows > 1 else np.array([min(mean, n)])
    lens[rng.uniform(size=rows) < 0.1 * (rows > 4)] = 0
    idx = _rows(rng, lens, n, order)
    ip = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    val = rng.normal(size=len(idx)).astype(np.float32)
    w = rng.uniform(0.1, 2.0, rows).astype(np.float32)
    w[::5] = 0.0
    row = np.repeat(np.arange(rows), lens)
    val[w[row] == 0.0] = np.nan                       # rows of weight 0 add nothing
    ok = (idx >= 0) & (idx < n) & (w[row] != 0.0)
    term = w[row[ok]].astype(np.float64) * val[ok].astype(np.float64)
    want = np.bincount(idx[ok], weights=term, minlength=n)
    size = np.bincount(idx[ok], weights=np.abs(term), minlength=n)
    many = np.bincount(idx[ok], minlength=n)
    D = CSR(torch.from_numpy(ip).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(), n)
    got = D.dose(torch.from_numpy(w).cuda()).cpu().numpy().astype(np.float64)
    # one rounding per product, one per addition (in any order)
    assert np.all(np.abs(got - want) <= (many + 1) * 2.0 ** -24 * size)
