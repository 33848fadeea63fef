"""Gradient on the beamlet rows: rows at the edges of a workgroup's step, on both sides of the
row count that decides its width, give the FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 63, 64, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 12345]


@pytest.mark.parametrize("rows,n", [(1, 20000), (20, 20000), (10240, 20000), (10241, 20000)])
def test_gradient_is_the_fp64_sum(rows, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    rng = np.random.default_rng(rows)
    lens = rng.poisson(20, rows)
    lens[:20] = EDGES[:min(rows, 20)] if rows > 1 else 4097
    ip = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = rng.integers(0, n, ip[-1]).astype(np.int32)
    val = rng.normal(size=len(idx)).astype(np.float32)
    bad = rng.uniform(size=len(idx)) < 0.1
    idx[bad] = rng.choice([-1, n, n + 3, 2 ** 31 - 1], size=int(bad.sum()))
    val[bad] = np.nan                                  # skipped, whatever they hold
    r = rng.uniform(-1.0, 1.0, n).astype(np.float32)
    ok = ~bad
    row = np.repeat(np.arange(rows), lens)[ok]
    term = val[ok].astype(np.float64) * r[idx[ok]].astype(np.float64)
    want = np.bincount(row, weights=term, minlength=rows)
    size = np.bincount(row, weights=np.abs(term), minlength=rows)
    many = np.bincount(row, minlength=rows)
    D = CSR(torch.from_numpy(ip).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(), n)
    rg = torch.from_numpy(r).cuda()
    got = D.gradient(rg)
    # one rounding per product, one per addition (in any order)
    assert np.all(np.abs(got.cpu().numpy() - want) <= (many + 1) * 2.0 ** -24 * size)
    assert torch.equal(D.gradient(rg), got)
