"""Gradient on the beamlet rows on both sides of the row counts that decide a row's threads and its
steps, and of whole sets of rows per XCD: rows at the edges of every step give the FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

STEPS = [1024, 2048, 4096]        # entries of a step: 256 threads by 4 or 8, 1024 by 4
EDGES = [0, 1, 255, 256, 257] + [m * s + d for s in STEPS for m in (1, 2) for d in (-1, 0, 1)] + [1024 + 1023, 6143, 9000]


@pytest.mark.parametrize("rows", [2048, 2049, 2048 + 255, 2048 + 256, 32768, 32769])
def test_gradient_is_the_fp64_sum(rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    n = 30000
    rng = np.random.default_rng(rows)
    lens = rng.poisson(12, rows)
    at = rng.choice(rows, 2 * len(EDGES), replace=False)
    lens[at] = EDGES * 2
    lens[-1] = 2049                                    # a row of the last, partial set
    ip = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = rng.integers(0, n, ip[-1]).astype(np.int32)
    val = rng.normal(size=len(idx)).astype(np.float32)
    bad = rng.uniform(size=len(idx)) < 0.05
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
