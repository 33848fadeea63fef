"""The transpose on rows cut into pieces (few long rows), runs with and without holes, runs at the
ends of the arrays, invalid columns and rows out of order: bit-exact against a stable sort by column."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# rows, entries per row, columns, kind
CASES = [
    (1, 1, 1, "dense"), (1, 5000, 5000, "dense"), (2, 1023, 4000, "dense"), (3, 1024, 1500, "dense"),
    (3, 1025, 1500, "dense"), (5, 40000, 50000, "dense"), (7, 30001, 100003, "holes"), (64, 3000, 3333, "holes"),
    (65, 3000, 9000, "dense"), (257, 700, 33, "dense"), (300, 31, 31, "dense"), (40, 9000, 20000, "outside"),
    (6, 20000, 30000, "reversed"), (6, 20000, 700, "repeated"), (9000, 40, 4000, "dense"), (12, 2500, 10 ** 6, "sparse"),
]


def _columns(rng, k, n, kind):
    lo = int(rng.integers(0, max(1, n - k + 1)))
    if kind == "repeated":
        return np.sort(rng.integers(0, n, k))
    if kind == "sparse":
        return np.sort(rng.choice(n, size=k, replace=False))
    c = np.arange(lo, min(n, lo + k))
    if kind == "holes":
        c = c[rng.uniform(size=len(c)) < 0.9]
    if kind == "outside":        # still ascending: a tail past the grid
        c = np.concatenate([c, np.arange(n, n + 37)])
    return c[::-1] if kind == "reversed" else c


@pytest.mark.parametrize("rows,k,n,kind", CASES)
def test_transpose_is_the_stable_sort(rows, k, n, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    rng = np.random.default_rng(rows + k)
    cols = [_columns(rng, k, n, kind).astype(np.int32) for _ in range(rows)]
    idx = np.concatenate(cols)
    ip = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    row = np.repeat(np.arange(rows, dtype=np.int32), np.diff(ip))
    val = rng.normal(size=len(idx)).astype(np.float32)
    order = np.argsort(idx, kind="stable")
    order = order[(idx[order] >= 0) & (idx[order] < n)]
    T = CSR(torch.from_numpy(ip).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(), n).transpose()
    m = len(order)
    np.testing.assert_array_equal(T.indptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(idx[order], minlength=n))]))
    np.testing.assert_array_equal(T.indices.cpu().numpy()[:m], row[order])
    np.testing.assert_array_equal(T.values.cpu().numpy()[:m], val[order])
