"""Dose on the beamlet rows through shares of thousands of entries: several windows a share, their
guessed ends, sets that do not ascend, columns outside the grid, windows given up part of the way,
and groups that take rows or pieces of rows.  A replay of the kernel's split on the host says which
of these a case reaches, and the dose is the FP64 sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# the kernel's constants
ROWS, FEW_ROWS, MANY, GROUPS = 32, 8, 512, 1024
WINDOW, MIN_ENTRIES, SLACK, SHARE, PIECE, SPREAD, GUESS = 2048, 64, 1024, 2048, 128, 8, 24
WAVES_PER_GROUP = 4
TOP = 0xffffffff


def _replay_share(col, p, end, n, seen_routes):
    """One wave's windows over the parts [p, end) of its rows; col: columns as unsigned."""
    p, guess, seen, out, windows = p.copy(), None, 0, 0, 0
    while np.any(p < end):
        windows += 1
        base = min(col[a] for a, b in zip(p, end) if a < b) & ~31
        stop = base + WINDOW if base < TOP - WINDOW else TOP
        lo, hi = p.copy(), np.minimum(end, p + WINDOW)
        if guess is not None:
            qa, qb = lo + guess - GUESS, lo + guess + GUESS
            ia, ib = (qa >= lo) & (qa < hi), qb < hi
            ca, cb = np.where(ia, col[np.where(ia, qa, 0)], 0), np.where(ib, col[np.where(ib, qb, 0)], 0)
            if ia.any() or ib.any():
                seen_routes.add("guess")
            hi = np.where(ib & (cb >= stop), qb, hi)
            lo = np.where(ib & (cb < stop), qb + 1, lo)
            ia &= qa >= lo
            hi = np.where(ia & (ca >= stop), qa, hi)
            lo = np.where(ia & (ca < stop), qa + 1, lo)
        while np.any(lo < hi):
            mid, go = lo + ((hi - lo) >> 1), lo < hi
            below = col[np.where(go, mid, 0)] < stop
            lo, hi = np.where(go & below, mid + 1, lo), np.where(go & ~below, mid, hi)
        cnt = lo - p
        guess = cnt
        if not np.any(cnt > 0):
            seen_routes.add("hole")
            return
        seen += int(cnt.sum())
        held = []
        for a, k in zip(p, cnt):
            for s in range(a, a + k, 64):
                c = col[s:min(s + 64, a + k)]
                asc = bool(np.all(c[1:] > c[:-1]))
                inside = (c < n) & (c - base >= 0) & (c - base < WINDOW)
                if not asc:
                    seen_routes.add("set out of order")
                elif not inside.all():
                    seen_routes.add("entry outside its window")
                if asc:
                    held.append(c[inside])
        out += len(np.unique(np.concatenate(held))) if held else 0
        p = lo
        if windows > 1:
            seen_routes.add("windows")
        if 4 * out > 3 * seen + SLACK or seen + SLACK < windows * MIN_ENTRIES:
            if np.any(p < end):
                seen_routes.add("given up")
            return


def _replay(ip, idx, w, n):
    """The routes that the waves of the first, middle and last group of rows take."""
    routes, rows = set(), len(ip) - 1
    col = (idx.astype(np.int64)) & TOP
    group = ROWS if rows >= MANY else FEW_ROWS
    groups = -(-rows // group)
    waves = WAVES_PER_GROUP * min(64, max(1, GROUPS // groups))
    for g in {0, groups // 2, groups - 1}:
        j = np.arange(g * group, min((g + 1) * group, rows))
        j = j[w[j] != 0.0]
        e0, length = ip[j], ip[j + 1] - ip[j]
        if length.sum() < SHARE * waves:
            routes.add("pieces" if min(waves // min(group, rows - g * group), length.sum() // len(j) // PIECE) > 1 else "rows")
            continue
        some = length > 0
        a, m, b = (np.where(some, col[np.minimum(e0 + k, len(col) - 1)], 0) for k in (0, length // 2, length - 1))
        if np.any((a > m) | (m > b)):
            routes.add("rows of no order")
            continue
        cut = lambda k: e0 + length // waves * k + length % waves * k // waves
        for me in {0, 1, waves * 2 // 5, waves // 2, waves - 2, waves - 1}:
            p, end = cut(me), cut(me + 1)
            lo, hi = col[p].astype(np.int64), col[end - 1].astype(np.int64)
            span = int(hi.max() - min(lo.min(), hi.max()))
            if span > SPREAD * int((end - p).sum()):
                routes.add("share without windows")
            else:
                _replay_share(col, p, end, n, routes)
    return routes


def _matrix(rng, rows, length, n, order):
    """Rows of ascending columns that start near one another, then disturbed."""
    lens = rng.integers(int(0.995 * length), length + 1, rows)
    idx = []
    for j, k in enumerate(lens):
        if order == "diverging":       # the first half of every row on the same columns, the second on its own
            half = k // 2
            c = np.concatenate([np.arange(half), length + 8 * np.arange(k - half) + j % 8])
        else:
            c = int(rng.integers(0, 200)) + np.cumsum(rng.integers(1, 4, k))
        c = c.astype(np.int64)
        x = rng.integers(1, max(2, k - 1), max(1, k // 500))
        x = x[(x != k // 2) & (x < k - 1)]
        if order == "swapped":
            c[x - 1], c[x] = c[x].copy(), c[x - 1].copy()
        elif order == "repeated":
            c[x] = c[x - 1]
        elif order == "outside":
            c[x] = rng.choice([-1, -9, n, n + 5, 2 ** 31 - 1], len(x))
        elif order == "hole":          # a stretch longer than a window, at the same place of every row
            c[int(0.4 * k):int(0.4 * k) + 3000] = -1
        elif order == "shuffled":
            c = rng.permutation(c)
        idx.append(c.astype(np.int32))
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), np.concatenate(idx)


CASES = [  # rows, entries, order, routes that the case is there for
    (8, 1000000, "ascending", {"windows", "guess"}), (8, 1000000, "swapped", {"windows", "set out of order"}),
    (8, 600000, "repeated", {"windows", "set out of order"}), (8, 1000000, "outside", {"windows", "set out of order"}),
    (8, 1000000, "diverging", {"windows", "given up"}), (3, 2000000, "hole", {"windows", "hole"}),
    (8, 400000, "shuffled", {"rows of no order"}), (1, 1000000, "ascending", {"windows"}), (1, 3000, "ascending", {"pieces"}),
    (8, 60000, "ascending", {"pieces"}), (520, 20000, "swapped", {"set out of order"}),
    (8192, 1400, "outside", {"set out of order"}), (8193, 600, "ascending", {"rows", "pieces"}),
    (33000, 340, "repeated", {"set out of order"}), (33000, 150, "outside", {"rows"}),
]


@pytest.mark.parametrize("rows,length,order,routes", CASES)
def test_dose_is_the_fp64_sum(rows, length, order, routes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_4417_amd import CSR
    rng = np.random.default_rng(rows + length)
    n = 10 * length + 4000
    ip, idx = _matrix(rng, rows, length, n, order)
    w = rng.uniform(0.1, 2.0, rows).astype(np.float32)
    w[3::7] = 0.0
    assert routes <= _replay(ip, idx, w, n)
    val = rng.normal(size=len(idx)).astype(np.float32)
    wr = np.repeat(w, np.diff(ip))
    val[wr == 0.0] = np.nan                           # rows of weight 0 add nothing
    ok = (idx >= 0) & (idx < n) & (wr != 0.0)
    term = wr[ok].astype(np.float64) * val[ok].astype(np.float64)
    want = np.bincount(idx[ok], weights=term, minlength=n)
    size = np.bincount(idx[ok], weights=np.abs(term), minlength=n)
    many = np.bincount(idx[ok], minlength=n)
    assert want.any()
    D = CSR(torch.from_numpy(ip).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(val).cuda(), n)
    got = D.dose(torch.from_numpy(w).cuda()).cpu().numpy().astype(np.float64)
    # one rounding per product, one per addition (in any order)
    assert np.all(np.abs(got - want) <= (many + 1) * 2.0 ** -24 * size)
