"""The one-pass clip search (csrc/clip_search.h) takes its ratio where only one is within K 2^-16 / 196 of the smallest error.  Both
ways of computing the errors, emulated in their own precision: wherever one pass decides, the sum per ratio decides alike, and the
difference to the smallest error differs between them by less than the margin: by 0.6 of it at most on these rows, for ratios far
from the best, and by 0.01 for those near it, ties included."""
import numpy as np
import pytest

F = np.float32


def fma(a, b, c):
    return (a.astype(np.float64) * np.float64(b) + np.float64(c)).astype(F)


def sums(y, amax, grid):
    """search_ratio: fp32 terms, eight at a time, those sums in fp64 (the order of the fp64 sums does not matter here)"""
    err = []
    for r in grid:
        d = F(F(r * amax) / F(7))
        inv15 = F(F(1) / F(F(15) * d))
        u = np.clip(fma(y, inv15, F(8 / 15)), F(0), F(1))
        u = fma(u, F(15), F(12582912))
        c = (u - F(12582920)).astype(F)
        e = (y.astype(np.float64) - np.float64(d) * c.astype(np.float64)).astype(F).reshape(-1, 8)
        even, odd = np.zeros(len(e), F), np.zeros(len(e), F)
        for k in range(0, 8, 2):
            even = (e[:, k].astype(np.float64) ** 2 + even).astype(F)
            odd = (e[:, k + 1].astype(np.float64) ** 2 + odd).astype(F)
        err.append((even + odd).astype(F).astype(np.float64).sum())
    return np.array(err) / float(amax) ** 2


def one_pass(y, amax, grid, q):
    """count_value and ratio_of_cells: errors without the common sum of squares"""
    top = 14 * q
    cell = (np.abs(y) * F(F(top) / amax)).astype(F).astype(np.int64)
    fixed = (np.abs(y) * F(F(2.0 ** 30) / amax)).astype(F).astype(np.int64)
    err = []
    for r in grid:
        a = int(r * F(q) + F(0.5))
        d, e = a / (7.0 * q), 0.0
        for j in range(1, 9):
            c = (2 * j - 1) * a
            above = (cell >= c) & (y < 0) if j == 8 else cell >= c
            if c <= top and above.any():
                e += d * (d * (2 * j - 1) * int(above.sum()) - 2.0 * int(fixed[above].sum()) * 2.0 ** -30)
        err.append(e)
    return np.array(err)


def rows(K, rng):
    for _ in range(6):
        yield rng.standard_normal(K)
        yield rng.standard_t(2, K)
        yield rng.integers(-7, 8, K) / 7.0                                       # codes of ratio 1
        yield (rng.integers(0, 8, K) - 0.5) / 7.0 * rng.choice([-1, 1], K)       # its rounding boundaries
        yield np.where(rng.random(K) < 0.02, rng.standard_normal(K), 0.0) + 1e-3
        for spike in (1.0, -1.0):
            v = rng.standard_normal(K) * rng.choice([0.005, 0.012, 0.02, 0.04])
            v[rng.integers(K)] = spike
            yield v
        yield np.sign(rng.standard_normal(K))


@pytest.mark.parametrize("n,lo,q", [(21, 0.5, 40), (11, 0.5, 20), (32, 0.69, 100), (2, 0.9, 10)])
@pytest.mark.parametrize("K", [2048, 14336])
def test_margin(K, n, lo, q):
    rng = np.random.default_rng(K + n)
    grid = (1.0 - (1.0 - lo) * np.arange(n) / (n - 1)).astype(F)
    margin, decided, worst, worst_near = K * 2.0 ** -16 / 196, 0, 0.0, 0.0
    for v in rows(K, rng):
        y = (v * rng.choice([1e-3, 0.7, 300.0])).astype(F)
        amax = F(np.abs(y).max())
        a, b = sums(y, amax, grid), one_pass(y, amax, grid, q)
        near = np.flatnonzero(b <= b.min() + margin)
        if len(near) == 1:
            decided += 1
            assert near[0] == a.argmin(), (near, a.argmin())
        best = a.argmin()
        off = np.abs((a - a[best]) - (b - b[best])) / margin
        worst, worst_near = max(worst, off.max()), max(worst_near, off[a <= a[best] + 4 * margin].max())
    assert decided > 10
    print("K %d, %d ratios: %d rows decided, differences off by %.3f of the margin, near the best by %.4f" % (K, n, decided, worst, worst_near))
    assert worst < 1 and worst_near < 0.1
