"""The bound by which the fast search leaves candidates out (CPU only).

k_fast evaluates a grid of candidates and excludes those between whose error is shown to
be past the threshold of the least value: the root of the summed squared error changes by at most
C(k) per candidate, C(k)^2 = min(N, U2/k^2 + U1/(Lk) + N/(4L^2)).  The selection is restated
in numpy (binary32 where the kernel has binary32) over the filter's own values, and the list of
candidates within the threshold has to be the one that the full row of values gives.
"""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from test_filter_bound import F32, adversarial_rows
from test_filter_bound_half_way import filter_half_way

GRID = 128


def threshold(mn, count, n):
    eps = n * 2.0 ** -21
    return mn + 2.0 * (3e-5 * mn + 2.0 * eps * np.sqrt(count * mn) + count * eps * eps + 1e-14 * n * n * count)


def slopes(w, n, bits):
    """C(1..n), as the kernel bounds it."""
    L = 2 ** (bits - 1) - 1
    a = np.abs(w).astype(np.float64)
    u1, u2 = (a / a.max() * n).sum(), np.square(a / a.max() * n).sum()
    k = np.arange(1, n + 1)
    return np.sqrt(np.minimum(len(w), u2 / k ** 2 + u1 / (L * k) + 0.25 * len(w) / L ** 2))


def pruned_list(values, C, count, n):
    log = 2
    while n >> log > GRID:
        log += 1
    step, points = 1 << log, n >> log
    root = np.sqrt(values.astype(F32))                       # of candidate k at k - 1
    grid = [k << log for k in range(1, points + 1)]
    near = F32(threshold(min(values[k - 1] for k in grid), count, n) * (1 + 1e-6))
    top = F32(np.sqrt(near) * F32(1.00002) + F32(6e-7) * F32(n) * np.sqrt(F32(count)))
    seen = list(grid)
    for i in range(points + 1):
        a = i << log
        if a == n:
            continue
        per = F32(1.0) / F32(1.0001 * C[a])                  # of candidate a + 1
        lo, hi = 1, (n - a if n - a < step else step - 1)
        if i > 0:
            d = (root[a - 1] - top) * per - F32(0.01)
            if d > 1:
                lo = int(np.ceil(d)) if d < step else step
        if i < points:
            d = (root[a + step - 1] - top) * per - F32(0.01)
            if d > 1:
                hi = step - int(np.ceil(d)) if d < step else 0
        seen += range(a + lo, a + hi + 1)
    thr = threshold(min(values[k - 1] for k in seen), count, n)
    return sorted(k for k in seen if values[k - 1] <= thr), len(seen)


@pytest.mark.parametrize("bits,n,K", [(2, 256, 300), (2, 1000, 64), (3, 2000, 200), (4, 257, 4096), (4, 1000, 576),
                                      (4, 1000, 2000), (5, 300, 1155), (6, 515, 700), (8, 1000, 2100), (4, 5000, 130)])
def test_the_list_is_that_of_the_full_row(bits, n, K):
    rng = np.random.default_rng(bits * 7919 + n)
    rows = [rng.standard_normal(K), rng.laplace(size=K), rng.standard_t(1.5, K), rng.uniform(-1, 1, K),
            rng.laplace(size=K) * np.where(rng.random(K) < 0.002, 10, 1), rng.choice([-1.0, 0.3, 0.0], K),
            np.exp(rng.uniform(-30, 0, K)), np.where(np.arange(K) == 5, 1.0, 0.01 * rng.standard_normal(K))]
    evaluated = []
    for w in rows:
        w = w.astype(F32)
        values = filter_half_way(w, n, bits)
        want = [k + 1 for k in np.flatnonzero(values <= threshold(values.min(), K, n))]
        got, seen = pruned_list(values, slopes(w, n, bits), K, n)
        assert got == want
        evaluated.append(seen)
    assert min(evaluated) < n                                # something is left out


@pytest.mark.parametrize("bits,n", [(2, 500), (4, 1000), (8, 300)])
def test_the_bound_on_adversarial_rows(bits, n):
    """Roots of the oracle's curve: neighbours at every distance up to 64 within C(k) of each other."""
    for w in adversarial_rows(600, n, bits, np.random.default_rng(bits)).values():
        w = np.asarray(w, dtype=F32)
        if not np.abs(w).max() > 0:
            continue
        m = float(np.abs(w).max())
        f = np.sqrt(R.search(w[None], bits, n, want_curve=True)["curve"][0]) / m * n
        C = slopes(w, n, bits)
        slack = 2.0 ** -21 * n * np.sqrt(len(w))             # the oracle's codes are decided in binary32
        for d in (1, 2, 5, 16, 64):
            # f(k) >= f(k') - |k - k'| C(k), k the candidate that is left out
            assert (f[:-d] >= f[d:] - d * C[:-d] - slack).all()
            assert (f[d:] >= f[:-d] - d * C[d:] - slack).all()
