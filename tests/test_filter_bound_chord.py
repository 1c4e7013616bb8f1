"""The chords by which the fast search leaves candidates out (CPU only).

Between two evaluated candidates k0, k1 the summed squared error lies above the chord of its values less
(k - k0) (k1 - k) (D1 - D0) / (k1 - k0), D = (2/L) (sum H in the tail - sum H in the centre).  Shown against the
exact error of every candidate, and the selection that k_fast makes of it, restated in numpy (binary32 where the kernel has
binary32), over the filter's own values: the list of candidates within the threshold has to be
that of the full row.
"""
import numpy as np
import pytest

from test_filter_bound import F32, adversarial_rows
from test_filter_bound_half_way import filter_half_way
from test_filter_bound_pruned import threshold


def rows(K, seed):
    rng = np.random.default_rng(seed)
    return [rng.standard_normal(K), rng.laplace(size=K), rng.standard_t(1.5, K), rng.uniform(-1, 1, K),
            rng.laplace(size=K) * np.where(rng.random(K) < 0.002, 10, 1), rng.choice([-1.0, 0.3, 0.0], K),
            np.exp(rng.uniform(-30, 0, K)), np.where(np.arange(K) == 5, 1.0, 0.01 * rng.standard_normal(K))]


def sums(w, n, bits):
    """sum H over the half-way points of the centre and of the tail for candidates 0..n, and the error, in binary64."""
    L = 2 ** (bits - 1) - 1
    u = np.abs(w).astype(np.float64)
    u = np.sort(u / u.max() * n)
    before = np.concatenate([[0.0], np.cumsum(u)])

    def H(b):
        c = np.searchsorted(u, b)
        return b * c - before[c]

    k, i = np.arange(n + 1), 2 * np.arange(L) + 1
    h = sum(H(j * k / (2 * L)) for j in i)
    t = sum(H(k + j * (n - k) / (2 * L)) for j in i)
    return h, t, np.square(n - u).sum() - 2 / L * (k * h + (n - k) * t)


def grid_of(n, bits):
    most = 32 if bits <= 3 else 64 if bits == 4 else 128
    log = 2
    while n >> log > most:
        log += 1
    points = min(n + (1 << log) - 1 >> log, most)               # of a full grid the last step may be up to two
    return np.append(np.arange(points) << log, n)


@pytest.mark.parametrize("bits,n,K", [(2, 300, 300), (3, 515, 64), (4, 1000, 2000), (5, 777, 1155), (8, 300, 700)])
def test_the_error_is_above_the_parabola(bits, n, K):
    L = 2 ** (bits - 1) - 1
    extra = [np.asarray(w, dtype=np.float64) for w in adversarial_rows(600, n, bits, np.random.default_rng(n)).values()]
    for w in rows(K, n) + [w for w in extra if np.abs(w).max() > 0]:
        h, t, sse = sums(w, n, bits)
        D = 2 / L * (t - h)
        assert abs(D[0] - 2 / L * h[n]) <= 1e-9 * abs(D[0]) and abs(sse[0] - sse[n]) <= 1e-9 * n * n * len(w)
        for step in (4, 16, 64):
            for k0 in range(0, n, step):
                k1 = min(k0 + step, n)
                x = np.arange(k1 - k0 + 1)
                low = sse[k0] + (sse[k1] - sse[k0]) * x / (k1 - k0) - (D[k1] - D[k0]) / (k1 - k0) * x * (k1 - k0 - x)
                assert (low <= sse[k0:k1 + 1] + 1e-12 * n * n * len(w)).all()


def pruned_list(values, D, count, n, grid):
    """values, D: of candidates 0..n."""
    f = F32
    near = threshold(min(values[k] for k in grid[1:]), count, n) * (1 + 1e-6)
    top = f(near * 1.00002 + 4e-14 * n * n * count)
    seen = list(grid[1:])
    for a, c in zip(grid[:-1], grid[1:]):
        s = f(c - a)
        v0, v1, d0, d1 = (f(x) for x in (values[a], values[c], D[a], D[c]))
        rs = f(1.000001) / s
        up = d1 - d0 + f(2e-7) * (abs(d0) + abs(d1))
        g = max(up * f(1.0001), f(0)) * rs + f(1e-6) * (v0 + v1 + top) * rs * rs
        b, v = (v1 - v0) * rs - g * s, v0 - top
        disc = b * b - 4 * g * v + f(4e-6) * (b * b + 4 * g * abs(v))
        if disc < 0:
            continue
        q = f(-0.5) * (b + (-1 if b < 0 else 1) * np.sqrt(disc))
        with np.errstate(all="ignore"):
            x = np.array([q / g, v / q])
        first, last = np.fmin(*x) - f(0.01), np.fmax(*x) + f(0.01)
        lo = 1 if first <= 1 else int(np.ceil(first)) if first < s else int(s)
        hi = int(s) - 1 if last >= s else min(int(last) if last > 0 else 0, int(s) - 1)
        seen += range(a + lo, a + hi + 1)
    thr = threshold(min(values[k] for k in seen), count, n)
    return sorted(k for k in seen if values[k] <= thr), len(seen)


@pytest.mark.parametrize("bits,n,K", [(2, 300, 300), (2, 1000, 64), (3, 2000, 200), (4, 301, 4096), (4, 1000, 576),
                                      (4, 1000, 2000), (5, 303, 1155), (3, 262, 500), (4, 519, 300), (6, 515, 700), (8, 1000, 2100), (4, 5000, 130)])
def test_the_list_is_that_of_the_full_row(bits, n, K):
    evaluated = []
    for w in rows(K, bits * 7919 + n):
        w = w.astype(F32)
        row = filter_half_way(w, n, bits)                    # of candidates 1..n
        values = np.concatenate([row[-1:], row])
        h, t, _ = sums(w, n, bits)
        D = (2 / (2 ** (bits - 1) - 1) * (t - h)).astype(F32)
        want = [k + 1 for k in np.flatnonzero(row <= threshold(row.min(), K, n))]
        got, seen = pruned_list(values, D, K, n, grid_of(n, bits))
        assert got == want
        evaluated.append(seen)
    assert min(evaluated) < n / (2 if bits < 8 else 1)       # much is left out
