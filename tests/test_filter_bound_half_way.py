"""The prefix-sum filter of the fast search against its own error bound, and against the
same sums over binary32 magnitudes (CPU only).

k_fast holds magnitudes as integers in units of 1/(2L q) of a candidate, q the
largest that keeps n candidates within 2^30 - 2^23 - 64, each one binary64 product
rounded once, and gets a candidate's squared error from H(b) = sum max(b - u, 0) at the
2L half-way points, which are integers too.  The same arithmetic is restated here in
numpy (integers where the kernel has integers) on the inputs of test_filter_bound.py:
every value has to lie within half the slack of the filter of the oracle's curve, and the
values have to be no further from the error in exact arithmetic than those of the binary32
magnitudes.
"""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from test_filter_bound import F32, adversarial_rows, half_slack, to_units

TOP = 2 ** 30 - 2 ** 23 - 64


def filter_half_way(w, n, bits):
    L = 2 ** (bits - 1) - 1
    q = TOP // (2 * L * n)
    top = 2 * L * q * n
    a = np.abs(w.astype(F32)).astype(np.float64)
    U = np.sort(np.rint(a * (float(top) / a.max())).astype(np.int64))
    assert 0 <= U[0] and U[-1] <= top
    C = np.concatenate([[0], np.cumsum(U)])
    A = float(sum(int(x) ** 2 for x in top - U)) / float(2 * L * q) ** 2
    odd = 2 * np.arange(L, dtype=np.int64) + 1
    k = np.arange(1, n + 1, dtype=np.int64)[:, None]
    h = []
    for b in (odd * (k * q), 2 * L * k * q + odd * ((n - k) * q)):
        N = np.searchsorted(U, b, side="right")
        h.append((b * N - C[N]).sum(1).astype(np.float64))
    kd = k[:, 0].astype(np.float64)
    sse = A - (kd * h[0] + (n - kd) * h[1]) / (float(L) * L * q)
    return np.maximum(sse, 0.0).astype(F32).astype(np.float64)


def prefix_sums_of_binary32(u, n, bits):
    """The yardstick of the precision test: cumulative counts and sums of the binary32
    magnitudes at the half-way points of the levels (half-way points in binary32, sums in
    binary64)."""
    Li = 2 ** (bits - 1) - 1
    Ld = float(Li)
    us = np.sort(u)
    c1 = np.concatenate([[0.0], np.cumsum(us.astype(np.float64))])
    c2 = np.concatenate([[0.0], np.cumsum(us.astype(np.float64) ** 2)])
    S1, S2, K = c1[-1], c2[-1], len(us)
    j = np.arange(Li)
    out = np.empty(n)
    for k in range(1, n + 1):
        kd = float(k)
        half_c = F32(kd / (2.0 * Ld))
        cn = np.searchsorted(us, (2 * j + 1).astype(F32) * half_c, side="right")
        sumC, sumN = c1[cn].sum(), int(((2 * j + 1) * cn).sum())
        nL = int(np.searchsorted(us, F32(k), side="right"))
        cL, s2L = c1[nL], c2[nL]
        s = kd / Ld
        sse = s2L - 2.0 * s * (Ld * cL - sumC) + s * s * (Ld * Ld * nL - sumN)
        if k < n:
            wd = float(n - k)
            half_t = F32(wd / (2.0 * Ld))
            b = ((2 * j + 1).astype(np.float64) * np.float64(half_t) + kd).astype(F32)     # fused
            cn = np.searchsorted(us, b, side="right")
            nt = cn - nL
            sumCt = ((c1[cn] - cL) - kd * nt).sum()
            sumNt = int(((2 * j + 1) * nt).sum())
            ntL = K - nL
            ctL = (S1 - cL) - kd * ntL
            s2t = (S2 - s2L) - 2.0 * kd * (S1 - cL) + kd * kd * ntL
            s = wd / Ld
            sse += s2t - 2.0 * s * (Ld * ctL - sumCt) + s * s * (Ld * Ld * ntL - sumNt)
        out[k - 1] = max(sse, 0.0)
    return out.astype(F32).astype(np.float64)


@pytest.mark.parametrize("bits,n,K", [(4, 1000, 1024), (2, 257, 700), (8, 500, 2048), (3, 2000, 1500),
                                      (4, 65535, 160), (4, 100, 8192), (8, 65535, 40), (2, 1, 64),
                                      (8, 32768, 120), (8, 33026, 120)])
def test_half_way_values_stay_within_half_the_slack(bits, n, K):
    rng = np.random.default_rng(bits * 100000 + n)
    for name, row in adversarial_rows(K, n, bits, rng).items():
        w = row.astype(F32)[None, :]
        ref = R.search(w, bits, n, want_curve=True)
        m = to_units(w[0], n)[1]
        T = ref["curve"][0] * (float(n) / float(m)) ** 2
        ratio = np.abs(filter_half_way(w[0], n, bits) - T) / half_slack(T, float(K), n, True)
        assert ratio.max() <= 1.0, (name, int(ratio.argmax()) + 1, float(ratio.max()))


def exact_errors(w, n, bits):
    """Squared error of every candidate in binary64: distance to the nearest level."""
    L = 2 ** (bits - 1) - 1
    a = np.abs(w.astype(F32)).astype(np.float64)
    u = a * (n / a.max())
    out = np.empty(n)
    for k in range(1, n + 1):
        s, t, v = k / L, (n - k) / L, u - k
        e = u - s * np.rint(u / s)
        if k < n:
            e = np.where(u <= k, e, v - t * np.rint(v / t))
        out[k - 1] = (e * e).sum()
    return out


@pytest.mark.parametrize("bits,n,K", [(4, 1000, 1024), (2, 257, 700), (8, 500, 2048), (3, 2000, 1500), (4, 100, 8192)])
def test_values_are_as_close_as_those_of_binary32_magnitudes(bits, n, K):
    """Root mean square over the candidates; the values are stored in binary32, so their own
    last half bit is allowed on top.  (A tile with more than 1/16 of its weights, and more than
    64, of one magnitude is evaluated element by element from binary32 magnitudes.)"""
    rng = np.random.default_rng(bits * 100000 + n)
    for name, row in adversarial_rows(K, n, bits, rng).items():
        w = row.astype(F32)
        equal = np.unique(np.abs(w[w != 0]), return_counts=True)[1].max()
        if equal > max(64, K // 16):
            continue
        E = exact_errors(w, n, bits)
        got, plain = (np.sqrt(np.mean((v - E) ** 2)) for v in
                      (filter_half_way(w, n, bits), prefix_sums_of_binary32(to_units(w, n)[0], n, bits)))
        stored = 2.0 ** -24 * np.sqrt(np.mean(E ** 2))
        assert got <= plain + stored, (name, got, plain, stored)
