"""The prefix-sum filter of the fast search against its own error bound (CPU only).

k_fast holds magnitudes as integers in units of 1/(2L q) of a candidate, q the
largest that keeps n candidates within 2^24 - 1 - 2^17, and gets a candidate's
squared error from H(b) = sum max(b - u, 0) at the 2L half-way points, which are
integers too.  The same arithmetic is restated here in numpy (integers where the
kernel has integers) and compared with the oracle's curve on the inputs of
test_filter_bound.py: every value has to lie within half the slack of the filter.
"""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from test_filter_bound import adversarial_rows, half_slack, to_units

TOP = 2 ** 24 - 1 - 2 ** 17


def filter_half_way(u, n, bits):
    L = 2 ** (bits - 1) - 1
    q = TOP // (2 * L * n)
    U = np.sort(np.rint(u * np.float32(2 * L * q)).astype(np.int64))       # binary32 product, then whole
    top = 2 * L * q * n
    assert 0 <= U[0] and U[-1] <= top
    C = np.concatenate([[0], np.cumsum(U)])
    A = float(sum(int(x) for x in (top - U) ** 2)) / float(2 * L * q) ** 2
    odd = 2 * np.arange(L, dtype=np.int64) + 1
    k = np.arange(1, n + 1, dtype=np.int64)[:, None]
    h = []
    for b in (odd * (k * q), 2 * L * k * q + odd * ((n - k) * q)):
        N = np.searchsorted(U, b, side="right")
        h.append((b * N - C[N]).sum(1).astype(np.float64))
    kd = k[:, 0].astype(np.float64)
    sse = A - (kd * h[0] + (n - kd) * h[1]) / (float(L) * L * q)
    return np.maximum(sse, 0.0).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("bits,n,K", [(4, 1000, 1024), (2, 257, 700), (8, 500, 2048), (3, 2000, 1500),
                                      (4, 65535, 160), (4, 100, 8192), (8, 65535, 40), (2, 1, 64)])
def test_half_way_values_stay_within_half_the_slack(bits, n, K):
    rng = np.random.default_rng(bits * 100000 + n)
    for name, row in adversarial_rows(K, n, bits, rng).items():
        w = row.astype(np.float32)[None, :]
        ref = R.search(w, bits, n, want_curve=True)
        u, m = to_units(w[0], n)
        T = ref["curve"][0] * (float(n) / float(m)) ** 2
        ratio = np.abs(filter_half_way(u, n, bits) - T) / half_slack(T, float(K), n, True)
        assert ratio.max() <= 1.0, (name, int(ratio.argmax()) + 1, float(ratio.max()))
