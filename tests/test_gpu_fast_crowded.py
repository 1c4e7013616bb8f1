"""k_fast's evaluation element by element, of tiles whose values crowd into a few buckets, against the oracle: in every
size of workgroup, with lengths that leave 0 to 3 elements past the last four and end before, at and after a chunk of 128, and
numbers of candidates that end in the middle of a wavefront, of a pair and of a round of pairs."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches
from test_gpu_fast_pruned import P  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


def crowded(K, rng):
    """Rows of K - 0 .. K - 9 weights other than zero, a third of them in each of three buckets."""
    w = rng.choice([-1.0, 0.7, -0.3, 0.3], (10, K)) * (1 - 1e-5 * rng.random((10, K)))
    for i in range(10):
        w[i, rng.choice(K, i, replace=False)] = 0.0
    return w.astype(np.float32)


@pytest.mark.parametrize("bits,n,K,tiles,want", [
    (4, 300, 256, 8192, "k_fast<64>"), (3, 449, 253, 8192, "k_fast<64>"), (2, 961, 255, 8192, "k_fast<64>"),
    (5, 255, 256, 2048, "k_fast<128>"), (4, 129, 254, 2048, "k_fast<128>"),
    (4, 256, 1023, 2048, "k_fast<256>"), (6, 500, 641, 2048, "k_fast<256>"),
    (4, 300, 1033, 2049, "k_fast<256>"), (4, 511, 1285, 2049, "k_fast<256>"), (4, 513, 1284, 2049, "k_fast<256>"),
    (4, 577, 2050, 2049, "k_fast<256>"), (2, 769, 4099, 2049, "k_fast<256>"), (3, 1025, 5120, 2049, "k_fast<256>"),
    (8, 300, 2041, 2048, "k_fast<512>"), (4, 513, 1027, 64, "k_fast<512>"), (4, 129, 5121, 64, "k_fast<1024>"),
    (4, 1025, 8192, 16, "k_fast<1024>")])
def test_crowded(P, bits, n, K, tiles, want):  # noqa: F811
    import torch
    w = crowded(K, np.random.default_rng(K + n))
    print(f"[case] bits={bits} n={n} K={K}", flush=True)
    before = P.set_small_call_tiles(0)
    try:
        many = torch.from_numpy(np.concatenate([w, np.repeat(w[:1], tiles - len(w), 0)])).cuda()
        got = {k: v.cpu().numpy()[:len(w)] for k, v in P.search(many, bits, n, fast=True).items()}
        assert P.last_kernels() == want
        assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")
    finally:
        P.set_small_call_tiles(before)
