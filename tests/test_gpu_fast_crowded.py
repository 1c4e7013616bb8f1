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


def full(K, runs, rng):
    """Runs of weights within one bucket, low, high and last, among others."""
    out = []
    for run in runs:
        w = rng.standard_normal(K) * 0.3
        w[0] = top = 2.0
        for at in (0.31, 0.77, 0.99999):
            v = w.copy()
            v[rng.choice(K, run, replace=False)] = top * at * (1 - rng.random(run) * 2.0 ** -14)
            out.append(v)
    return np.stack(out).astype(np.float32)


@pytest.mark.parametrize("bits,n,K,beside", [(4, 300, 200, 600), (3, 1000, 255, 1000), (4, 1000, 300, 0), (2, 700, 1023, 0), (4, 301, 1100, 0),
                                             (4, 1000, 2064, 0), (5, 400, 4096, 0)])
def test_buckets_as_full_as_256_threads_walk(P, bits, n, K, beside):  # noqa: F811
    import torch
    most = max(64, K // 16) * 2
    w = full(K, (65, most - 1, most, min(most + 1, K)), np.random.default_rng(K))
    many = torch.from_numpy(np.concatenate([w, np.repeat(w[:1], 2049, 0)])).cuda()
    more = [torch.randn((20, beside), generator=torch.Generator().manual_seed(1)).cuda()] if beside else []
    print(f"[case] bits={bits} n={n} K={K}", flush=True)
    got = P.search_list(P.TensorList([many] + more, P.PER_CHANNEL), bits, n, fast=True)
    assert P.last_kernels() == "k_fast<256>"
    assert_search_matches({k: v.cpu().numpy()[:len(w)] for k, v in got.items()}, R.search(w, bits, n, want_curve=True),
                          f"bits={bits} n={n} K={K}")
