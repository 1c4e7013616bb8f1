"""Many short tiles of the fast search in one wavefront each, against the oracle, and either side of the limits."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches
from test_gpu_fast_pruned import P  # noqa: F401  (the module's fixture)
from test_gpu_routes import searched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,n", [(2, 1000), (3, 470), (4, 300), (4, 1000), (2, 500), (3, 2000), (4, 2000)])
def test_one_wavefront(P, bits, n):  # noqa: F811
    import torch
    rng = np.random.default_rng(10 * bits + n)
    ws = []
    for K in (9, 10, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256):
        w = rng.standard_normal((640, K)) * np.exp(rng.normal(0, 3, (640, 1)))
        w[:20] *= rng.random((20, K)) < 0.5                    # zeros
        w[20:30] = rng.choice([-1.0, 1.0, 0.25], (10, K))      # crowded buckets
        w[30:40] = np.exp(rng.normal(0, 6, (10, K)))
        w[40], w[41], w[42, 0] = 0.0, np.inf, 1e30
        w[43] *= 1e-38
        ws.append(w.astype(np.float32))
    print(f"[case] bits={bits} n={n}", flush=True)
    got = P.search_list(P.TensorList([torch.from_numpy(w).cuda() for w in ws], P.PER_CHANNEL), bits, n, fast=True)
    assert P.last_kernels() == "k_fast<64>"
    got = {k: v.cpu().numpy() for k, v in got.items()}
    at = 0
    for w in ws:
        part = {k: v[at:at + 80] for k, v in got.items()}
        assert_search_matches(part, R.search(w[:80], bits, n, want_curve=True), f"bits={bits} n={n} K={w.shape[1]}")
        at += len(w)


@pytest.mark.parametrize("shapes,bits,n,want", [
    ([(8192, 256)], 4, 300, "k_fast<64>"), ([(8191, 256)], 4, 300, "k_fast<128>"), ([(8192, 257)], 4, 300, "k_fast<256>"),
    ([(8192, 256)], 4, 299, "k_fast<128>"), ([(8192, 256)], 4, 2000, "k_fast<64>"), ([(8192, 256)], 4, 2001, "k_fast<128>"),
    ([(8192, 256)], 5, 1000, "k_fast<128>"), ([(4096, 9), (4096, 100)], 2, 500, "k_fast<64>")])
def test_either_side_of_the_limits(P, shapes, bits, n, want):  # noqa: F811
    assert searched(P, shapes, bits, n, fast=True) == want
