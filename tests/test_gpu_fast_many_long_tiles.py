"""k_fast in 256 threads for launches of many tiles of 1025 to 5120 elements: tiles that end inside a wavefront,
between two and at a batch of a thread's elements, with zeros and crowded ones among them, with the grid of candidates
and without, either side of the rule that chooses it, against the oracle."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches
from test_gpu_fast_pruned import P, rows  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,n,K", [(4, 300, 1025), (2, 1000, 1087), (3, 515, 1280), (5, 400, 2048), (4, 100, 2111),
                                      (4, 1000, 3072), (3, 2000, 4032), (4, 357, 4096), (2, 2500, 4097), (5, 1001, 4608),
                                      (4, 1024, 5056), (5, 160, 5119), (4, 513, 5120)])
def test_many_long_tiles(P, bits, n, K):  # noqa: F811
    import torch
    rng = np.random.default_rng(K)
    w = rows(K, rng)
    w = np.concatenate([w, w[:2] * (rng.random((2, K)) < 0.3), w[:1] * 1e-37, np.zeros_like(w[:1]), np.full_like(w[:1], np.inf),
                        w[:1] * np.nan]).astype(np.float32)
    print(f"[case] bits={bits} n={n} K={K}", flush=True)
    many = torch.from_numpy(np.concatenate([w, np.repeat(w[:1], 2049 - len(w), 0)])).cuda()
    got = {k: v.cpu().numpy()[:len(w)] for k, v in P.search(many, bits, n, fast=True).items()}
    assert P.last_kernels() == "k_fast<256>"
    assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")


@pytest.mark.parametrize("C,K,bits,n,want", [
    (2049, 1025, 4, 1000, 256), (2048, 1025, 4, 1000, 512),           # more than 2048 tiles
    (2049, 2000, 5, 300, 256), (2049, 2000, 6, 300, 512),             # to five bits
    (2049, 2000, 4, 299, 256), (2049, 2000, 5, 166, 256), (2049, 2000, 5, 167, 512)])     # few candidates, or a grid of them
def test_either_side_of_the_rule(P, C, K, bits, n, want):  # noqa: F811
    import torch
    P.search(torch.randn((C, K), device="cuda"), bits, n, fast=True)
    assert P.last_kernels() == f"k_fast<{want}>"
