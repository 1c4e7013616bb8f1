"""The fast search's grid of candidates at its edges, against the oracle: as few candidates as
the grid takes and one less, a last interval of one candidate and of a full step, more
candidates between the grid points than its list holds, more within the threshold than it
keeps (equal errors everywhere), and tiles that are not a group of their own."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available()
    from paper_2002_00104_amd import pwlq
    return pwlq


def rows(K, rng):
    w = np.stack([rng.standard_normal(K), rng.standard_t(1.2, K), rng.uniform(-1, 1, K),
                  rng.laplace(0, 1, K) * np.where(rng.random(K) < 0.002, 10, 1),
                  rng.choice([-1.0, 1.0, 0.0], K), rng.choice([1.0, 0.3, -0.7], K),
                  np.where(np.arange(K) == 5, 1.0, 0.01 * rng.standard_normal(K)), np.exp(rng.uniform(-30, 0, K))])
    return w.astype(np.float32)


@pytest.mark.parametrize("bits,n,K", [(6, 299, 600), (6, 300, 600), (4, 512, 130), (5, 513, 1030), (4, 515, 257),
                                      (2, 1500, 64), (4, 1000, 5121), (3, 1024, 700), (7, 1025, 2816), (7, 300, 6000), (8, 1500, 4200),
                                      (5, 2049, 1155), (8, 4100, 4200), (4, 20000, 600), (6, 1000, 8193), (2, 65535, 600)])
def test_fast_search_of_many_candidates(P, bits, n, K):
    import torch
    w = rows(K, np.random.default_rng(bits * 1000 + n))
    w = np.concatenate([w, w[:1] * 1e-37, np.zeros_like(w[:1]), np.full_like(w[:1], np.inf), w[:1] * np.nan])
    print(f"[case] bits={bits} n={n} K={K}", flush=True)
    before = P.set_small_call_tiles(0)
    try:
        # 2048 more groups: the look-ups, not the passes of few tiles
        many = np.concatenate([w, np.repeat(w[:1], 2048, 0)])
        got = {k: v[:len(w)].cpu().numpy() for k, v in P.search(torch.from_numpy(many).cuda(), bits, n, fast=True).items()}
        assert "k_fast" in P.last_kernels()
        assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")
    finally:
        P.set_small_call_tiles(before)
