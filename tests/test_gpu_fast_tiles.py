"""Fast search at the edges of its tile sizes, against the oracle: the shortest tiles it
takes, the lengths where a launch changes its workgroup, tiles cut from a longer group, values
in the few octaves of a bell and in the many of a heavy tail, pruned and equal weights."""
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
    w = np.stack([rng.standard_normal(K), rng.standard_t(1.2, K), rng.laplace(0, 1, K),
                  rng.standard_normal(K) * (rng.random(K) < 0.1), np.full(K, 0.37) * np.sign(rng.standard_normal(K)),
                  np.exp(rng.uniform(-30, 0, K))])
    return w.astype(np.float32)


@pytest.mark.parametrize("bits,n,lengths", [(4, 100, (119, 120, 121, 255, 256, 257, 1023, 1024, 1025)),
                                            (4, 1000, (64, 120, 2816, 2817, 5120, 5121)),
                                            (2, 60, (23, 24, 25, 8191, 8192, 8193)),
                                            (3, 2000, (56, 57, 1500, 16385)), (8, 130, (2039, 2040, 2041, 8200))])
def test_fast_search_at_the_edges_of_its_tiles(P, bits, n, lengths):
    import torch
    rng = np.random.default_rng(bits * 1000 + n)
    before = P.set_small_call_tiles(0)
    try:
        for K in lengths:
            w = rows(K, rng)
            print(f"[case] bits={bits} n={n} K={K}", flush=True)
            got = P.search(torch.from_numpy(w).cuda(), bits, n, fast=True)
            got = {k: v.cpu().numpy() for k, v in got.items()}
            assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")
    finally:
        P.set_small_call_tiles(before)


@pytest.mark.parametrize("bits,n,K", [(4, 300, 8192), (3, 1000, 2000), (8, 130, 4300)])
def test_full_buckets_and_tiny_scales(P, bits, n, K):
    """Runs of 62 to K/16 weights within one bucket (walked three and then four at a time; from
    K/16 on a tile is evaluated element by element), also in the last bucket, and scales down
    to where n / max|w| overflows binary32 (below about 3e-36 for n = 1000)."""
    import torch
    rng = np.random.default_rng(bits * 1000 + K)
    base = rng.standard_normal(K)
    out = []
    for run in (62, 63, 64, 65, K // 16 - 1, K // 16, K // 16 + 1):
        w = base.copy()
        top = np.abs(w).max()
        for at in (0.31, 0.77, 0.99999):
            i = rng.choice(K, run, replace=False)
            w[i] = top * at * (1 - rng.random(run) * 2.0 ** -14)
        out.append(w)
    out += [base * s for s in (1e-30, 4e-36, 1e-36, 1e-37, 1e-38)]
    w = np.stack(out).astype(np.float32)
    before = P.set_small_call_tiles(0)
    try:
        print(f"[case] bits={bits} n={n} K={K}", flush=True)
        got = {k: v.cpu().numpy() for k, v in P.search(torch.from_numpy(w).cuda(), bits, n, fast=True).items()}
        assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")
    finally:
        P.set_small_call_tiles(before)


@pytest.mark.parametrize("bits,n", [(4, 100), (5, 700)])
def test_where_the_wavefronts_of_1024_threads_have_all_of_their_elements(P, bits, n):
    """Eight elements to a thread: from 7232 on the first wavefront has all of them, from 8192 on the last; short tiles beside
    them; a wavefront with zeros and one without."""
    import torch
    rng = np.random.default_rng(n)
    ws = []
    for K in (7231, 7232, 7233, 7295, 7296, 8128, 8191, 8192, 600, 2049):
        w = rows(K, rng)
        w[2, 64:128] = 0.0
        ws.append(w)
    print(f"[case] bits={bits} n={n}", flush=True)
    before = P.set_small_call_tiles(0)
    try:
        got = P.search_list(P.TensorList([torch.from_numpy(w).cuda() for w in ws], P.PER_CHANNEL), bits, n, fast=True)
        assert P.last_kernels() == "k_fast<1024>"
    finally:
        P.set_small_call_tiles(before)
    got, at = {k: v.cpu().numpy() for k, v in got.items()}, 0
    for w in ws:
        part = {k: v[at:at + len(w)] for k, v in got.items()}
        assert_search_matches(part, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={w.shape[1]}")
        at += len(w)
