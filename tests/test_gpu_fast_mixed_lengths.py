"""Calls of the fast search with tiles of very different lengths: which launches the short ones are in, either side of the
numbers that decide it, how the passes beside the look-ups are cut into units, and results against the oracle."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches
from test_gpu_fast_pruned import P  # noqa: F401  (the module's fixture)
from test_gpu_routes import searched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,bits,n,want", [
    # short tiles behind a few that get 1024 or 512 threads: from 2048 on in a launch of their own, below in passes
    ([(500, 8000), (2100, 9)], 4, 1000, "k_fast<1024> k_fast<128>"), ([(500, 8000), (2047, 9)], 4, 1000, "k_fast<1024> k_search"),
    ([(500, 8000), (2048, 9)], 4, 1000, "k_fast<1024> k_fast<128>"), ([(10, 5121), (2048, 250)], 4, 100, "k_fast<1024> k_fast<128>"),
    ([(10, 5121), (2047, 250)], 4, 100, "k_fast<1024>"), ([(20, 2000), (2048, 600)], 6, 500, "k_fast<512> k_fast<256>"),
    ([(20, 2000), (2047, 600)], 6, 500, "k_fast<512>"),
    ([(30, 6000), (1500, 300), (900, 9)], 4, 1000, "k_fast<1024> k_fast<256>"),
    # behind tiles that get 256: only those that get fewer, from 6144 on where they look up a grid, and from 8192
    ([(900, 2000), (2100, 9)], 4, 1000, "k_fast<256>"), ([(10, 1025), (6143, 50)], 4, 1000, "k_fast<256>"),
    ([(10, 1025), (6144, 50)], 4, 1000, "k_fast<512> k_fast<128>"), ([(10, 600), (8191, 50)], 2, 300, "k_fast<256>"),
    ([(10, 600), (8192, 50)], 2, 300, "k_fast<256> k_fast<64>"), ([(10, 1025), (9000, 300)], 4, 1000, "k_fast<256>"),
    # nine weights to a tile, alone or nearly so
    ([(5461, 9)], 3, 469, "k_fast<128>"), ([(5462, 9)], 3, 469, "k_search"), ([(5462, 9)], 3, 470, "k_fast<128>"),
    ([(3000, 9), (2462, 10)], 3, 469, "k_fast<128>"), ([(16384, 9)], 2, 500, "k_fast<64>"), ([(16385, 9)], 2, 500, "k_search"),
    ([(16385, 9)], 2, 704, "k_fast<64>"), ([(12288, 9)], 5, 1000, "k_fast<128>"), ([(12289, 9)], 5, 1024, "k_search"),
    ([(12289, 9)], 5, 1025, "k_fast<128>")])
def test_launches(P, shapes, bits, n, want):  # noqa: F811
    assert searched(P, shapes, bits, n, fast=True) == want


@pytest.mark.parametrize("bits,n,shapes", [(4, 1000, [(40, 8000), (2100, 9)]), (4, 100, [(3, 9000), (2060, 250), (30, 70)]),
                                           (3, 600, [(20, 1100), (15, 400), (6150, 31)]), (6, 400, [(9, 3000), (2050, 600), (40, 100)])])
def test_results(P, bits, n, shapes):  # noqa: F811
    import torch
    rng = np.random.default_rng(n)
    ws = [(rng.laplace(0, 1, s) * np.exp(rng.normal(0, 2, (s[0], 1)))).astype(np.float32) for s in shapes]
    print(f"[case] bits={bits} n={n} {shapes}", flush=True)
    got = P.search_list(P.TensorList([torch.from_numpy(w).cuda() for w in ws], P.PER_CHANNEL), bits, n, fast=True)
    assert len(P.last_kernels().split()) > 1
    got, at = {k: v.cpu().numpy() for k, v in got.items()}, 0
    for w in ws:
        some = min(len(w), 60)
        part = {k: v[at:at + some] for k, v in got.items()}
        assert_search_matches(part, R.search(w[:some], bits, n, want_curve=True), f"bits={bits} n={n} {w.shape}")
        at += len(w)
