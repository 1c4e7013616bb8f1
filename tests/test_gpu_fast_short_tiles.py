"""The fast search of many short tiles from 300 candidates on, down to nine elements each, against the oracle, and either
side of the lengths and numbers at which they are k_fast's."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from parity import assert_search_matches
from test_gpu_fast_pruned import P  # noqa: F401  (the module's fixture)
from test_gpu_routes import searched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,n", [(2, 300), (3, 1000), (4, 300), (4, 1000), (4, 3001), (5, 1000)])
def test_short_tiles(P, bits, n):  # noqa: F811
    import torch
    rng = np.random.default_rng(bits + n)
    ws = []
    for K in (9, 10, 15, 16, 17, 18, 31, 33, 47, 63, 64, 65, 111):
        w = rng.standard_normal((180, K)) * np.exp(rng.normal(0, 3, (180, 1)))
        w[:20] *= rng.random((20, K)) < 0.5                    # zeros, whole rows of them among the shortest
        w[20:30] = rng.choice([-1.0, 1.0, 0.25], (10, K))
        w[30] = np.inf
        w[31] *= 1e-38
        ws.append(w.astype(np.float32))
    print(f"[case] bits={bits} n={n}", flush=True)
    got = P.search_list(P.TensorList([torch.from_numpy(w).cuda() for w in ws], P.PER_CHANNEL), bits, n, fast=True)
    assert P.last_kernels() == "k_fast<128>"
    got = {k: v.cpu().numpy() for k, v in got.items()}
    at = 0
    for w in ws:
        part = {k: v[at:at + len(w)] for k, v in got.items()}
        assert_search_matches(part, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={w.shape[1]}")
        at += len(w)


@pytest.mark.parametrize("shapes,bits,n,want", [
    ([(2048, 9)], 4, 300, "k_fast<128>"), ([(2047, 9)], 4, 300, "k_search"), ([(2048, 9)], 4, 299, "k_search"), ([(4096, 8)], 4, 1000, "k_search"),
    ([(2048, 9)], 4, 7417, "k_fast<128>"), ([(2048, 9)], 4, 7419, "k_search"),
    ([(1000, 9), (1047, 55)], 3, 300, "k_search"), ([(1000, 9), (1048, 55)], 3, 300, "k_fast<128>"),
    ([(2048, 64)], 5, 300, "k_fast<128>"), ([(2048, 63)], 5, 999, "k_search"), ([(2048, 9)], 5, 1000, "k_fast<128>"),
    ([(2048, 150)], 6, 1000, "k_fast<128>"), ([(2048, 149)], 6, 1000, "k_search"), ([(2048, 150)], 6, 999, "k_search")])
def test_either_side_of_the_line(P, shapes, bits, n, want):  # noqa: F811
    assert searched(P, shapes, bits, n, fast=True) == want
