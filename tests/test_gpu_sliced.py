"""Searches of few tiles, whose elements are cut into slices: calls of one to eight slices,
candidate blocks that do not fill a workgroup, tiles from a longer group, with and without
the order by candidate, and a list of unequal tensors; against the oracle."""
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


def check(P, ws, bits, n, mode):
    import torch
    tl = P.TensorList([torch.from_numpy(w).cuda() for w in ws], mode)
    got = {k: v.cpu().numpy() for k, v in P.search_list(tl, bits, n).items()}
    for w, g in zip(ws, tl.group_offsets):
        G = w.shape[0] if mode == 0 else 1
        assert_search_matches({k: v[g:g + G] for k, v in got.items()}, R.search(w, bits, n, mode, want_curve=True),
                              f"{w.shape} n={n} mode={mode}")


@pytest.mark.parametrize("C,K,n,mode", [(3, 255, 64, 0), (3, 256, 64, 0), (5, 2047, 333, 0), (6, 2048, 1000, 0),
                                        (40, 1030, 100, 0), (130, 1025, 1025, 0), (2, 20000, 90, 0),
                                        (9, 3001, 2049, 0), (3, 8193, 65, 1), (4, 5000, 2000, 1), (1, 100000, 40, 1)])
def test_few_tiles(P, C, K, n, mode):
    rng = np.random.default_rng(C * K + n)
    w = (rng.standard_t(3, (C, K)) * 0.02).astype(np.float32)
    before = P.set_small_call_tiles(0)
    try:
        for bits in (2, 4, 7):
            print(f"[case] {C}x{K} n={n} mode={mode} bits={bits}", flush=True)
            check(P, [w], bits, n, mode)
    finally:
        P.set_small_call_tiles(before)


def test_list_of_unequal_tensors(P):
    rng = np.random.default_rng(5)
    ws = [rng.laplace(0, 0.1, s).astype(np.float32) for s in ((2, 9000), (7, 1500), (20, 300), (30, 65), (16, 17), (8, 9))]
    for mode in (0, 1):
        check(P, ws, 4, 200, mode)
