"""The fast search's grid of candidates at its edges, against the oracle: as few candidates as
the grid takes and one less, a last interval of one candidate, of a full step and of almost two, more
candidates between the grid points than its list holds, more within the threshold than it
keeps (equal errors everywhere), and tiles that are not a group of their own.

Whether a tile took the grid is seen in the workspace: it leaves a list of candidates there, whose
first word is their number (192 at most) with the sign bit, in place of a row of values, which
are not negative."""
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


def search(P, tensors, bits, n):
    """The outputs of a fast search, and how many tiles left a list in the workspace."""
    import torch
    tl = P.TensorList([torch.from_numpy(w).cuda() for w in tensors], P.PER_CHANNEL)
    ws = torch.zeros((P.search_list_workspace_bytes(tl, bits, n) + 3) // 4, dtype=torch.int32, device="cuda")
    got = P.search_list(tl, bits, n, ws.view(torch.uint8), P.alloc_search_outputs(tl.n_groups, "cuda"), True)
    assert "k_fast" in P.last_kernels()
    count = ws.bitwise_xor(-2 ** 31)                          # 1 .. 192 in a list's first word
    return {k: v.cpu().numpy() for k, v in got.items()}, int(((count >= 1) & (count <= 192)).sum())


@pytest.mark.parametrize("bits,n,K,pruned", [
    (6, 299, 600, False), (6, 300, 600, True), (4, 512, 130, True), (5, 513, 1030, True), (4, 515, 257, True),
    (2, 1500, 64, True), (4, 1000, 5121, False), (4, 1700, 5121, True), (3, 1024, 700, True), (7, 1025, 2816, True),
    (7, 300, 6000, True), (8, 1500, 4200, True), (5, 2049, 1155, True), (8, 4100, 4200, False), (4, 20000, 600, False),
    (6, 1000, 8193, False), (2, 65535, 600, False), (4, 519, 700, True), (3, 1039, 130, True), (2, 4159, 1100, True)])
def test_fast_search_of_many_candidates(P, bits, n, K, pruned):
    w = rows(K, np.random.default_rng(bits * 1000 + n))
    w = np.concatenate([w, w[:1] * 1e-37, np.zeros_like(w[:1]), np.full_like(w[:1], np.inf), w[:1] * np.nan])
    print(f"[case] bits={bits} n={n} K={K}", flush=True)
    before = P.set_small_call_tiles(0)
    try:
        # 2048 more groups: the look-ups, not the passes of few tiles
        many = np.concatenate([w, np.repeat(w[:1], 2048, 0)])
        got, lists = search(P, [many], bits, n)
        got = {k: v[:len(w)] for k, v in got.items()}
        # rows of equal or crowded magnitudes have no list, Gaussian rows do
        assert lists >= 2048 if pruned else lists == 0
        assert_search_matches(got, R.search(w, bits, n, want_curve=True), f"bits={bits} n={n} K={K}")
    finally:
        P.set_small_call_tiles(before)


@pytest.mark.parametrize("shape,bits,n,without", [
    # threads of a workgroup: 512, 1024, 256, 128; 11 pairs of look-ups a thread, or 20 below 256 workgroups
    ((256, 1500), 4, 805, 804), ((255, 1500), 4, 1463, 1462), ((256, 6000), 4, 1610, 1609), ((513, 600), 6, 300, 299),
    ((1025, 200), 2, 1408, 1407),
    # most candidates: 112 of n sqrt(6e-5 + 2.4e-5 L), and 8000
    ((300, 1500), 4, 7417, 7418), ((300, 1500), 6, 3949, 3950), ((300, 4200), 8, 2008, 2010), ((300, 600), 3, 8000, 8001),
    # at 7 and 8 bits: a round of 512 fewer, or 600 and 1500 candidates, or at 7 bits many tiles
    ((255, 2400), 7, 854, 855), ((255, 2400), 7, 513, 512), ((60, 4200), 8, 1537, 1536),
    ((256, 2400), 7, 600, 599), ((2048, 1500), 7, 300, 299), ((256, 4200), 8, 1500, 1499)])
def test_either_side_of_where_the_grid_is_taken(P, shape, bits, n, without):
    before = P.set_small_call_tiles(0)
    try:
        w = np.random.default_rng(n).laplace(0, 1, shape).astype(np.float32)
        assert search(P, [w], bits, n)[1] > shape[0] // 2
        assert search(P, [w], bits, without)[1] == 0
    finally:
        P.set_small_call_tiles(before)


def test_a_launch_of_tiles_that_are_groups_and_of_parts_of_groups(P):
    rng = np.random.default_rng(8)
    tensors = [rng.standard_normal((1100, 1500)).astype(np.float32), rng.laplace(0, 1, (40, 9000)).astype(np.float32)]
    before = P.set_small_call_tiles(0)
    try:
        got, lists = search(P, tensors, 4, 1700)
        assert P.last_kernels() == "k_fast<1024>" and 1000 <= lists <= 1100
        for w, at in ((tensors[0][:30], 0), (tensors[1], 1100)):
            part = {k: v[at:at + len(w)] for k, v in got.items()}
            assert_search_matches(part, R.search(w, 4, 1700, want_curve=True), f"groups {at}..")
    finally:
        P.set_small_call_tiles(before)
