"""The inner product in tiles of 256 rows by 128 channels (k_linear_wide) at its edges, against the oracle:
every bit width, reductions that end in a step of 128 at each of its eight pieces or before the first whole one,
remainders of the row and of the channel tile, rows of y that are no whole vectors or start between two, and the
calls either side of the limits of the rule that chooses it."""
import numpy as np
import pytest

from test_gpu_linear import P, case  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 80, 112, 128, 144, 208, 256, 272, 304, 384, 480, 512, 1120])
def test_steps(P, K):  # noqa: F811
    for bits in range(2, 9):
        case(P, 70, K, 16520 - bits, bits, seed=K + bits, check_rows=[0, 15, 16, 63, 64, 69])
        # (case ends with the call of y alone)
        assert P.last_kernels() == f"k_linear_wide<{bits}>"


@pytest.mark.parametrize("M,N", [(65, 16385), (127, 16511), (128, 16512), (255, 16513), (256, 16386), (257, 8193), (321, 8320),
                                 (512, 8321), (513, 5505), (1025, 3326), (4097, 904)])
def test_tile_edges(P, M, N):  # noqa: F811
    rows = np.unique([r for r in (0, 15, 16, 63, 64, 127, 128, 255, 256, 319, 320, 511, 512, M - 2, M - 1) if r < M])
    for bits in (3, 4, 8):
        case(P, M, 400, N, bits, seed=M + N + bits, dist="normal", check_rows=rows)
        assert P.last_kernels() == f"k_linear_wide<{bits}>"


def test_y_between_vectors(P):  # noqa: F811
    import torch
    M, K, N, bits = 300, 272, 8400, 4
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(-128, 128, (M, K), generator=g, device="cuda").to(torch.int8)
    c, f = (torch.randint(0, 256, (N * K * b // 8,), generator=g, device="cuda").to(torch.uint8) for b in (bits, 1))
    p = torch.rand(N, generator=g, device="cuda") + 0.1
    want, _ = P.linear_i8(x, 0.01, -0.3, c, f, N, bits, p, p + 1)
    room = torch.full((M * N + 8,), 7.0, device="cuda")
    got = room[1:1 + M * N].view(M, N)
    P.linear_i8(x, 0.01, -0.3, c, f, N, bits, p, p + 1, out=(got, None))
    assert P.last_kernels() == "k_linear_wide<4>"
    assert torch.equal(got, want)
    assert room[0] == 7.0 and bool((room[1 + M * N:] == 7.0).all())


@pytest.mark.parametrize("M,K,N,want", [
    (65, 336, 16400, "k_linear_wide<4>"), (64, 336, 16400, "k_linear<4, 2>"),            # a quarter of a tile's rows
    (2049, 336, 1408, "k_linear<4, 2>"), (2305, 336, 1280, "k_linear_wide<4>"),           # 99 and 100 tiles
    (128, 1024, 16384, "k_linear_split<4>"), (128, 1024, 16385, "k_linear_wide<4>"),      # 128 and 129
    # by the estimate: y in short reductions, few tiles in a second pass
    (4096, 4096, 4096, "k_linear_wide<4>"), (4096, 64, 4096, "k_linear<4, 2>"), (4096, 256, 11008, "k_linear<4, 2>"),
    (2048, 4096, 1600, "k_linear<4, 2>"), (4096, 8192, 1000, "k_linear<4, 2>"),
    (1721, 7968, 6440, "k_linear_wide<4>"),
    # rows of y that are no whole vectors, in one pass
    (1072, 16, 3782, "k_linear<4, 2>"), (1072, 16, 3784, "k_linear_wide<4>"), (1183, 592, 2977, "k_linear<4, 2>"),
    (2791, 32, 1719, "k_linear<4, 2>"), (2791, 32, 1720, "k_linear_wide<4>")])
def test_rule(P, M, K, N, want):  # noqa: F811
    import torch
    x = torch.zeros((M, K), dtype=torch.int8, device="cuda")
    z = torch.zeros(N * K, dtype=torch.uint8, device="cuda")
    p = torch.ones(N, device="cuda")
    P.linear_i8(x, 1.0, 0.0, z, z, N, 4, p, p)
    assert P.last_kernels() == want
