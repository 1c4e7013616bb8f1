"""The inner product for tiles that do not fill the chip (k_linear_split) at its edges, against
the oracle: the shortest reduction, halves of an even and of an odd number of steps, remainders of the
row tile (128) and of the channel tile (64), reductions that it leaves to k_linear, and the last
number of workgroups (384) that it takes."""
import numpy as np
import pytest

from test_gpu_linear import P, case  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4, 6, 8])
@pytest.mark.parametrize("M,K,N", [(1025, 512, 1729), (1023, 640, 1728), (768, 768, 2497), (897, 896, 2495),
                                   (250, 1024, 7297), (1025, 528, 1729), (1025, 448, 1729),
                                   (768, 512, 4096), (768, 512, 4097)])
def test_tile_edges(P, M, K, N, bits):  # noqa: F811
    rows = np.unique(np.r_[0:M:61, 31, 32, 63, 64, 127, 128, M - 2, M - 1])
    case(P, M, K, N, bits, seed=M * 7 + K + N + bits, dist="normal" if bits & 1 else "laplace", check_rows=rows)


@pytest.mark.parametrize("M,K,N", [(64, 1024, 8321), (64, 1152, 11008), (250, 1152, 8321), (250, 2176, 2113)])
def test_eight_bits_either_side_of_the_longest_reduction_by_borrows(P, M, K, N):  # noqa: F811
    """Weights are decoded by borrows up to K = 1024 and by look-ups beyond."""
    case(P, M, K, N, 8, seed=M + K + N, check_rows=np.unique(np.r_[0:M:31, M - 1]))
    assert P.last_kernels() in ("k_linear_split<8>", "k_linear_rows<8, 2, 32, 2>")
