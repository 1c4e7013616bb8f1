"""The inner product for few rows or few channels (k_linear_rows) at its edges, against
the oracle: the last row count of each tile height (one row of the tile is ones), the
channel tile's remainder, reductions shorter than a step, with every remainder of it and
with more steps than wavefronts, and row counts either side of the switch to k_linear."""
import numpy as np
import pytest

from test_gpu_linear import P, case  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("M,K,N", [(15, 256, 16), (16, 272, 17), (31, 16, 31), (32, 512, 33), (63, 2304, 64),
                                    (64, 144, 65), (126, 80, 5), (127, 128, 32), (1, 4352, 15)])
def test_tile_edges(P, M, K, N, bits):  # noqa: F811
    case(P, M, K, N, bits, seed=M * 7 + K + N + bits, dist="normal" if bits & 1 else "laplace")


@pytest.mark.parametrize("bits", [2, 3, 4, 5, 8])
@pytest.mark.parametrize("M,K,N", [(63, 16, 5473), (32, 528, 4129), (63, 656, 4097), (64, 592, 2753), (126, 560, 2049),
                                   (127, 544, 1665), (63, 2000, 4111)])
def test_tile_edges_of_63_rows_by_32_channels(P, M, K, N, bits):  # noqa: F811
    """The same for the largest workgroups, which calls of few channels do not get."""
    rows = np.unique(np.r_[0, 1, 31, 32, M // 2 - 1:M // 2 + 2, M - 2, M - 1])
    case(P, M, K, N, bits, seed=M + K + N + bits, dist="normal" if bits & 1 else "laplace", check_rows=rows[rows < M])
    assert P.last_kernels() == f"k_linear_rows<{bits}, 2, 32, 2>"


@pytest.mark.parametrize("M,N", [(16, 8192), (31, 8193), (31, 11007)])
def test_either_side_of_three_workgroups_per_cu(P, M, N):  # noqa: F811
    """At 4 bits, 31 rows by 16 channels and the sums apart: other registers past 512 workgroups."""
    case(P, M, 528, N, 4, seed=M + N, check_rows=np.array([0, M // 2, M - 1]))


@pytest.mark.parametrize("M,K,N", [(63, 2064, 8193), (63, 2064, 8177), (63, 2048, 8193)])
def test_eight_bits_by_borrows_and_by_look_ups(P, M, K, N):  # noqa: F811
    """Past 256 workgroups and K = 2048 codes are decoded by borrows."""
    case(P, M, K, N, 8, seed=K + N, check_rows=np.array([0, 31, 32, 62]))
    assert P.last_kernels() == "k_linear_rows<8, 2, 32, 2>"


@pytest.mark.parametrize("extra", range(16, 257, 48))
def test_what_is_left_of_a_step(P, extra):  # noqa: F811
    for M in (9, 20, 40):
        case(P, M, 512 + extra, 40, 4, seed=extra + M)


@pytest.mark.parametrize("M,N", [(64, 14400), (64, 14432)])
def test_either_side_of_the_switch(P, M, N):  # noqa: F811
    """Two tiles of 63 rows by 450 tiles of 32 channels are 900 workgroups: the last call by rows."""
    case(P, M, 64, N, 4, seed=N, check_rows=np.arange(0, M, 9))
