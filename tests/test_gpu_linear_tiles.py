"""k_linear itself against the oracle, at sizes that k_linear_rows, k_linear_split and k_linear_wide leave
to it: every bit width, reductions of one to six steps of 64 whose last step holds one to four
pieces of 16, and remainders of the row tile (256, or 192 with the sums apart) and of the
channel tile (64)."""
import numpy as np
import pytest

from test_gpu_linear import P, case  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 32, 48, 64, 80, 96, 112, 128, 160, 176, 192, 240, 256, 272, 304, 352, 368, 400, 1040])
def test_steps(P, K):  # noqa: F811
    import torch
    M, N = 1025, 1761
    rows = np.unique(np.r_[0:M:97, 31, 191, 192, 255, 256, M - 1])
    for bits in range(2, 9):
        case(P, M, K, N, bits, seed=K + bits, dist="normal" if bits & 1 else "laplace", check_rows=rows)
        assert P.last_kernels() == f"k_linear<{bits}, 2>"
    z = torch.zeros(N * K, dtype=torch.uint8, device="cuda")
    p = torch.ones(N, device="cuda")
    P.linear_i8(torch.zeros((M, K), dtype=torch.int8, device="cuda"), 1.0, 0.0, z, z, N, 8, p, p, want_acc=True)
    assert P.last_kernels() == "k_linear<8, 3>"


@pytest.mark.parametrize("M,N", [(1728, 1088), (1729, 1089), (1792, 1025), (2049, 1100), (64, 30000)])
def test_tile_edges(P, M, N):  # noqa: F811
    rows = np.unique([r for r in [*range(0, M, 131), 191, 192, 255, 256, M - 1] if r < M])
    for bits in (3, 4, 7):
        case(P, M, 336, N, bits, seed=M + N + bits, check_rows=rows)
        assert P.last_kernels() == f"k_linear<{bits}, 2>"
