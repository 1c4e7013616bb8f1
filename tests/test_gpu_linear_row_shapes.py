"""The workgroup shapes of k_linear_rows where 63 rows by 32 channels would leave CUs idle, against the
oracle and by the kernels launched: either side of each limit, rows and channels that do not
fill the last tile, reductions shorter than a step and of every remainder of it."""
import pytest

from test_gpu_linear import P, case  # noqa: F401  (P is the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,K,N,tile,mt", [
    (32, 16, 65, 16, 2), (63, 272, 70, 16, 2), (64, 1040, 100, 16, 2), (93, 2048, 129, 16, 2), (94, 512, 65, 16, 2),
    (63, 528, 1365, 32, 1), (125, 1296, 900, 32, 1), (62, 96, 6000, 32, 1),
    (126, 544, 2016, 16, 4), (250, 784, 1001, 16, 4), (249, 528, 1007, 16, 4)])
def test_shapes(P, M, K, N, tile, mt, bits):  # noqa: F811
    case(P, M, K, N, bits, seed=M + K + N + bits, dist="normal" if bits & 1 else "laplace")
    assert P.last_kernels() in (f"k_linear_rows<{bits}, 2, {tile}, {mt}>", f"k_linear_rows<{bits}, 3, {tile}, {mt}>")


@pytest.mark.parametrize("M,K,N,want", [
    (62, 1024, 2048, "16, 2"), (62, 1024, 2049, "32, 1"), (62, 1024, 4096, "32, 1"), (63, 1024, 4080, "16, 4"),
    (63, 1024, 4096, "32, 2"), (62, 512, 8192, "32, 1"), (62, 512, 8193, "32, 2"), (63, 512, 64, "16, 2"), (63, 512, 65, "16, 2"),
    (63, 2304, 64, "16, 2"), (1900, 1024, 64, "16, 2"), (2048, 1024, 64, "32, 1")])
def test_either_side_of_each_limit(P, M, K, N, want):  # noqa: F811
    import torch
    x = torch.zeros((M, K), dtype=torch.int8, device="cuda")
    z = torch.zeros(N * K, dtype=torch.uint8, device="cuda")
    p = torch.ones(N, device="cuda")
    P.linear_i8(x, 1.0, 0.0, z, z, N, 4, p, p)
    assert P.last_kernels() == f"k_linear_rows<4, 2, {want}>"


@pytest.mark.parametrize("M,K,N,bits,acc,want", [
    # 16 channels by 63 rows while the activations are at most 4 MiB, at 8 bits in the folded form always
    (1024, 4096, 230, 4, False, "4, 2, 16, 4"), (1025, 4096, 230, 4, False, "4, 2, 32, 2"), (1024, 4112, 230, 4, False, "4, 2, 32, 2"),
    (3000, 1392, 80, 4, True, "4, 3, 16, 4"), (3000, 4096, 80, 4, True, "4, 3, 32, 2"), (3000, 4096, 80, 2, False, "2, 2, 32, 2"),
    (3000, 4096, 80, 8, False, "8, 2, 16, 4"), (3000, 4096, 80, 8, True, "8, 3, 32, 2")])
def test_activations_that_fit_the_l2(P, M, K, N, bits, acc, want):  # noqa: F811
    import torch
    x = torch.zeros((M, K), dtype=torch.int8, device="cuda")
    z = torch.zeros(N * K, dtype=torch.uint8, device="cuda")
    p = torch.ones(N, device="cuda")
    P.linear_i8(x, 1.0, 0.0, z, z, N, bits, p, p, want_acc=acc)
    assert P.last_kernels() == f"k_linear_rows<{want}>"
