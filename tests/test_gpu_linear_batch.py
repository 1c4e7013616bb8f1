"""A row of y does not depend on the rows beside it: the same activations as the only rows of
a call, among a few, among hundreds and among thousands give the same bits, in both forms, whichever
kernels the calls take: with y alone k_linear_rows, k_linear_split, k_linear and k_linear_wide."""
import numpy as np
import pytest

from test_gpu_linear import P  # noqa: F401  (the module's fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4, 5, 8])
@pytest.mark.parametrize("want_acc", [False, True])
def test_rows_are_the_same_bits_in_every_batch(P, bits, want_acc):  # noqa: F811
    import torch
    K, N = 640, 2050
    rng = np.random.default_rng(bits)
    w = torch.from_numpy(rng.laplace(0, 0.02, (N, K)).astype(np.float32)).cuda()
    s = P.search(w, bits, 100, fast=True)
    pc, pf, _ = P.quantize_packed(w, bits, s["p_star"], s["m"], want_w_hat=False)
    x = torch.from_numpy(rng.integers(-128, 128, (2600, K)).astype(np.int8)).cuda()

    kernels = set()

    def rows(M):
        y = P.linear_i8(x[:M].contiguous(), 0.0123, -0.57, pc, pf, N, bits, s["p_star"], s["m"], want_acc=want_acc)[0]
        kernels.add(P.last_kernels().split("<")[0])
        return y

    whole = rows(2600)
    for M in (1, 8, 31, 63, 64, 200, 700, 1100, 1500):
        print(f"[case] bits={bits} acc={want_acc} M={M}", flush=True)
        differ = int((rows(M).view(torch.int32) != whole[:M].view(torch.int32)).sum())
        assert differ == 0, f"{differ} of {M * N} values differ between {M} and 2600 rows"
    assert kernels == {"k_linear_rows", "k_linear"} | (set() if want_acc else {"k_linear_split", "k_linear_wide"})
