"""Fast search of more tiles than one launch of 1024 threads each can take (2^22 and more): a
list of 1024 views of one tensor, whose groups must all come out as the tensor's own."""
import pytest

pytestmark = pytest.mark.gpu


def test_four_million_long_tiles():
    import torch
    from paper_2002_00104_amd import pwlq as P
    C, K, bits, n = 4096, 5121, 2, 3
    g = torch.Generator(device="cuda").manual_seed(1)
    w = torch.randn((C, K), generator=g, device="cuda")
    one = P.search(w, bits, n)
    tl = P.TensorList([w] * 1024 + [w[:1]], 0)
    print("[case] 4 194 305 tiles of 5121", flush=True)
    out = P.search_list(tl, bits, n, fast=True)
    torch.cuda.synchronize()
    assert P.last_kernels() == "k_fast<1024>"
    for name in ("k_star", "p_star", "m", "mse"):
        got = out[name]
        assert torch.equal(got[:-1].view(1024, C), one[name].expand(1024, C)), name
        assert got[-1] == one[name][0]
