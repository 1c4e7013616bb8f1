"""Selectors and error over lists that hold groups of one tile, of a few and of sixteen and
more in any order of the caller's, and over many tensors of a group or two each; against the
oracle, and the same bits as each tensor alone."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from test_gpu_selectors import MSE_RTOL, P, assert_select_matches  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [
    [(70, 8192), (2, 140000), (5, 64), (3, 30000), (130, 33), (1, 131072), (1, 131073), (2, 8193)],
    [(3, 17), (2, 150000), (64, 40), (1, 122880), (65, 41)],
    [(2, 150000), (1020, 33), (3, 25000), (1, 8192)], [(2, 150000), (1020, 33), (3, 25000), (2, 8192)],
    [(1 + i % 3, 20 + i) for i in range(200)], [(1, 40)] * 130 + [(129, 50)] + [(1, 41)] * 70])
@pytest.mark.parametrize("mode", [0, 1])
def test_lists(P, shapes, mode):  # noqa: F811
    import torch
    rng = np.random.default_rng(len(shapes) + mode)
    ws = [(rng.standard_normal(s) * np.exp(rng.normal(-3, 0.5))).astype(np.float32) for s in shapes]
    dev = [torch.from_numpy(w).cuda() for w in ws]
    print(f"[case] {shapes[:3]} mode={mode}", flush=True)
    tl = P.TensorList(dev, mode)
    for sel in (R.GAUSS_FIT, R.GAUSS_SOLVE, R.LAPLACE_SOLVE):
        p, m = P.select_analytic_list(tl, sel)
        mse = P.mse_list(tl, 4, p, m)
        for i, (w, g) in enumerate(zip(ws, tl.group_offsets)):
            G = w.shape[0] if mode == 0 else 1
            at = slice(g, g + G)
            if i < 8:
                p1, m1 = P.select_analytic(dev[i], sel, mode)
                e1 = P.mse(dev[i], 4, p1, m1, mode)
                assert torch.equal(p[at], p1) and torch.equal(m[at], m1) and torch.equal(mse[at], e1), (sel, w.shape)
            pr, mr = R.select_analytic(w, sel, mode)
            assert_select_matches(p[at].cpu().numpy(), m[at].cpu().numpy(), pr, mr, f"selector {sel} {w.shape}")
            terms = w.shape[1] if mode == 0 else w.size
            np.testing.assert_allclose(mse[at].cpu().numpy(),
                                       R.mse(w, 4, p[at].cpu().numpy(), m[at].cpu().numpy(), mode),
                                       rtol=max(MSE_RTOL, terms * 2.0 ** -53))
