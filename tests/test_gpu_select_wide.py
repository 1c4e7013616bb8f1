"""Selectors and error of groups of many tiles (one wavefront per group from 16 tiles on),
of few, and of both in one call; and of more tensors than the kernels' arguments carry;
against the oracle."""
import numpy as np
import pytest

from oracle import pwlq_ref as R
from test_gpu_selectors import MSE_RTOL, P, assert_select_matches  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(1, 8192 * 15)], [(1, 8192 * 15 + 1)], [(3, 50000), (700, 8192), (5, 33)],
                                    [(2, 16385), (64, 9)], [(4, 40 + i) for i in range(56)],
                                    [(4, 40 + i) for i in range(57)], [(2, 140000)] + [(3, 17)] * 60])
@pytest.mark.parametrize("mode", [0, 1])
def test_lists(P, shapes, mode):  # noqa: F811
    import torch
    rng = np.random.default_rng(len(shapes) + mode)
    ws = [(rng.standard_normal(s) * np.exp(rng.normal(-3, 0.5))).astype(np.float32) for s in shapes]
    print(f"[case] {shapes[:3]} mode={mode}", flush=True)
    tl = P.TensorList([torch.from_numpy(w).cuda() for w in ws], mode)
    for sel in (R.GAUSS_FIT, R.GAUSS_SOLVE, R.LAPLACE_SOLVE):
        p, m = P.select_analytic_list(tl, sel)
        mse = P.mse_list(tl, 4, p, m)
        p, m, mse = (v.cpu().numpy() for v in (p, m, mse))
        for w, g in zip(ws, tl.group_offsets):
            G = w.shape[0] if mode == 0 else 1
            pr, mr = R.select_analytic(w, sel, mode)
            assert_select_matches(p[g:g + G], m[g:g + G], pr, mr, f"selector {sel} {w.shape}")
            # the oracle adds a group's positive terms one after the other: its own sum is
            # within (terms) * 2^-53 of the exact one, which passes 1e-12 from 9000 terms on
            terms = w.shape[1] if mode == 0 else w.size
            np.testing.assert_allclose(mse[g:g + G], R.mse(w, 4, p[g:g + G], m[g:g + G], mode),
                                       rtol=max(MSE_RTOL, terms * 2.0 ** -53))
