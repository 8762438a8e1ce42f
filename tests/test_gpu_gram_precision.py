"""The Gram matrices that a query leaves, where the precision of the solve changes
between calls: the weights and the gradient of lambda are those of that precision,
whatever was formed before. lambda = 0.1 bounds the condition number by 11: fp32
systems are within (D + 48) 2^-24 11 of FP64 ones."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu

LAM = 0.1


def test_precision_changes():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    g = GpuWorkload(synthdata.scaled(synthdata.WORKLOADS["diff"], dict_images=8, dict_hr=128, n_dict=5000, L=8, k=6,
                                     w=40.0, test_h=40, test_w=44, cap=24))
    K, Q, ctx = 5, g.Q, g.ctx
    w = torch.empty((Q, K), device="cuda")
    out = torch.empty((2 * g.h, 2 * g.w), device="cuda")
    grad = torch.from_numpy(np.random.default_rng(0).standard_normal((2 * g.h, 2 * g.w)).astype(np.float32)).cuda()
    g_resid, g_lam = torch.empty_like(g.resid), torch.empty(1, device="cuda")

    def opts(fp64):
        ctx.set_query_opts(cap=24, rerank=0, proj=1, lle_fp64=fp64)

    def weights():
        ctx.lle_weights(LAM)
        ctx.get_results(w=w)
        ctx.sync()
        return w.cpu().numpy().astype(np.float64)

    def gradient():
        ctx.reconstruct(out)
        ctx.backward(grad, g_resid, g_lam)
        ctx.sync()
        return float(g_lam)

    ref = {}
    for p in (0, 1):
        opts(p)
        ctx.query(g.lr, g.h, g.w, 2, K)
        ref[p] = weights()
        if p == 1:
            lam_ref = gradient()
    tol = (g.D + 48) * 2.0 ** -24 * (1 + 1 / LAM) * np.abs(ref[1]).max()
    assert np.abs(ref[0] - ref[1]).max() <= tol
    for first in (0, 1):
        opts(first)
        ctx.query(g.lr, g.h, g.w, 2, K)
        for p in (1 - first, first, 1 - first, 1 - first, first):
            opts(p)
            got = weights()
            assert np.abs(got - ref[p]).max() <= tol, (first, p)
            assert abs(gradient() - lam_ref) <= 1e-3 * abs(lam_ref), (first, p)
    # all matches between them, which takes the neighbours of the last search as they stand
    opts(1)
    ctx.query(g.lr, g.h, g.w, 2, K)
    opts(0)
    weights()
    opts(1)
    ctx.lle_all(LAM)
    assert np.array_equal(weights(), ref[1])
