"""The adjoint of the back-projection iterations on images around its tiles' edges
(16 or 8 LR and 32 HR places a side), at every zoom factor, with the smallest
and largest radius of the bilateral filter and on both sides of the line between
the two tile sizes (5, 6), with and without the range weight: gradients of the
residual patches and of lambda against the FP64 oracle, at the bar of the other
gradient tests (1e-4 relative)."""
import math

import numpy as np
import pytest

import synthdata
from oracle import backward as obw
from oracle import imaging, pipeline

pytestmark = pytest.mark.gpu

REL = 1e-4


@pytest.mark.parametrize("scale,H,W,sigma_s,sigma_r", [
    (1, 33, 47, 2.0, 0.1), (1, 16, 65, 0.3, 0.1), (2, 66, 34, 1.6, 0.1), (2, 62, 68, 2.66, 0.1), (2, 32, 64, 1.7, math.inf),
    (3, 51, 99, 2.6, 0.1), (3, 48, 24, 0.3, 0.1), (4, 68, 36, 2.66, 0.1), (4, 32, 100, 1.5, math.inf)])
def test_gradients(scale, H, W, sigma_s, sigma_r):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["diff"], bp_iters=2, sigma_s=sigma_s, sigma_r=sigma_r, test_h=H, test_w=W,
                          dict_images=6, dict_hr=120, n_dict=3000, L=8, k=4, w=32.0, K=5, scale=scale)
    g = GpuWorkload(wl)
    g.set_mode(cap=0, rerank=0, proj=1, lle_fp64=1)
    pre = pipeline.prepare(wl.dictionary_images(), wl.positions(), scale, wl.feat_mode, wl.L, wl.k, wl.w, wl.hash_seed)
    lr = imaging.degrade(wl.test_image().astype(np.float64), scale)
    rec = obw.forward(pre, lr, scale, wl.K, wl.lam, 2, sigma_s, sigma_r, cap=0)
    g.forward_record(g.lr, wl.lam)
    g_out = np.random.default_rng(3).standard_normal(rec.out.shape) * 1e-3
    want, want_lam = obw.backward(rec, pre, g_out)
    g_resid = torch.empty_like(g.resid)
    g_lambda = torch.empty(1, dtype=torch.float32, device="cuda")
    g.ctx.backward(torch.from_numpy(g_out.astype(np.float32)).cuda(), g_resid, g_lambda)
    got = g_resid.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(want) > 0
    assert np.linalg.norm(got - want) <= REL * np.linalg.norm(want)
    assert abs(float(g_lambda.item()) - want_lam) <= REL * abs(want_lam) + 1e-12
