"""Calls between a query and the calls that use its results."""
import pytest

import synthdata

pytestmark = pytest.mark.gpu


def _workload(**kw):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    base = dict(dict_images=4, dict_hr=96, n_dict=2000, L=4, k=6, w=40.0, test_h=40, test_w=44, cap=16)
    return torch, GpuWorkload(synthdata.scaled(synthdata.WORKLOADS["diff"], **{**base, **kw}))


def test_features_between_query_and_image():
    """Features of another image without their means leave the query's means."""
    torch, g = _workload()
    ref, out = torch.empty((80, 88), device="cuda"), torch.empty((80, 88), device="cuda")
    other = torch.from_numpy(synthdata.fractal_voronoi_image(5, 90, 70)).cuda()
    feat = torch.empty((86 * 66, g.D), device="cuda")
    g.set_mode(cap=16, rerank=0, proj=1, lle_fp64=1)
    for hr, between in ((ref, False), (out, True)):
        g.ctx.query(g.lr, g.h, g.w, 2, 4)
        g.ctx.lle_weights(1e-3)
        if between:
            g.ctx.features(other, 90, 70, g.wl.feat_mode, feat)
        g.ctx.reconstruct(hr)
    g.ctx.sync()
    assert torch.equal(ref, out)
