"""The bin ranking's lists where they hold more patches than there are workgroups for
them, and where most patches have few entries: the result of each patch is that of the
same patch in a strip of the image (a workgroup a patch, no lists), bit for bit."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu

H, W, STRIP = 190, 200, 40


@pytest.mark.parametrize("width,ordinary", [(16.0, 16384 + 8192), (8.0, 2000)])
@pytest.mark.parametrize("t,K", [(1, 16), (2, 3)])
def test_strips(width, ordinary, t, K):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], test_h=H, test_w=W, dict_images=4, w=width, n_dict=3000)
    g = GpuWorkload(wl)
    g.set_mode(cap=0, rerank=0, proj=1, lle_fp64=1)

    def run(img, t):
        h = img.shape[0]
        Q = (h - 4) * (W - 4)
        out = [torch.empty((Q, K), dtype=torch.int32, device="cuda"), torch.empty((Q, K), device="cuda"),
               torch.empty(Q, dtype=torch.int32, device="cuda"), torch.empty(Q, dtype=torch.int32, device="cuda")]
        g.ctx.query(img, h, W, wl.scale, K)
        if t > 1:
            g.ctx.knn_t(t)
        g.ctx.get_results(ids=out[0], d2=out[1], m=out[2], ncand=out[3])
        g.ctx.sync()
        return [o.cpu().numpy() for o in out]

    union = run(g.lr, 1)[3]   # IDs of the unions: each has 1 to L entries
    assert (union > 64).sum() > ordinary and (union <= 64 // wl.L).sum() > 1000
    whole = run(g.lr, t)
    strips = [run(g.lr[r:min(r + STRIP, H)].contiguous(), t) for r in range(0, H - 4, STRIP - 4)]
    for i, a in enumerate(whole):
        assert np.array_equal(a, np.concatenate([s[i] for s in strips])), i
