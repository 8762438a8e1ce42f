"""An image with enough patches that those with more entries than a window of
the bin ranking are listed first and the longest taken in shares: the result of
each patch is that of the same patch in a strip of the image (too few patches
for a list), bit for bit. Bins of a few entries, of thousands (a share or a few
a patch), of nearly every row (more shares than the list holds: the other
patches take their turn) and flat patches (equal distances go by ID)."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu

CASES = [dict(w=4.0, n_dict=3000), dict(w=64.0, n_dict=6000), dict(w=2000.0, n_dict=2500), dict(amp=0.0, n_dict=6000)]


@pytest.mark.parametrize("kw", CASES)
@pytest.mark.parametrize("t,K", [(1, 16), (2, 5)])
def test_strips(kw, t, K):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    h, w = 100, 110
    wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], test_h=h, test_w=w, dict_images=4, **kw)
    g = GpuWorkload(wl)
    g.set_mode(cap=0, rerank=0, proj=1, lle_fp64=1)
    lr = g.lr

    def run(img):
        Q = (img.shape[0] - 4) * (img.shape[1] - 4)
        out = dict(ids=torch.empty((Q, K), dtype=torch.int32, device="cuda"), d2=torch.empty((Q, K), device="cuda"),
                   m=torch.empty(Q, dtype=torch.int32, device="cuda"), n=torch.empty(Q, dtype=torch.int32, device="cuda"))
        g.ctx.query(img, img.shape[0], img.shape[1], wl.scale, K)
        if t > 1:
            g.ctx.knn_t(t)
        g.ctx.lle_weights(wl.lam)
        g.ctx.get_results(out["ids"], out["d2"], out["m"], None, out["n"])
        g.ctx.sync()
        return {k: v.cpu().numpy() for k, v in out.items()}

    assert (h - 4) * (w - 4) >= 8192
    whole = run(lr)
    cut = 60
    strips = [run(lr[:cut].contiguous()), run(lr[cut - 4:].contiguous())]
    for k in whole:
        both = np.concatenate([s[k] for s in strips])
        assert np.array_equal(whole[k], both), k
    assert whole["n"].max() > (0 if kw.get("w") == 4.0 else 100)
