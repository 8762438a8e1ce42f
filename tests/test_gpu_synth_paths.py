"""Synthesis and blend of one image: small images write their patches out and
sum them per pixel, larger ones (and every image of a batch) sum tiles of
patch rows and columns. Both give the same bits: images around the tile edges
(40 patch columns to x2, 16 from x3 on; 8 rows), each alone and in a batch, and
one image on each side of the line between the two forms."""
import pytest

import synthdata

pytestmark = pytest.mark.gpu

SIZES = {1: [(12, 44), (13, 45), (21, 90)], 2: [(12, 44), (14, 49), (30, 131)], 3: [(12, 20), (13, 21), (30, 45)],
         4: [(11, 20), (21, 38)]}
# patch rows and columns that cut into just below and just above 200 tiles
LARGE = {2: [(4 + 8 * 39, 4 + 40 * 5), (4 + 8 * 40, 4 + 40 * 5)], 3: [(4 + 8 * 19, 4 + 16 * 10 + 1)]}


@pytest.mark.parametrize("scale", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [3, 12])
def test_written_out_equals_tiled(scale, K):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["diff"], dict_images=8, dict_hr=128, n_dict=5000, L=8, k=8, test_h=16,
                          test_w=16, scale=scale, cap=24)
    g = GpuWorkload(wl)
    sizes = SIZES[scale] + (LARGE.get(scale, []) if K == 3 else [])
    lrs = [torch.from_numpy(synthdata.fractal_voronoi_image(synthdata.SEED_BASE + 9000 + i, h, w)).cuda()
           for i, (h, w) in enumerate(sizes)]
    outs = [torch.empty((scale * h, scale * w), device="cuda") for h, w in sizes]
    single = []
    covered = 0
    for lr in lrs:
        out = torch.empty((scale * lr.shape[0], scale * lr.shape[1]), device="cuda")
        g.zoom(lr=lr, K=K, out=out)
        m = g.results(K=K)["m"]
        covered += int((m > 0).any()) + int((m == 0).any())
        single.append(out)
    assert covered >= len(lrs), "patches with and without neighbours"
    g.ctx.run_batch(lrs, outs, [scale] * len(lrs), K, wl.lam, 0, wl.sigma_s, wl.sigma_r)
    g.ctx.sync()
    for a, b, size in zip(single, outs, sizes):
        assert torch.equal(a, b), size
