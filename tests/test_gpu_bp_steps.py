"""Where the steps of a back-projection call read and write: any number of steps
in one call gives the bits of as many calls of one step, with an odd and an even
number, kept for the adjoint or not, alone and in a batch, on images around the
edges of the LR error's tiles (8 x 32)."""
import pytest

import synthdata

pytestmark = pytest.mark.gpu

SIZES = [(9, 33), (16, 64), (5, 7), (41, 95)]


@pytest.mark.parametrize("scale", [1, 2, 3, 4])
def test_steps(scale):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["diff"], dict_images=8, dict_hr=128, n_dict=3000, L=4, k=8, test_h=16,
                          test_w=16, scale=scale, cap=24)
    g = GpuWorkload(wl)
    sig = (wl.sigma_s, wl.sigma_r)
    lrs = [torch.from_numpy(synthdata.fractal_voronoi_image(synthdata.SEED_BASE + 9500 + i, h, w)).cuda()
           for i, (h, w) in enumerate(SIZES)]
    want = {T: [] for T in range(5)}
    for lr, (h, w) in zip(lrs, SIZES):
        g.ctx.query(lr, h, w, scale, 3)
        g.ctx.lle_weights(wl.lam)
        start = torch.empty((scale * h, scale * w), device="cuda")
        g.ctx.reconstruct(start)
        one = start.clone()
        for T in range(5):
            if T:
                g.ctx.backproject_lr(one, lr, h, w, scale, 1, *sig)
            got = start.clone()
            g.ctx.backproject_lr(got, lr, h, w, scale, T, *sig)
            kept = torch.empty_like(start)
            g.ctx.query(lr, h, w, scale, 3)
            g.ctx.lle_weights(wl.lam)
            g.ctx.reconstruct(kept)
            g.ctx.backproject(kept, T, *sig)
            g.ctx.sync()
            assert torch.equal(got, one) and torch.equal(kept, one), (T, h, w)
            assert T == 0 or not torch.equal(one, start)
            want[T].append(one.clone())
    for T in range(5):
        outs = [torch.empty_like(x) for x in want[T]]
        g.ctx.run_batch(lrs, outs, [scale] * len(lrs), 3, wl.lam, T, *sig)
        g.ctx.sync()
        for a, b, size in zip(want[T], outs, SIZES):
            assert torch.equal(a, b), (T, size)
