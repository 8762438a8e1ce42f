"""Synthesis and blend of images of few tiles, a workgroup a row of LR cells of a
tile's region: bitwise the whole tiles' sums (a batch takes those always), at the
lines between the two forms, on images that hold patches with neighbours and patches
without; lists past 16 entries, in 16-byte loads and entry by entry, against FP64
sums. And the scratch: no more than the tiles' regions, also under a memory limit."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu


def _workload(scale, **kw):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    base = dict(dict_images=10, dict_hr=160, n_dict=4000, L=6, k=10, w=12.0, test_h=16, test_w=16, scale=scale, cap=24)
    return torch, GpuWorkload(synthdata.scaled(synthdata.WORKLOADS["diff"], **{**base, **kw}))


def _tiles(scale, h, w):
    cols = 40 if scale <= 2 else 16
    return -(-(h - 4) // 8) * -(-(w - 4) // cols)


# sides that cut into just below and just above 200 and 300 tiles, one row and column more than whole tiles
SIZES = {1: [(13, 45), (4 + 8 * 39, 4 + 40 * 5), (5 + 8 * 39, 5 + 40 * 4)],
         2: [(9, 9), (13, 45), (4 + 8 * 39, 4 + 40 * 5), (5 + 8 * 39, 4 + 40 * 5), (4 + 8 * 49, 4 + 40 * 6),
             (5 + 8 * 49, 4 + 40 * 6)],
         3: [(12, 21), (3 + 8 * 20, 5 + 16 * 14)],
         4: [(11, 20), (4 + 8 * 12, 4 + 16 * 16), (4 + 8 * 20, 5 + 16 * 14)]}


@pytest.mark.parametrize("scale", [1, 2, 3, 4])
@pytest.mark.parametrize("K", [1, 5, 8, 16])
def test_rows_equal_tiles(scale, K):
    torch, g = _workload(scale)
    lrs = [torch.from_numpy(synthdata.fractal_voronoi_image(synthdata.SEED_BASE + 9100 + i, h, w)).cuda()
           for i, (h, w) in enumerate(SIZES[scale])]
    outs = [torch.empty((scale * lr.shape[0], scale * lr.shape[1]), device="cuda") for lr in lrs]
    with_n = without = 0
    single = []
    for lr in lrs:
        out = torch.empty((scale * lr.shape[0], scale * lr.shape[1]), device="cuda")
        g.zoom(lr=lr, K=K, out=out)
        m = g.results(K=K)["m"]
        with_n += int((m > 0).any())
        without += int((m == 0).any())
        single.append(out)
    assert with_n > 0 and without > 0, (with_n, without)
    wl = g.wl
    g.ctx.run_batch(lrs, outs, [scale] * len(lrs), K, wl.lam, 0, wl.sigma_s, wl.sigma_r)
    g.ctx.sync()
    for a, b, size in zip(single, outs, SIZES[scale]):
        assert torch.equal(a, b), (size, _tiles(scale, *size))


@pytest.mark.parametrize("scale", [1, 2, 3, 4])
@pytest.mark.parametrize("cap", [18, 20])
def test_long_lists(scale, cap):
    """A pixel is the mean of at most 25 patch values, each mu and a sum of cap
    products in fp32: within (cap + 30) 2^-23 of the largest |mu| + sum |w r|."""
    torch, g = _workload(scale, cap=cap, k=4, w=60.0)
    h, w = 17, 49
    lr = torch.from_numpy(synthdata.fractal_voronoi_image(77, h, w)).cuda()
    Q, ps = (h - 4) * (w - 4), 5 * scale
    ids = torch.empty((Q, cap), dtype=torch.int32, device="cuda")
    wt = torch.empty((Q, cap), device="cuda")
    out = torch.empty((scale * h, scale * w), device="cuda")
    g.set_mode(cap=cap, rerank=0, proj=1, lle_fp64=1)
    g.ctx.query(lr, h, w, scale, 4)
    g.ctx.lle_all(1e-3, ids, wt)
    g.ctx.reconstruct(out)
    g.ctx.sync()
    ids, wt = ids.cpu().numpy(), wt.cpu().numpy().astype(np.float64)
    resid, img = g.resid.cpu().numpy().astype(np.float64), lr.cpu().numpy().astype(np.float64)
    acc, cnt, size = np.zeros((scale * h, scale * w)), np.zeros((scale * h, scale * w)), 0.0
    lengths = set()
    for q in range(Q):
        m = int((ids[q] >= 0).sum())
        lengths.add(m)
        if m == 0:
            continue
        i, j = divmod(q, w - 4)
        mu, r = img[i:i + 5, j:j + 5].mean(), resid[ids[q, :m]]
        acc[scale * i:scale * i + ps, scale * j:scale * j + ps] += mu + (wt[q, :m] @ r).reshape(ps, ps)
        cnt[scale * i:scale * i + ps, scale * j:scale * j + ps] += 1
        size = max(size, abs(mu) + (np.abs(wt[q, :m]) @ np.abs(r)).max())
    assert cap in lengths and len(lengths) > 3
    err = np.abs(out.cpu().numpy() - acc / np.maximum(cnt, 1))[cnt > 0]
    assert err.max() <= (cap + 30) * 2.0 ** -23 * size


@pytest.mark.parametrize("scale", [2, 4])
def test_scratch_under_a_limit(monkeypatch, scale):
    """The smallest limit under which the weights are had leaves room for the image
    with the tiles' regions (10.6 KB a tile at x2, 16.2 at x4) and no more on top."""
    torch, g = _workload(scale, L=2, n_dict=500)
    from paper_1004_3980_amd import zoomhash as zb
    wl = g.wl
    h, w = {2: (200, 216), 4: (120, 131)}[scale]
    lr = torch.from_numpy(synthdata.fractal_voronoi_image(3, h, w)).cuda()
    out = torch.empty((scale * h, scale * w), device="cuda")

    def run(limit, image):
        monkeypatch.setenv("ZH_MEM_LIMIT", str(limit))
        c = zb.Context(0)
        try:
            c.build_tables(g.feat, g.resid, g.feat.shape[0], g.D, scale, wl.feat_mode, wl.L, wl.k, wl.w, 5)
            c.set_query_opts(cap=24, rerank=0, proj=1, lle_fp64=1)
            c.query(lr, h, w, scale, 4)
            c.lle_weights(1e-3)
            if image:
                c.reconstruct(out)
                c.sync()
            return True
        except zb.ZHError as e:
            assert e.status == zb.ZH_ENOMEM
            return False
        finally:
            c.close()

    lo, hi = 0, 512 << 20
    assert run(hi, False)
    while hi - lo > 1 << 16:
        mid = (lo + hi) // 2
        if run(mid, False):
            hi = mid
        else:
            lo = mid
    room = _tiles(scale, h, w) * ((12 * 44 * 4 + 12 * 44) if scale == 2 else (12 * 20 * 16 + 12 * 20)) * 4
    assert run(hi + room, True)
