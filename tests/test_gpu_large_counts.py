"""More patches and pairs than a one-dimensional grid of one workgroup each holds
(threads along x below 2^32): the results of patches at the image's corners and
around its middle are those of the same patches in small images, and a training
position outside its image is found past 2^24 positions."""
import pytest

pytestmark = pytest.mark.gpu


def _ctx(n=600, L=3):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    g = torch.Generator(device="cuda").manual_seed(1)
    feat = torch.randn((n, 25), device="cuda", generator=g) * 0.1
    feat -= feat.mean(1, keepdim=True)
    resid = torch.zeros((n, 25), device="cuda")
    ctx = zb.Context(0)
    ctx.build_tables(feat, resid, n, 25, 1, 0, L, 2, 2.0, 1)
    ctx.set_query_opts(cap=0, rerank=0, proj=1, lle_fp64=1)
    return torch, zb, ctx


# past 2^24 patches (a workgroup of 256 threads each) and past 2^26 (a wave each)
@pytest.mark.parametrize("h,w,K", [(4101, 4102, 3), (8197, 8196, 9)])
def test_patches(h, w, K):
    torch, _, ctx = _ctx()
    Q = (h - 4) * (w - 4)
    assert Q > (1 << 24 if K == 3 else 1 << 26)
    g = torch.Generator(device="cuda").manual_seed(2)
    img = torch.rand((h, w), device="cuda", generator=g) * 0.3

    def run(lr, t):
        hh, ww = lr.shape
        q = (hh - 4) * (ww - 4)
        out = [torch.empty((q, K), dtype=torch.int32, device="cuda"), torch.empty((q, K), device="cuda"),
               torch.empty(q, dtype=torch.int32, device="cuda"), torch.empty((q, K), device="cuda"),
               torch.empty(q, dtype=torch.int32, device="cuda")]
        ctx.query(lr, hh, ww, 1, K)
        if t:
            ctx.knn_t(t)
        ctx.lle_weights(1e-3)
        ctx.get_results(ids=out[0], d2=out[1], m=out[2], w=out[3], ncand=out[4])
        ctx.sync()
        return [o.view(hh - 4, ww - 4, *o.shape[1:]) for o in out]

    crops = [(0, 0), (h - 14, w - 24), (h // 2, w // 3), ((1 << 24) // (w - 4) - 3, 40), (h - 14, 0)]
    for t in (0, 2):
        big = run(img, t)
        assert int((big[2] > 1).sum()) > Q // 50, "patches with neighbours"
        for i, j in crops:
            small = run(img[i:i + 14, j:j + 24].contiguous(), t)
            for a, b in zip(big, small):
                assert torch.equal(a[i:i + 10, j:j + 20], b), (t, i, j)
        del big


def test_positions():
    torch, zb, ctx = _ctx()
    n, side = (1 << 24) + 100, 64
    hr = torch.rand((1, side, side), device="cuda")
    pos = torch.zeros((n, 3), dtype=torch.int32, device="cuda")
    pos[:, 1] = torch.arange(n, device="cuda") % 57
    feat = torch.zeros((n, 25), device="cuda")
    resid = torch.zeros((n, 25), device="cuda")
    args = (hr, 1, side, side, pos, n, 1, 1.0, 0, feat, resid)
    for bad in (n - 1, 1 << 24):
        pos[bad, 1] = 60
        with pytest.raises(zb.ZHError) as e:
            ctx.make_dictionary(*args)
        assert e.value.status == zb.ZH_EINVAL
        ctx.sync()
        assert not feat.any() and not resid.any()
        pos[bad, 1] = bad % 57
    ctx.make_dictionary(*args)
    ctx.sync()
    assert torch.equal(feat[57:n], feat[:n - 57]) and torch.equal(resid[57:n], resid[:n - 57])


def test_one_row_searches_say_so():
    """The early stop's searches take a wave a patch in one row: past 2^26 patches the
    call fails and says so."""
    torch, zb, ctx = _ctx()
    h, w = 8197, 8196
    img = torch.zeros((h, w), device="cuda")
    ctx.set_query_opts(cap=8, rerank=0, proj=1, lle_fp64=1)
    for metric in ("l2", "l1"):
        ctx.set_query_metric(metric)
        with pytest.raises(zb.ZHError) as e:
            ctx.query(img, h, w, 1, 3)
        assert e.value.status == zb.ZH_EDEVICE
        with pytest.raises(zb.ZHError) as e:   # nothing stands
            ctx.lle_weights(1e-3)
        assert e.value.status == zb.ZH_ESTATE
    ctx.set_query_metric("l2")
    ctx.query(img[:40, :40].contiguous(), 40, 40, 1, 3)
    ctx.sync()
