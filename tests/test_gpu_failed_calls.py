"""Calls that fail for want of memory leave no state that later calls would read
from buffers that are gone or were never written."""
import pytest

import synthdata

pytestmark = pytest.mark.gpu


def _limited(monkeypatch, run):
    """The smallest limit (to 64 KB) under which run(limit) is true."""
    lo, hi = 0, 256 << 20
    assert run(hi)
    while hi - lo > 1 << 16:
        mid = (lo + hi) // 2
        if run(mid):
            hi = mid
        else:
            lo = mid
    return hi


def test_lists_of_all_matches(monkeypatch):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["diff"], dict_images=4, dict_hr=96, n_dict=2000, L=4, k=6, w=40.0,
                          test_h=260, test_w=270, cap=8)
    g = GpuWorkload(wl)
    out = torch.empty((2 * g.h, 2 * g.w), device="cuda")

    def start(limit):
        monkeypatch.setenv("ZH_MEM_LIMIT", str(limit))
        c = zb.Context(0)
        c.build_tables(g.feat, g.resid, g.feat.shape[0], g.D, 2, wl.feat_mode, wl.L, wl.k, wl.w, 5)
        c.set_query_opts(cap=8, rerank=0, proj=1, lle_fp64=1)
        c.query(g.lr, g.h, g.w, 2, 4)
        c.lle_all(1e-3)
        c.reconstruct(out)
        c.sync()
        return c

    def run(limit):
        try:
            start(limit).close()
            return True
        except zb.ZHError as e:
            assert e.status == zb.ZH_ENOMEM
            return False

    limit = _limited(monkeypatch, run)
    for first in ("lists", "weights"):
        # room for the longer lists alone, and for neither
        for room in (0, 4 * g.Q * 80):
            c = start(limit + room)
            c.set_query_opts(cap=80, rerank=0, proj=1, lle_fp64=1)
            with pytest.raises(zb.ZHError) as e:
                c.lle_all(1e-3)
            assert e.value.status == zb.ZH_ENOMEM
            with pytest.raises(zb.ZHError) as e:
                c.reconstruct(out)
            assert e.value.status == zb.ZH_ESTATE
            if first == "weights":   # the neighbours still stand
                c.lle_weights(1e-3)
                c.reconstruct(out)
            c.set_query_opts(cap=8, rerank=0, proj=1, lle_fp64=1)
            c.lle_all(1e-3)
            c.reconstruct(out)
            c.sync()
            c.close()
