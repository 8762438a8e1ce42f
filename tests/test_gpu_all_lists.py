"""The lists and weights over every match do not depend on where the neighbours
came from before the call: the search with the same options (its union alone is
listed again) or one with others, the l1 ranking or the neighbours of two bins
(the search runs again). Lists ascending without repeats, neighbours and counts
afterwards those of the search, bit for bit in every case."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1, 24, 65, 80])
@pytest.mark.parametrize("rerank", [0, 32])
def test_lists(cap, rerank):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    wl = synthdata.scaled(synthdata.WORKLOADS["mid"], n_dict=8000, dict_images=8, test_h=19, test_w=23,
                          w=200.0)   # wide hashes: enough candidates to reach the cap
    g = GpuWorkload(wl)
    K, Q = 5, 15 * 19

    def query(rr=rerank):
        g.ctx.set_query_opts(cap=cap, rerank=rr, proj=1, lle_fp64=1)
        g.ctx.query(g.lr, g.h, g.w, wl.scale, K)

    def other_options():
        query(16 if rerank else 32)
        g.ctx.set_query_opts(cap=cap, rerank=rerank, proj=1, lle_fp64=1)

    def l1():
        g.ctx.set_query_metric("l1")
        query()
        g.ctx.set_query_metric("l2")

    def two_bins():
        query()
        g.ctx.knn_t(2)

    def hashed():
        query()
        f = g.feat[:64]
        keys = torch.empty((64, wl.L), dtype=torch.int64, device="cuda")
        g.ctx.hash(wl.scale, f, 64, None, keys)

    got = []
    for before in (query, other_options, l1, two_bins, hashed, query):
        before()
        for _ in range(2):
            ids = torch.full((Q, cap), -7, dtype=torch.int32, device="cuda")
            w = torch.full((Q, cap), -7.0, device="cuda")
            g.ctx.lle_all(wl.lam, ids, w)
            r = [torch.empty((Q, K), dtype=torch.int32, device="cuda"), torch.empty((Q, K), device="cuda"),
                 torch.empty(Q, dtype=torch.int32, device="cuda"), torch.empty(Q, dtype=torch.int32, device="cuda")]
            g.ctx.get_results(r[0], r[1], r[2], None, r[3])
            st = g.ctx.stats()
            g.ctx.sync()
            got.append([x.cpu().numpy() for x in (ids, w, *r)] + [np.array([st["rank_fallbacks"], st["truncated"],
                                                                             st["codes_fixed"], st["lle_fp64"]])])
    ids, n = got[0][0], got[0][5]
    assert n.max() == cap or cap > 24
    for q in range(Q):
        assert (np.diff(ids[q, :n[q]]) > 0).all() and (ids[q, n[q]:] == -1).all()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
