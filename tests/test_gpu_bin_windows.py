"""Neighbours among the IDs of at least t bins where a patch's bins hold more
entries than one window of the ranking (2048): unions of tens of thousands of
entries, bins of very different sizes, and images whose flat patches give
thousands of equal rows (ties go by ID). IDs, counts and distances are those
of the oracle (FP64 sums in index order on both sides) bit for bit, for the
t-of-L neighbours and for the query without a stop (t = 1)."""
import numpy as np
import pytest

import synthdata
from oracle import pipeline

pytestmark = pytest.mark.gpu

SMALL = dict(test_h=13, test_w=14)
WIDE = ("tiny", dict(SMALL, w=64.0))                   # bins of thousands in every table
ALL = ("tiny", dict(SMALL, w=2000.0))                  # nearly every row in every bin
FLAT = ("tiny", dict(SMALL, amp=0.0))                  # piecewise constant: equal rows
FEW = ("tiny", dict(SMALL, w=1.0))                     # empty and tiny bins
GRAD = ("mid", dict(SMALL, w=200.0, n_dict=20_000, dict_images=8))
_cache = {}


def _case(name, kw):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    key = (name, tuple(sorted(kw.items())))
    if key not in _cache:
        wl = synthdata.scaled(synthdata.WORKLOADS[name], **kw)
        pre = pipeline.prepare(wl.dictionary_images(), wl.positions(), wl.scale, wl.feat_mode, wl.L, wl.k, wl.w,
                               wl.hash_seed)
        _cache[key] = (wl, GpuWorkload(wl), pre)
    return _cache[key]


@pytest.mark.parametrize("case,most", [(WIDE, 8192), (ALL, 100_000), (FLAT, 8192), (FEW, 0), (GRAD, 8192)])
@pytest.mark.parametrize("t,K", [(1, 1), (1, 16), (2, 5), (8, 16)])
def test_neighbours_over_windows(case, most, t, K):
    wl, g, pre = _case(*case)
    lr = g.lr.cpu().numpy()
    qr = pipeline.query(pre, lr, K, wl.lam, t=t, synthesize=False)
    assert qr.bucket_sizes.sum(axis=1).max() >= most
    counts = np.array([len(c) for c in qr.cand], dtype=np.int32)
    g.set_mode(cap=0, rerank=0, proj=1, lle_fp64=1)
    forms = ["query"] if t == 1 else []
    for form in forms + ["t-of-L"]:
        g.ctx.query(g.lr, g.h, g.w, wl.scale, K)
        if form == "t-of-L":
            g.ctx.knn_t(t)
        g.ctx.lle_weights(wl.lam)
        r = g.results(K=K)
        assert np.array_equal(r["ncand"], counts), form
        assert np.array_equal(r["m"], qr.m), form
        assert np.array_equal(r["ids"], np.where(qr.ids >= 0, qr.ids, -1).astype(np.int32)), form
        for q in np.nonzero(qr.m > 0)[0]:
            assert np.array_equal(r["d2"][q, :qr.m[q]], qr.d2[q, :qr.m[q]].astype(np.float32)), (form, q)
    if t == 1:
        total = qr.bucket_sizes.sum(axis=1)
        g.ctx.query(g.lr, g.h, g.w, wl.scale, K)
        st = g.ctx.stats()
        assert (st["deferred"], st["streamed"]) == ((total > 2048).sum(), (total > 8192).sum())
