"""Ranking over the bins' windows where few IDs are left: no bin at all, up to 64 IDs
(one wave's list, nothing to join) and just above, below and above the number of
patches from which long patches are listed. Candidates by the oracle, distances the
FP64 sum over the coordinates in order, ties by ID."""
import numpy as np
import pytest

import synthdata
from oracle import lsh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,h,w,width", [(0, 40, 44, 4.0), (0, 100, 101, 3.0), (1, 40, 44, 24.0), (1, 98, 100, 20.0)])
def test_ranking(mode, h, w, width):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    n, D, L, k, seed = 3000, (25, 100)[mode], 6, 5, 7
    wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], n_dict=n, dict_images=2, test_h=h, test_w=w)
    ctx = zb.Context(0)
    hr = torch.from_numpy(wl.dictionary_images()).cuda()
    pos = torch.from_numpy(wl.positions().astype(np.int32)).cuda()
    feat, resid = torch.empty((n, D), device="cuda"), torch.empty((n, 100), device="cuda")
    ctx.make_dictionary(hr, hr.shape[0], hr.shape[1], hr.shape[2], pos, n, 2, 1.0, mode, feat, resid)
    ctx.build_tables(feat, resid, n, D, 2, mode, L, k, width, seed)
    lr = torch.from_numpy(wl.test_image()).cuda()
    Q = (h - 4) * (w - 4)
    qf = torch.empty((Q, D), device="cuda")
    ctx.features(lr, h, w, mode, qf)
    ctx.sync()
    x, qv = feat.cpu().numpy(), qf.cpu().numpy()
    a, b = lsh.hash_params(seed, L, k, D, width)
    tables = lsh.Tables(lsh.bucket_keys(lsh.codes(x, a, b, width), L, k))
    qkeys = lsh.bucket_keys(lsh.codes(qv, a, b, width), L, k)
    ctx.set_query_opts(cap=0, rerank=0, proj=1, lle_fp64=1)
    seen = set()
    for K in (1, 16):
        for t in (1, 2):
            cand = lsh.candidates_t(tables, qkeys, t)
            ctx.query(lr, h, w, 2, K)
            if t > 1:
                ctx.knn_t(t)
            ids = torch.empty((Q, K), dtype=torch.int32, device="cuda")
            d = torch.empty((Q, K), device="cuda")
            m = torch.empty(Q, dtype=torch.int32, device="cuda")
            nc = torch.empty(Q, dtype=torch.int32, device="cuda")
            ctx.get_results(ids=ids, d2=d, m=m, ncand=nc)
            ctx.sync()
            ids, d, m, nc = (v.cpu().numpy() for v in (ids, d, m, nc))
            assert np.array_equal(nc, [len(c) for c in cand]) and np.array_equal(m, np.minimum(nc, K))
            for q in range(Q):
                c = cand[q]
                seen.add(0 if len(c) == 0 else 1 if len(c) <= 64 else 2 if len(c) <= 128 else 3)
                s = np.zeros(len(c))
                for i in range(D):
                    z = qv[q, i].astype(np.float64) - x[c, i].astype(np.float64)
                    s = s + z * z
                o = np.lexsort((c, s))[:K]
                assert np.array_equal(ids[q, :m[q]], c[o]) and (ids[q, m[q]:] == -1).all(), (K, t, q)
                assert np.array_equal(d[q, :m[q]], s[o].astype(np.float32)) and (d[q, m[q]:] == 0).all(), (K, t, q)
    assert {0, 1, 2} <= seen, seen
