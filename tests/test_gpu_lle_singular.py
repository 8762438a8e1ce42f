"""fp32 systems that fp32 cannot hold: sixteen copies of every training row, exact
or a millionth apart, and a lambda whose lambda tr(G) is at the rounding of the
Gram matrix, so that pivots come out at zero or below it. Each is solved again in
FP64 and counted. Against numpy's FP64 solve: the condition number is at most
1 + 1/lambda, both sides round sums of D terms and an elimination of at most 16
rows, |dw| <= (D + 3 * 16^2) 2^-52 (1 + 1/lambda) max|w| and 2^-23 |w| for the fp32
weights."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu

LAM = 1e-8


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("noise", [0.0, 1e-6, 1e-5])
@pytest.mark.parametrize("K", [3, 8, 12, 16])
def test_redone_in_fp64(mode, noise, K):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    D, base, copies = (25, 100)[mode], 200, 16
    n = base * copies
    wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], n_dict=base, dict_images=2, test_h=20, test_w=22)
    ctx = zb.Context(0)
    hr = torch.from_numpy(wl.dictionary_images()).cuda()
    pos = torch.from_numpy(wl.positions().astype(np.int32)).cuda()
    feat = torch.empty((base, D), device="cuda")
    resid = torch.empty((base, 100), device="cuda")
    ctx.make_dictionary(hr, hr.shape[0], hr.shape[1], hr.shape[2], pos, base, 2, 1.0, mode, feat, resid)
    g = np.random.default_rng(K)
    feat = feat.repeat_interleave(copies, 0).contiguous()
    feat += torch.from_numpy((noise * g.standard_normal((n, D))).astype(np.float32)).cuda()
    resid = resid.repeat_interleave(copies, 0).contiguous()
    ctx.build_tables(feat, resid, n, D, 2, mode, 6, 3, 20.0, 3)
    lr = torch.from_numpy(wl.test_image()).cuda()
    Q = 16 * 18
    qf = torch.empty((Q, D), device="cuda")
    ctx.features(lr, 20, 22, mode, qf)
    ctx.set_query_opts(cap=64, rerank=0, proj=1, lle_fp64=0)
    ctx.query(lr, 20, 22, 2, K)
    ctx.lle_weights(LAM)
    ids = torch.empty((Q, K), dtype=torch.int32, device="cuda")
    w = torch.empty((Q, K), device="cuda")
    ctx.get_results(ids=ids, w=w)
    redone = ctx.stats()["lle_fp64"]
    ids, w = ids.cpu().numpy(), w.cpu().numpy().astype(np.float64)
    x, q64 = feat.cpu().numpy().astype(np.float64), qf.cpu().numpy().astype(np.float64)
    full = 0
    tol = (D + 3 * 16 ** 2) * 2.0 ** -52 * (1.0 + 1.0 / LAM)
    for q in range(Q):
        m = int((ids[q] >= 0).sum())
        if m < 3:   # two rows: rounding can leave a pivot just above 1e-6 of the other
            continue
        Z = q64[q] - x[ids[q, :m]]
        G = Z @ Z.T
        t = np.trace(G)
        if t == 0:
            continue
        full += 1
        s = np.linalg.solve(G + LAM * t * np.eye(m), np.ones(m))
        ref = s / s.sum()
        assert (np.abs(w[q, :m] - ref) <= 2.0 ** -23 * np.abs(ref) + tol * np.abs(ref).max()).all(), (q, m, w[q], ref)
    assert full > 100 and redone >= full // 2, (full, redone)
