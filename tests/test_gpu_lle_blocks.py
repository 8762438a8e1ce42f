"""The wave-per-patch LLE solver at the edges of its blocks of 16 rows,
against numpy's FP64 solve of the same systems: K = 9 .. 16 neighbours and
lists of up to 80 matches (one to five blocks, full and with one row over),
both feature dimensions.

FP64 form: both sides solve in FP64 (condition number at most 1 + 1/lambda)
and the weights are rounded to fp32: |dw| <= 2^-23 |w| + 1e-9 max|w|. fp32
form: Gram sums of D terms and an elimination of at most 16 rows,
|dw| <= (D + 48) 2^-24 (1 + 1/lambda) max|w|."""
import numpy as np
import pytest

import synthdata

pytestmark = pytest.mark.gpu

TINY = ("tiny", dict(w=16.0))
MID = ("mid", dict(w=80.0, test_h=40, test_w=44, n_dict=30_000, dict_images=8))
_cache = {}


def _workload(name, kw):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    if name not in _cache:
        g = GpuWorkload(synthdata.scaled(synthdata.WORKLOADS[name], **kw))
        feat = g.feat.cpu().numpy().astype(np.float64)
        q = torch.empty((g.Q, g.D), dtype=torch.float32, device="cuda")
        g.ctx.features(g.lr, g.h, g.w, g.wl.feat_mode, q)
        _cache[name] = (torch, g, feat, q.cpu().numpy().astype(np.float64))
    return _cache[name]


def _check(ids, w, feat, qf, lam, rel, floor):
    sizes = set()
    for q in range(len(ids)):
        m = int((ids[q] >= 0).sum())
        sizes.add(m)
        assert (w[q, m:] == 0).all(), q
        if m == 0:
            continue
        Z = qf[q] - feat[ids[q, :m]]
        G = Z @ Z.T
        t = np.trace(G)
        x = np.linalg.solve(G + lam * t * np.eye(m), np.ones(m)) if t > 0 else np.ones(m)
        ref = x / x.sum()
        assert (np.abs(w[q, :m] - ref) <= rel * np.abs(ref) + floor * np.abs(ref).max()).all(), (q, m)
    return sizes


@pytest.mark.parametrize("wl", [TINY, MID])
@pytest.mark.parametrize("K", [9, 15, 16])
@pytest.mark.parametrize("fp64", [0, 1])
def test_k_above_eight(wl, K, fp64):
    torch, g, feat, qf = _workload(*wl)
    g.set_mode(cap=48, rerank=0, proj=1, lle_fp64=fp64)
    g.ctx.query(g.lr, g.h, g.w, g.wl.scale, K)
    g.ctx.lle_weights(g.wl.lam)
    ids = torch.empty((g.Q, K), dtype=torch.int32, device="cuda")
    w = torch.empty((g.Q, K), dtype=torch.float32, device="cuda")
    g.ctx.get_results(ids=ids, w=w)
    g.ctx.sync()
    lam = g.wl.lam
    rel, floor = (2.0 ** -23, 1e-9) if fp64 else (0.0, (g.D + 48) * 2.0 ** -24 * (1.0 + 1.0 / lam))
    sizes = _check(ids.cpu().numpy(), w.cpu().numpy().astype(np.float64), feat, qf, lam, rel, floor)
    assert K in sizes and len(sizes) > 3


@pytest.mark.parametrize("wl", [TINY, MID])
@pytest.mark.parametrize("cap", [1, 16, 17, 33, 64, 65, 80])
def test_all_matches_blocks(wl, cap):
    torch, g, feat, qf = _workload(*wl)
    g.set_mode(cap=cap, rerank=0, proj=1, lle_fp64=1)
    g.ctx.query(g.lr, g.h, g.w, g.wl.scale, 5)
    ids = torch.full((g.Q, cap), -7, dtype=torch.int32, device="cuda")
    w = torch.full((g.Q, cap), -7.0, dtype=torch.float32, device="cuda")
    g.ctx.lle_all(g.wl.lam, ids, w)
    g.ctx.sync()
    ids = ids.cpu().numpy()
    assert ((ids == -1) | (ids >= 0)).all()
    sizes = _check(ids, w.cpu().numpy().astype(np.float64), feat, qf, g.wl.lam, 2.0 ** -23, 1e-9)
    assert cap in sizes
