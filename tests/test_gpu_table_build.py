"""Bins of the tables where the build can go wrong: one row, fewer rows than a
sort tile or a wave, one row over, bins that hold nearly every row, more than
one group of tables, and key counts on both sides of the sort's digit widths.
Every patch's candidates without a stop are the oracle's, IDs ascending, and
two builds of the same rows give the same bins."""
import numpy as np
import pytest

import synthdata
from oracle import lsh

pytestmark = pytest.mark.gpu


def _images(n):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], n_dict=n, dict_images=max(2, n // 2500), test_h=12, test_w=13)
    return torch, wl


# (rows, tables, hashes, width): 2 n <= cap picks the sort's bits
@pytest.mark.parametrize("n,L,k,w", [(1, 3, 2, 4.0), (63, 5, 3, 4.0), (64, 1, 1, 50.0), (1025, 7, 4, 8.0),
                                     (4096, 3, 2, 3000.0), (4097, 64, 2, 6.0), (20_001, 9, 6, 4.0)])
def test_bins(n, L, k, w):
    torch, wl = _images(n)
    from paper_1004_3980_amd import zoomhash as zb
    ctx = zb.Context(0)
    hr = torch.from_numpy(wl.dictionary_images()).cuda()
    pos = torch.from_numpy(wl.positions().astype(np.int32)).cuda()
    feat = torch.empty((n, 25), device="cuda")
    resid = torch.empty((n, 100), device="cuda")
    ctx.make_dictionary(hr, hr.shape[0], hr.shape[1], hr.shape[2], pos, n, 2, 1.0, 0, feat, resid)
    lr = torch.from_numpy(wl.test_image()).cuda()
    Q = 8 * 9
    qf = torch.empty((Q, 25), device="cuda")
    ctx.features(lr, 12, 13, 0, qf)
    fn, qn = feat.cpu().numpy(), qf.cpu().numpy()
    a, b = lsh.hash_params(7, L, k, 25, w)
    tables = lsh.Tables(lsh.bucket_keys(lsh.codes(fn, a, b, w), L, k))
    qkeys = lsh.bucket_keys(lsh.codes(qn, a, b, w), L, k)
    ref = lsh.candidates_t(tables, qkeys, 1)
    got = []
    for _ in range(2):
        ctx.build_tables(feat, resid, n, 25, 2, 0, L, k, w, 7)
        ctx.set_query_opts(cap=0, rerank=0, proj=1, lle_fp64=1)
        ctx.query(lr, 12, 13, 2, 1)
        counts = torch.zeros(Q, dtype=torch.int32, device="cuda")
        ids = torch.full((Q, n), -1, dtype=torch.int32, device="cuda")
        ctx.candidates(n, counts, ids)
        ctx.sync()
        got.append((counts.cpu().numpy(), ids.cpu().numpy(), ctx.table_entropy(2, L)))
    for q in range(Q):
        assert got[0][0][q] == len(ref[q]), q
        assert np.array_equal(got[0][1][q, :len(ref[q])], ref[q]), q
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    for l in range(L):
        _, c = np.unique(tables.sorted_keys[l], return_counts=True)
        p = c / n
        assert abs(got[0][2][l] + (p * np.log2(p)).sum()) <= 1e-12 * max(1.0, np.log2(max(n, 2)))


# the screen's basis in a saved file (its last two parts: the bf16 split of Phi,
# 64 rows): one row, fewer rows than directions, more
@pytest.mark.parametrize("mode,D", [(0, 25), (1, 100)])
@pytest.mark.parametrize("n", [1, 40, 5000])
def test_screen_basis(tmp_path, mode, D, n):
    """Rows of unit length, orthogonal, that turn the rows' covariance to its
    largest eigenvalues in order. The split holds a row within 2^-17 of its
    length, so products of rows are within 2^-16 and entries of Phi C Phi^T
    within 2^-16 of the largest eigenvalue, twice over to be safe."""
    torch, wl = _images(max(n, 2))
    from paper_1004_3980_amd import zoomhash as zb
    ctx = zb.Context(0)
    hr = torch.from_numpy(wl.dictionary_images()).cuda()
    pos = torch.from_numpy(wl.positions().astype(np.int32)).cuda()
    feat = torch.empty((n, D), device="cuda")
    resid = torch.empty((n, 100), device="cuda")
    ctx.make_dictionary(hr, hr.shape[0], hr.shape[1], hr.shape[2], pos, n, 2, 1.0, mode, feat, resid)
    ctx.build_tables(feat, resid, n, D, 2, mode, 2, 2, 8.0, 7)
    ctx.save_tables(2, str(tmp_path / "t"))
    m, DP = min(D, 56), (D + 31) // 32 * 32
    raw = np.fromfile(tmp_path / "t", dtype=np.uint16)[-2 * 64 * DP:].reshape(2, 64, DP)
    split = (raw.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    assert not raw[:, m:].any() and not raw[:, :, D:].any()
    phi = (split[0] + split[1])[:m, :D]
    x = feat.cpu().numpy().astype(np.float64)
    c = x.T @ x
    top = np.linalg.eigvalsh(c)[::-1][:m]
    tol = 2.0 ** -15
    assert np.abs(phi @ phi.T - np.eye(m)).max() <= tol
    assert np.abs(phi @ c @ phi.T - np.diag(top)).max() <= tol * top[0]
