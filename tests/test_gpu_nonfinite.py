"""Features that are not finite: training rows of NaN and of infinities leave the
tables, the screen's basis and the neighbours of everything else as they are, and
a distance that is not a number ranks last, by ID, in every search, so that each
neighbour named is one of the candidates."""
import numpy as np
import pytest

import synthdata
from oracle import lsh

pytestmark = pytest.mark.gpu

N, SCALE, L, K_HASH, WIDTH, SEED = 3000, 2, 6, 4, 6.0, 7
BAD = {5: np.nan, 1500: np.inf, 2222: -np.inf}


class Tables:
    """A dictionary with a row of NaN and two of infinities, its tables, a query
    image, and what the oracle says of them. The codes of the rows that are not
    finite are the library's own (no definition gives them)."""

    def __init__(self, mode):
        import torch
        assert torch.cuda.is_available(), "GPU test needs a GPU"
        from paper_1004_3980_amd import zoomhash as zb
        self.torch, self.mode, self.D = torch, mode, 25 if mode == 0 else 100
        wl = synthdata.scaled(synthdata.WORKLOADS["tiny"], n_dict=N, dict_images=2, test_h=24, test_w=27)
        ctx = self.ctx = zb.Context(0)
        hr = torch.from_numpy(wl.dictionary_images()).cuda()
        pos = torch.from_numpy(wl.positions().astype(np.int32)).cuda()
        self.feat = torch.empty((N, self.D), device="cuda")
        self.resid = torch.empty((N, 100), device="cuda")
        ctx.make_dictionary(hr, hr.shape[0], hr.shape[1], hr.shape[2], pos, N, SCALE, 1.0, mode, self.feat, self.resid)
        for r, v in BAD.items():
            self.feat[r] = v
        ctx.build_tables(self.feat, self.resid, N, self.D, SCALE, mode, L, K_HASH, WIDTH, SEED)
        self.h, self.w = 24, 27
        self.Q = 20 * 23
        lr = wl.test_image()
        lr[:9, :11] = 0.5   # flat patches: all codes 0, as those of rows of NaN
        self.lr = torch.from_numpy(lr).cuda()
        qf = torch.empty((self.Q, self.D), device="cuda")
        ctx.features(self.lr, self.h, self.w, mode, qf)
        self.x, self.q = self.feat.cpu().numpy(), qf.cpu().numpy()
        self.a, self.b = lsh.hash_params(SEED, L, K_HASH, self.D, WIDTH)
        codes = torch.empty((N, L * K_HASH), dtype=torch.int32, device="cuda")
        keys = torch.empty((N, L), dtype=torch.int64, device="cuda")
        ctx.hash(SCALE, self.feat, N, codes, keys)
        ctx.sync()
        self.codes, self.keys = codes.cpu().numpy(), keys.cpu().numpy().view(np.uint64)
        good = self.good = np.setdiff1d(np.arange(N), list(BAD))
        ref = lsh.codes(self.x[good], self.a, self.b, WIDTH)
        assert np.array_equal(self.codes[good], ref)
        assert np.array_equal(self.keys[good], lsh.bucket_keys(ref, L, K_HASH))
        self.tables = lsh.Tables(self.keys)
        qkeys = lsh.bucket_keys(lsh.codes(self.q, self.a, self.b, WIDTH), L, K_HASH)
        self.cand = {t: lsh.candidates_t(self.tables, qkeys, t) for t in (1, 2)}
        self.qkeys = qkeys

    def early(self, cap):
        return self.tables.candidates(self.qkeys, cap)[0]

    def use_image(self, lr):
        """Another image, whose keys are the library's own."""
        t = self.torch
        self.lr = t.from_numpy(lr).cuda()
        qf = t.empty((self.Q, self.D), device="cuda")
        self.ctx.features(self.lr, self.h, self.w, self.mode, qf)
        keys = t.empty((self.Q, L), dtype=t.int64, device="cuda")
        self.ctx.hash(SCALE, qf, self.Q, None, keys)
        self.ctx.sync()
        self.q, self.qkeys = qf.cpu().numpy(), keys.cpu().numpy().view(np.uint64)
        self.cand = {n: lsh.candidates_t(self.tables, self.qkeys, n) for n in (1, 2)}

    def dist(self, q, ids, l1=False):
        """Distances in FP64, what is not a number as the largest."""
        with np.errstate(invalid="ignore", over="ignore"):
            z = self.q[q].astype(np.float64) - self.x[ids].astype(np.float64)
            d = np.abs(z).sum(1) if l1 else (z * z).sum(1)
        return np.where(np.isnan(d), np.inf, d)

    def results(self, K):
        t = self.torch
        ids = t.empty((self.Q, K), dtype=t.int32, device="cuda")
        d = t.empty((self.Q, K), device="cuda")
        m = t.empty(self.Q, dtype=t.int32, device="cuda")
        nc = t.empty(self.Q, dtype=t.int32, device="cuda")
        self.ctx.get_results(ids=ids, d2=d, m=m, ncand=nc)
        self.ctx.sync()
        return [v.cpu().numpy() for v in (ids, d, m, nc)]

    def check(self, K, lists, l1=False, exact=True):
        ids, d, m, nc = self.results(K)
        bad = 0
        for q in range(self.Q):
            c = np.asarray(lists[q])
            assert nc[q] == len(c) and m[q] == min(K, len(c)), q
            bad += len(set(c) & set(BAD))
            dist = self.dist(q, c, l1)
            order = np.lexsort((c, dist))[:K]
            got = ids[q, :m[q]]
            assert (ids[q, m[q]:] == -1).all()
            if not exact:
                assert len(set(got)) == m[q] and set(got) <= set(c), q
                continue
            if not np.array_equal(got, c[order]):
                # equal up to the rounding of sums that the oracle takes in another order
                assert len(set(got)) == m[q] and set(got) <= set(c), q
                gd = self.dist(q, got, l1)
                fin = np.isfinite(dist[order])
                assert np.array_equal(np.isfinite(gd), fin), q
                assert np.allclose(gd[fin], dist[order][fin], rtol=1e-12, atol=0), q
                assert np.array_equal(got[~fin], c[order][~fin]), q
        return bad


@pytest.mark.parametrize("mode", [0, 1])
def test_tables_and_neighbours(mode, tmp_path):
    t = Tables(mode)
    t.ctx.save_tables(SCALE, str(tmp_path / "t"))
    DP = (t.D + 31) // 32 * 32
    raw = np.fromfile(tmp_path / "t", dtype=np.uint16)[-2 * 64 * DP:].reshape(2, 64, DP)
    split = (raw.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    m = min(t.D, 56)
    phi = (split[0] + split[1])[:m, :t.D]
    # orthonormal rows, as for features that are finite
    assert np.isfinite(phi).all() and np.abs(phi @ phi.T - np.eye(m)).max() <= 2.0 ** -15
    t.ctx.set_query_opts(cap=0, rerank=0, proj=1, lle_fp64=1)
    for K in (1, 7):
        t.ctx.query(t.lr, t.h, t.w, SCALE, K)
        assert t.check(K, t.cand[1]) > 0, "no patch met a row that is not finite"
    t.ctx.knn_t(2)
    t.check(7, t.cand[2])


def test_every_row_not_finite():
    import torch
    from paper_1004_3980_amd import zoomhash as zb
    for mode, D in ((0, 25), (1, 100)):
        ctx = zb.Context(0)
        feat = torch.full((70, D), float("nan"), device="cuda")
        resid = torch.zeros((70, 100), device="cuda")
        ctx.build_tables(feat, resid, 70, D, SCALE, mode, 3, 2, 4.0, SEED)
        keys = torch.empty((70, 3), dtype=torch.int64, device="cuda")
        ctx.hash(SCALE, feat, 70, None, keys)
        ctx.sync()
        assert (keys == keys[0]).all()


def _forms(t, K):
    """Every search and ranking of one image: the neighbours against the oracle's
    (the forms that rank by bounds or halves of the features: that they are
    candidates), and the path behind them to its end."""
    c, bad = t.ctx, 0
    out = t.torch.empty((SCALE * t.h, SCALE * t.w), device="cuda")

    def finish():
        c.lle_weights(1e-3)
        c.reconstruct(out)
        c.sync()

    for cap in (8, 40):
        early = t.early(cap)
        for rerank in (0, 16):
            for fp64 in (1, 0):
                c.set_query_opts(cap=cap, rerank=rerank, proj=1, lle_fp64=fp64)
                c.query(t.lr, t.h, t.w, SCALE, K)
                bad += t.check(K, early, exact=rerank == 0)
                finish()
        c.knn_l1()
        t.check(K, early, l1=True)
        finish()
        c.lle_all(1e-3)
        c.reconstruct(out)
        c.set_query_metric("l1")
        c.query(t.lr, t.h, t.w, SCALE, K)
        t.check(K, early, l1=True)
        finish()
        c.set_query_metric("l2")
    for rerank in (0, 16):
        c.set_query_opts(cap=0, rerank=rerank, proj=1, lle_fp64=1)
        c.query(t.lr, t.h, t.w, SCALE, K)
        t.check(K, t.cand[1], exact=rerank == 0)
        finish()
    c.knn_t(2)
    t.check(K, t.cand[2])
    finish()
    return bad


@pytest.mark.parametrize("K", [3, 7, 12])
@pytest.mark.parametrize("mode", [0, 1])
def test_searches(mode, K):
    t = Tables(mode)
    assert _forms(t, K) > 0, "no patch met a row that is not finite"


@pytest.mark.parametrize("K", [3, 12])
@pytest.mark.parametrize("mode", [0, 1])
def test_queries_not_finite(mode, K):
    t = Tables(mode)
    lr = t.lr.cpu().numpy()
    lr[3, 4] = np.nan
    lr[20, 9] = np.inf
    lr[12:18, 15:21] = -np.inf
    t.use_image(lr)
    bad_rows = ~np.isfinite(t.q).all(1)
    assert bad_rows.any() and any(len(t.cand[1][q]) for q in np.nonzero(bad_rows)[0])
    _forms(t, K)
