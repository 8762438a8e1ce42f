"""Codes and keys at the edges of the hash kernels: table heights that do and
do not fill a quad of rows or a tile, an odd table count, one row, ragged rows
around one and two row tiles a wave, rows off 16-byte boundaries, and features
whose codes the MFMA bound leaves open in most tables (the lists run over and
whole rows go to the recomputation). Bitwise against the oracle: the codes are
defined by the FP64 sum, so there is no tolerance."""
import numpy as np
import pytest

from oracle import lsh

pytestmark = pytest.mark.gpu


def _tables(torch, zoomhash, mode, L, k, w, seed):
    D = 25 if mode == 0 else 100
    g = np.random.default_rng(seed)
    n = 300
    feat = torch.from_numpy(g.standard_normal((n, D)).astype(np.float32) * 8).cuda()
    resid = torch.zeros((n, 100), dtype=torch.float32, device="cuda")
    ctx = zoomhash.Context(0)
    ctx.build_tables(feat, resid, n, D, 2, mode, L, k, w, seed)
    return ctx, feat, resid, D


@pytest.mark.parametrize("proj", [0, 1])
@pytest.mark.parametrize("mode,L,k", [(0, 1, 1), (0, 5, 8), (0, 3, 13), (1, 4, 7), (1, 3, 20), (1, 5, 32), (1, 64, 4)])
def test_codes_at_tile_edges(mode, L, k, proj):
    import torch
    from paper_1004_3980_amd import zoomhash

    w = 16.0
    ctx, _, _resid, D = _tables(torch, zoomhash, mode, L, k, w, 5 + k)
    ctx.set_query_opts(cap=16, proj=proj)
    alpha, beta = lsh.hash_params(5 + k, L, k, D, w)
    g = np.random.default_rng(100 + k)
    # the last size is past the line from which a wave takes two row tiles
    for n, off, scale in [(1, 0, 8.0), (17, 1, 8.0), (129, 4, 8.0), (95, 0, 4e5), (2085, 2, 8.0), (2085, 0, 4e3),
                          (32768 + 37, 0, 30.0)]:
        if n > 4000 and L * k > 64:
            continue
        x = (g.standard_normal((n, D)) * scale).astype(np.float32)
        if n > 100:
            x[3] = 0.0
            x[5] *= np.float32(1e-30)
        buf = torch.zeros(n * D + off, dtype=torch.float32, device="cuda")
        buf[off:] = torch.from_numpy(x.reshape(-1)).cuda()
        codes = torch.empty((n, L * k), dtype=torch.int32, device="cuda")
        keys = torch.empty((n, L), dtype=torch.int64, device="cuda")
        ctx.hash(2, buf[off:].view(n, D), n, codes, keys)
        ctx.sync()
        ref = lsh.codes(x, alpha, beta, w)
        assert np.array_equal(codes.cpu().numpy(), ref), (n, off, scale)
        kref = lsh.bucket_keys(ref, L, k)
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), kref), (n, off, scale)
        keys.zero_()   # without the codes
        ctx.hash(2, buf[off:].view(n, D), n, None, keys)
        ctx.sync()
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), kref), (n, off, scale)
