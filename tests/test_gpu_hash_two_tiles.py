"""Codes and keys where a wave of the split-bf16 projection takes two row tiles: from
ceil(n / 128) parts >= 512 on, the tables in one part there. Odd table counts, hashes
that do not fill a tile, rows off 16-byte boundaries, a second tile that is full,
ragged, one row or empty, with and without the codes, and features whose lists run
over. Bitwise against the oracle, as the codes are defined by the FP64 sum."""
import numpy as np
import pytest

from oracle import lsh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,L,k", [(0, 5, 8), (0, 3, 13), (0, 1, 1), (1, 3, 7), (1, 3, 20), (1, 2, 13), (1, 1, 32)])
def test_two_row_tiles(mode, L, k):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    D, w = (25, 100)[mode], 16.0
    g = np.random.default_rng(k)
    ctx = zb.Context(0)
    feat = torch.from_numpy(g.standard_normal((300, D)).astype(np.float32) * 8).cuda()
    resid = torch.zeros((300, 100), device="cuda")
    ctx.build_tables(feat, resid, 300, D, 2, mode, L, k, w, 5 + k)
    ctx.set_query_opts(cap=16, proj=1)
    alpha, beta = lsh.hash_params(5 + k, L, k, D, w)
    # rows of the last workgroup (128 rows, 32 a wave), offset in floats, scale; the last: the lists run over
    for rows, off, scale in [(1, 0, 8.0), (17, 1, 8.0), (32 + 16, 0, 8.0), (96 + 29, 2, 8.0), (128, 4, 8.0), (77, 0, 4e4)]:
        n = 511 * 128 + rows
        assert -(-n // 128) >= 512
        x = (g.standard_normal((n, D)) * scale).astype(np.float32)
        x[n - 1] *= np.float32(1e-30)
        x[70] = 0.0
        buf = torch.zeros(n * D + off, device="cuda")
        buf[off:] = torch.from_numpy(x.reshape(-1)).cuda()
        v = buf[off:].view(n, D)
        codes = torch.empty((n, L * k), dtype=torch.int32, device="cuda")
        keys = torch.empty((n, L), dtype=torch.int64, device="cuda")
        ctx.hash(2, v, n, codes, keys)
        ctx.sync()
        ref = lsh.codes(x, alpha, beta, w)
        kref = lsh.bucket_keys(ref, L, k)
        assert np.array_equal(codes.cpu().numpy(), ref), (rows, off, scale)
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), kref), (rows, off, scale)
        keys.zero_()
        ctx.hash(2, v, n, None, keys)
        ctx.sync()
        assert np.array_equal(keys.cpu().numpy().view(np.uint64), kref), (rows, off, scale)
    if L > 2:   # a list takes 32 tables of 16 rows
        assert ctx.stats()["codes_fixed"] > 32 * n // 16, "the last size's lists run over"
