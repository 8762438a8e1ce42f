"""Memory of a table build: what a context keeps after it, and the limit that a
build fits into; and the bins of a table whose sort takes three passes (the
sorted values end where the IDs are kept, whatever the number of passes)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _own(n, D, L):
    """Bytes of a dictionary and its tables."""
    cap = 1
    while cap < 2 * n:
        cap *= 2
    return n * (2 * ((D + 3) // 4 * 4 + 11 & ~7) + 2 * D + 4 * D + 64 + 4 * L) + L * cap * 16 + L * cap // 2


def _context():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd import zoomhash as zb
    return torch, zb


def test_kept_after_a_build():
    torch, zb = _context()
    n, L = 300_000, 24
    feat = torch.randn((n, 25), device="cuda") * 4
    resid = torch.zeros((n, 25), device="cuda")
    ctx = zb.Context(0)
    ctx.build_tables(feat[:100], resid[:100], 100, 25, 1, 0, 2, 2, 8.0, 1)   # the library's own first allocations
    ctx.sync()
    free = torch.cuda.mem_get_info()[0]
    kept = []
    for _ in range(8):   # the runtime gives freed memory back when it gets to it
        ctx.build_tables(feat, resid, n, 25, 1, 0, L, 8, 8.0, 1)
        ctx.sync()
        time.sleep(0.05)
        kept.append(free - torch.cuda.mem_get_info()[0])
    kept = min(kept)
    # the lists of the hash kernels (32 bytes a row and the masks), the basis' 8 MB, whole pages
    assert kept <= _own(n, 25, L) + 48 * n + (32 << 20), (kept, _own(n, 25, L))


@pytest.mark.parametrize("mode,n,L", [(1, 100_000, 24), (0, 200_000, 16), (0, 3000, 8)])
def test_fits_a_limit(monkeypatch, mode, n, L):
    torch, zb = _context()
    D = 25 if mode == 0 else 100
    feat = torch.randn((n, D), device="cuda") * 4
    resid = torch.zeros((n, 25), device="cuda")
    # keys, slots of one table, the hash kernels' lists (few rows: in several parts), counts, parameters; or the basis first
    need = max(_own(n, D, L) + 8 * n * L + 4 * n + max(48 * n, 2 << 20) + (3 << 19),
               n * (8 * D + 128) + (10 << 20))
    monkeypatch.setenv("ZH_MEM_LIMIT", str(need))
    ctx = zb.Context(0)
    ctx.build_tables(feat, resid, n, D, 1, mode, L, 8, 8.0, 1)
    ctx.sync()


# slots of 22, 23 and 24 bits: two passes, three, three; and of 11 and 12: one, two
@pytest.mark.parametrize("n,L", [(2_000_000, 2), (2_200_000, 3), (4_300_000, 1), (1000, 9), (1100, 9)])
def test_passes_of_the_sort(tmp_path, n, L):
    torch, zb = _context()
    g = torch.Generator(device="cuda").manual_seed(n)
    feat = torch.randn((n, 25), device="cuda", generator=g) * 2
    feat[::7] = feat[0]          # a bin of many rows
    resid = torch.zeros((n, 25), device="cuda")
    ctx = zb.Context(0)
    ctx.build_tables(feat, resid, n, 25, 1, 0, L, 2, 4.0, 3)
    keys = torch.empty((n, L), dtype=torch.int64, device="cuda")
    ctx.hash(1, feat, n, None, keys)
    ctx.sync()
    keys = keys.cpu().numpy().view(np.uint64)
    ctx.save_tables(1, str(tmp_path / "t"))
    tail = 64 * n + 2 * (2 * 64 * 32)     # screen rows, the two planes of Phi
    size = (tmp_path / "t").stat().st_size
    ids = np.fromfile(tmp_path / "t", dtype=np.uint32, offset=size - tail - 4 * L * n, count=L * n).reshape(L, n)
    entropy = ctx.table_entropy(1, L)
    for l in range(L):
        assert np.array_equal(np.sort(ids[l]), np.arange(n, dtype=np.uint32))
        k = keys[ids[l], l]
        first = np.concatenate(([True], k[1:] != k[:-1]))
        _, counts = np.unique(keys[:, l], return_counts=True)
        assert first.sum() == len(counts)                                  # each bin in one piece
        assert (np.diff(ids[l].astype(np.int64))[~first[1:]] > 0).all()     # IDs ascending in it
        p = counts / n
        assert abs(entropy[l] + (p * np.log2(p)).sum()) <= 1e-12 * np.log2(n)
