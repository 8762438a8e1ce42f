"""A tuning choice that other kernels timed is not taken from the cache: entries
keyed before the update's persistent workgroups went."""
import ctypes

import pytest

import synthdata

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1
GOLDEN = 0x9E3779B97F4A7C15


def _fmix64(z):
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9 & M64
    z = (z ^ (z >> 27)) * 0x94D049BB133111EB & M64
    return z ^ (z >> 31)


def _key(torch, kernels, sizes, K, iters, opts):
    rt = ctypes.c_int()
    assert ctypes.CDLL("libamdhip64.so").hipRuntimeGetVersion(ctypes.byref(rt)) == 0
    prop = torch.cuda.get_device_properties(0)
    h = _fmix64(0x5A17 + rt.value + ((kernels - 1) << 32) & M64)
    for v in [*prop.name.encode(), *prop.gcnArchName.encode(), len(sizes), *[x for s in sizes for x in s], K, iters, *opts]:
        h = _fmix64(h ^ (v + GOLDEN & M64))
    return h


def test_older_kernels_choice(tmp_path, monkeypatch):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    from paper_1004_3980_amd.pipeline import GpuWorkload
    g = GpuWorkload(synthdata.scaled(synthdata.WORKLOADS["diff"], dict_images=4, dict_hr=96, n_dict=2000, L=4, k=6,
                                     test_h=24, test_w=24, cap=16))
    sizes = [(31, 40, 2), (24, 29, 2)]
    lrs = [torch.from_numpy(synthdata.fractal_voronoi_image(i, h, w)).cuda() for i, (h, w, _) in enumerate(sizes)]
    outs = [torch.empty((2 * h, 2 * w), device="cuda") for h, w, _ in sizes]
    g.set_mode(cap=16, rerank=0, proj=1, lle_fp64=1)
    path = tmp_path / "tune.jsonl"
    monkeypatch.setenv("ZH_TUNE_CACHE", str(path))

    def tune(kernels):
        key = _key(torch, kernels, sizes, 4, 2, (16, 0, 1, 1))
        path.write_text('{"key": "%016x", "bp_tile": 16, "bp_grid_per_cu": 2, "synth_rows": 4}\n' % key)
        return g.ctx.tune_batch(lrs, outs, [2, 2], 4, 1e-3, 2, 1.5, 0.1)

    assert tune(1)["from_cache"] == 0
    info = tune(2)   # the key as it is now, which shows that the one above was the older one
    assert info["from_cache"] == 1 and (info["bp_tile"], info["bp_grid_per_cu"], info["synth_rows"]) == (16, 2, 4)
