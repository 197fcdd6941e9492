"""The ordering of records and tile keys at the sizes where its method
changes: counting (up to 16384 records, 8192 tile keys, 4096 records of the
size classes), passes whose scatter walks the digit columns, and passes with
column kernels.

- The tile lists are those of a stable sort of the slots by tile in depth
  order, and the ranges are their bounds.
- Culled Gaussians appended to a scene take every stage across its line and
  leave the images and gradients bitwise as they were.
"""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu


def _scene(n, seed, extra=0, F=1):
    W, H = 200, 150
    sc = scenes.tiny_scene(seed=seed, n=n, W=W, H=H, f=160.0, n_frames=F, sh_degree=0, ls_mean=-5.0,
                           ls_sigma=0.8, opacity_sigma=1.0)
    if extra:  # not finite: culled in every frame
        for k in ("means", "log_scales", "quats", "opacity", "sh"):
            a = getattr(sc, k)
            pad = np.repeat(a[:1], extra, axis=0)
            if k == "means":
                pad = np.full_like(pad, np.nan)
            setattr(sc, k, np.concatenate([a, pad]))
    return sc


@pytest.fixture(scope="module")
def rast():
    from paper_2411_17660_amd.raster import Rasterizer
    return Rasterizer()


@pytest.mark.parametrize("n,F", [(1, 1), (63, 1), (64, 1), (65, 2), (700, 3), (2731, 3),
                                 (8191, 1), (8193, 1), (16384, 1), (16385, 1), (33000, 2),
                                 (150000, 2)])
def test_lists_are_the_stable_order(rast, n, F):
    from gpu_util import gpu_forward
    gpu_forward(rast, _scene(n, 5, F=F))
    L = rast.debug_lists()
    T = rast.stats()["n_tiles"]
    keys, vals, nt = L["tile_keys"].astype(np.int64), L["tile_vals"].astype(np.int64), L["ntiles"]
    assert len(keys) == int(nt.sum())
    # every record once per tile of its rect
    np.testing.assert_array_equal(np.bincount(vals, minlength=n * F), nt)
    # tiles ascend, and inside a tile (depth, record)
    dk = L["depth_key"].astype(np.int64)[vals]
    np.testing.assert_array_equal(np.lexsort((vals, dk, keys)), np.arange(len(keys)))
    want = np.stack([np.searchsorted(keys, np.arange(T)),
                     np.searchsorted(keys, np.arange(T), side="right")], 1)
    want[want[:, 0] == want[:, 1]] = 0
    np.testing.assert_array_equal(L["ranges"].reshape(T, 2), want)


@pytest.mark.parametrize("n,extra", [(1, 63), (1, 64), (500, 3596), (500, 3597), (500, 7692),
                                     (5000, 12000), (5000, 300000)])
def test_culled_records_change_nothing(rast, n, extra):
    import torch
    from gpu_util import gpu_forward
    P = 200 * 150
    gen = torch.Generator().manual_seed(3)
    G = [torch.randn(k * P, generator=gen).cuda() for k in (3, 1, 1)]
    out = []
    for e in (0, extra):
        _, *im = gpu_forward(rast, _scene(n, 9, e))
        g = rast.backward(*G)
        out.append(([x.clone() for x in im], g))
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)
    for k, a in out[0][1].items():
        if k == "twist":  # its sum over the Gaussians runs in waves of their count
            assert float((a - out[1][1][k]).norm()) <= 1e-6 * float(a.norm())
        else:
            assert torch.equal(a, out[1][1][k][:n]), k
            assert not out[1][1][k][n:].any()


@pytest.mark.parametrize("blocks", [1254, 1255])
def test_digit_columns_of_many_blocks(rast, blocks):
    """5 digit bits (30 tiles, every one under every Gaussian), blocks of 4096
    keys: the last count of blocks whose scatter walks the columns, and the
    first whose columns have kernels."""
    from gpu_util import gpu_forward
    n = (blocks * 4096) // 30
    assert -(-n * 30 // 4096) == blocks
    sc = scenes.tiny_scene(seed=2, n=n, W=96, H=80, f=80.0, sh_degree=0, ls_mean=2.0, ls_sigma=0.1)
    sc.opacity = np.full_like(sc.opacity, -3.0)
    gpu_forward(rast, sc)
    L = rast.debug_lists()
    keys, vals, nt = L["tile_keys"].astype(np.int64), L["tile_vals"].astype(np.int64), L["ntiles"]
    dk = L["depth_key"].astype(np.int64)
    kept = nt > 0
    assert (nt[kept] == 30).all() and -(-len(keys) // 4096) == blocks
    # each tile's list: the kept records by (depth, index)
    order = np.lexsort((np.arange(n), dk))[:kept.sum()]
    np.testing.assert_array_equal(keys, np.repeat(np.arange(30), kept.sum()))
    np.testing.assert_array_equal(vals.reshape(30, -1), np.broadcast_to(order, (30, len(order))))


@pytest.mark.parametrize("n", [0, 100, 16384, 16385])
def test_every_stage_of_a_forward_is_timed(rast, n):
    from gpu_util import gpu_forward
    rast.timings()
    gpu_forward(rast, _scene(n, 5), timing=True)
    t = rast.timings()
    for stage in ("preprocess", "depth_sort", "offsets", "keygen", "tile_sort", "ranges",
                  "composite_fwd"):
        assert t[stage][1] == 1, stage
