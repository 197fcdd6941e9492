"""The test of an entry against an 8 x 8 block (its ellipse against the part of
the block in its box) drops nothing that a pixel would blend: a forward that
counts its pairs visits every entry in its box, and its images are bitwise
those of one that culls.  Thin, tilted, faint and near entries, where the
ellipse and its margins are tight or give way to the box."""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu

CASES = [dict(), dict(zrange=(0.21, 0.6)), dict(opacity=-4.5), dict(opacity=6.0),
         dict(ls_mean=-4.5), dict(ls_mean=0.5)]


@pytest.fixture(scope="module")
def rast():
    from paper_2411_17660_amd.raster import Rasterizer
    return Rasterizer(0)


def _scene(W, H, case):
    kw = dict(dict(ls_mean=-2.2, zrange=(1.5, 4.0)), **case)
    shift = kw.pop("opacity", 0.0)
    sc = scenes.tiny_scene(seed=3, n=400, W=W, H=H, f=0.7 * W, sh_degree=1, ls_sigma=0.5,
                           opacity_sigma=1.0, **kw)
    sc.opacity = sc.opacity + np.float32(shift)
    return sc


def _same(forward):
    import torch
    a = [x.clone() for x in forward(False)]
    b = forward(True)
    for x, y in zip(a, b):
        assert torch.isfinite(x).all() and torch.equal(x, y)
    assert float(a[2].max()) > 0


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16)])
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("thin", [0.0, 2.0, 4.0])
def test_gaussians(rast, thin, case, tile):
    """thin: natural logarithm of the axes' ratio."""
    from gpu_util import to_dev
    sc = _scene(333, 250, case)
    ls = np.array(sc.log_scales)
    ls[:, 1:] -= thin
    sc.log_scales = ls
    d = to_dev(sc)
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")]
    _same(lambda count: rast.forward(*args, sc.cams, sc.sh_degree, sc.background, tile=tile,
                                     count_pairs=count))


@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16)])
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("tilt", [0.2, 1.5, 20.0])
@pytest.mark.parametrize("thin", [0.0, 3.0])
def test_surfels(rast, thin, tilt, case, tile):
    """tilt: size of the quaternions' vector parts against their 1."""
    import torch
    from gpu_util import to_dev
    sc = _scene(333, 250, case)
    d = to_dev(sc)
    d["log_scales"] = d["log_scales"][:, :2].contiguous()
    d["log_scales"][:, 1] -= thin
    q = torch.randn(sc.n, 4, generator=torch.Generator().manual_seed(1)) * tilt
    q[:, 0] = 1.0
    d["quats"] = q.cuda()
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")]
    _same(lambda count: rast.forward_surfel(*args, sc.cams, sc.sh_degree, sc.background,
                                            tile=tile, count_pairs=count))
