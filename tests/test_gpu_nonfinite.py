"""An upstream gradient that is not finite, or whose product with an entry's
values overflows FP32, reaches through an entry's alpha gradient only what that
feeds: the SH gradients, which are sums of the colour gradients times blending
weights, stay bitwise as they are without it, and so does every gradient of a
Gaussian that no such pixel sees.  (A key's sums over its pixels are matrix
products, whose zeros must not meet the bad value.)  Both primitives, each
number of blocks per backward wave, and lists in segments."""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu

NAN, INF = float("nan"), float("inf")
BIG = 3e38  # finite; times a depth or distortion weight above 1.2 it is not in FP32
# one block per wave (and the lists in segments), two, four
SIZES = [((40, 30), 150, -2.6), ((85, 61), 3000, -1.5), ((785, 689), 150, -2.6),
         ((1030, 1025), 150, -2.6)]


@pytest.fixture(scope="module")
def rast():
    from paper_2411_17660_amd.raster import Rasterizer
    return Rasterizer(0)


def _check(good, got, bad):
    assert np.isfinite(good["means"]).all()
    hit = ~np.isfinite(got["means"]).all(1)
    assert hit.any() and not hit.all()
    assert np.array_equal(good["sh"], got["sh"])
    if bad == BIG:  # (an entry near the depth behind it keeps a finite product)
        return
    for k in ("means", "log_scales", "quats", "opacity"):
        assert np.array_equal(good[k][~hit], got[k][~hit]), k


@pytest.mark.parametrize("channel,bad", [("alpha", NAN), ("alpha", INF), ("depth", NAN),
                                         ("depth", -INF), ("depth", BIG)])
@pytest.mark.parametrize("size,n,ls_mean", SIZES)
def test_gaussians(rast, size, n, ls_mean, channel, bad):
    from gpu_util import gpu_backward, gpu_forward
    W, H = size
    sc = scenes.tiny_scene(seed=5, n=n, W=W, H=H, f=0.7 * max(W, H), sh_degree=1,
                           ls_mean=ls_mean, ls_sigma=0.5)
    G = [np.array(x) for x in scenes.upstream(6, sc)]
    gpu_forward(rast, sc)
    good = gpu_backward(rast, G)
    at = H // 2 * W + W // 2
    G[2 if channel == "alpha" else 1][at:at + 3] = bad
    gpu_forward(rast, sc)
    _check(good, gpu_backward(rast, G), bad)


@pytest.mark.parametrize("channel,bad", [(2, NAN), (2, INF), (1, INF), (1, BIG), (3, NAN),
                                         (4, INF)])
@pytest.mark.parametrize("size,n,ls_mean", SIZES)
def test_surfels(rast, size, n, ls_mean, channel, bad):
    """channel: the upstream of rgb, depth, alpha, normal, dist."""
    import torch
    from gpu_util import to_dev
    W, H = size
    sc = scenes.tiny_scene(seed=5, n=n, W=W, H=H, f=0.7 * max(W, H), sh_degree=1,
                           ls_mean=ls_mean, ls_sigma=0.5)
    d = to_dev(sc)
    d["log_scales"] = d["log_scales"][:, :2].contiguous()
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")]
    gen = torch.Generator().manual_seed(2)
    G = [torch.randn(k * W * H, generator=gen).cuda() for k in (3, 1, 1, 3, 1)]

    def run():
        rast.forward_surfel(*args, sc.cams, sc.sh_degree, sc.background)
        g = rast.backward_surfel(*G)
        return {k: v.cpu().numpy() for k, v in g.items()}
    good = run()
    at = H // 2 * W + W // 2
    G[channel][at:at + 3] = bad
    _check(good, run(), bad)
