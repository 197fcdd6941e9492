"""Millions of records, over many small frames of one pose, where the offsets'
scan changes its way of working."""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames", [4096, 4097])  # 4096 records each
def test_offsets_over_many_blocks(frames):
    """Up to 4,096 blocks of 4,096 records each adds up the sums in front of it,
    beyond a kernel does: every frame's image is that of the frame alone, and the
    keys are as many times its keys."""
    import torch
    from gpu_util import to_dev
    from paper_2411_17660_amd.raster import Rasterizer
    n, W, H = 4096, 40, 24
    sc = scenes.tiny_scene(seed=4, n=n, W=W, H=H, f=30.0, sh_degree=0, ls_mean=-3.0)
    means = np.array(sc.means)
    means[200:] = np.nan  # culled
    sc.means = means
    d = to_dev(sc)
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh")]
    rast = Rasterizer(0)
    one = [x.clone() for x in rast.forward(*args, d["poses"], sc.cams, 0, sc.background)]
    keys = rast.stats()["n_keys"]
    assert keys > 200
    poses = d["poses"].expand(frames, 3, 4).contiguous()
    many = rast.forward(*args, poses, list(sc.cams) * frames, 0, sc.background)
    st = rast.stats()
    assert st["n_records"] == frames * n and st["n_keys"] == frames * keys
    for a, b in zip(one, many):
        assert torch.equal(b.view(frames, -1), a[None].expand(frames, -1))


def test_capture_of_fewer_records():
    """Just below 2^22 records the scan takes its sums in smaller blocks; a
    capture there after an uncaptured call just above needs no more workspace."""
    import torch
    from gpu_util import to_dev
    from paper_2411_17660_amd.raster import Rasterizer
    from test_gpu_capture_sizes import _check_capture
    n, W, H = 4096, 40, 24
    sc = scenes.tiny_scene(seed=4, n=n, W=W, H=H, f=30.0, sh_degree=0, ls_mean=-3.0)
    means = np.array(sc.means)
    means[200:] = np.nan
    sc.means = means
    d = to_dev(sc)
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh")]

    def fit(r, frames):
        poses = d["poses"].expand(frames, 3, 4).contiguous()
        out = tuple(torch.empty(k * W * H * frames, device="cuda") for k in (3, 1, 1))

        def call():
            r.forward(*args, poses, list(sc.cams) * frames, 0, sc.background,
                      key_capacity=2000000, out=out)
        return list(out), call
    rast = Rasterizer(0)
    fit(rast, 1025)[1]()
    outputs, call = fit(rast, 1024)
    _check_capture(rast, outputs, call, *fit(Rasterizer(0), 1024))
