"""The rendering loss at the sizes where its work is cut: strips of 118 output
columns, segments of 11 c - 22 rows chosen by the batch, single pixels, frames
of unlike sizes, against the FP64 oracle; and a colour gradient written over an
input image.

The kernel works in FP64 from FP32 inputs and rounds once: 1e-6 relative per
element, plus 1e-10 of the largest entry where two FP64 evaluations cancel."""
import numpy as np
import pytest

import oracle
from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rast():
    from paper_2411_17660_amd.raster import Rasterizer
    return Rasterizer()


def _close(name, got, ref):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    bound = 1e-6 * np.abs(ref) + 1e-10 * (np.abs(ref).max() if ref.size else 0.0)
    assert np.all(np.abs(got - ref) <= bound), name


@pytest.mark.parametrize("sizes", [[(1, 1)], [(5, 7)], [(117, 11)], [(118, 12)], [(119, 33)],
                                   [(128, 45), (236, 10)], [(237, 131)], [(355, 267), (3, 200)],
                                   [(64, 48)] * 5 + [(121, 90)]])
def test_loss_units_match_oracle(rast, sizes):
    import torch
    from gpu_util import gpu_forward
    gpu_forward(rast, scenes.layout_scene(sizes))
    imgs = scenes.loss_images(11, sizes, depth_invalid=0.2)
    l1, l2 = float(np.float32(0.8)), float(np.float32(0.2))
    loss, g_rgb, g_dep, g_alp, ssim = oracle.render_loss(*imgs, l1, l2, sizes)
    dev = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in imgs]
    out = rast.loss_render(*dev, l1, l2)
    for name, ref in (("loss", loss), ("g_rgb", g_rgb), ("g_depth", g_dep), ("g_alpha", g_alp),
                      ("ssim", ssim)):
        _close(name, out[name].cpu().numpy(), np.reshape(ref, -1))
    # over the rendered image, and over the target
    for k in (0, 2):
        im = [t.clone() for t in dev]
        o = dict(out, g_rgb=im[k])
        rast.loss_render(*im, l1, l2, out={n: (t if n == "g_rgb" else t.clone())
                                           for n, t in o.items()})
        assert torch.equal(im[k], out["g_rgb"])
