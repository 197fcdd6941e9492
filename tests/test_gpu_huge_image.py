"""The largest frame that the entry points take, 65535 x 65535: its 2^32 pixels
are more threads than one launch may have.  Against the frame without its first
16 rows, which is not.  Needs 130 GB on the card."""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu

SIDE, F, CUT = 65535, 60000.0, 16


def test_largest_frame():
    import torch
    from gpu_util import to_dev
    from paper_2411_17660_amd.raster import Rasterizer
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("130 GB of device memory")
    c = 32767.5
    at = [(3, 40), (32770, 40001), (65530, 65529)]
    sc = scenes.tiny_scene(seed=1, n=3, W=32, H=32, f=30.0, sh_degree=0, ls_mean=-9.0, ls_sigma=0.1)
    z = 2.0
    sc.means = np.array([((x - c) * z / F, (y - c) * z / F, z) for x, y in at], np.float32)
    sc.poses = np.eye(3, 4, dtype=np.float32)[None]
    d = to_dev(sc)
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")]

    def render(rows, cy):
        """Windows around the Gaussians and the number of pixels they cover."""
        P = SIDE * rows
        out = tuple(torch.full((k * P,), float("nan"), device="cuda") for k in (3, 1, 1))
        rast = Rasterizer(0)
        rast.forward(*args, [(SIDE, rows, F, F, c, cy, 0.2)], 0, sc.background, out=out)
        windows = []
        for x, y in at:
            x0, y0 = max(x - 20, 0), y - 20 - (SIDE - rows)
            windows += [im.view(-1, rows, SIDE)[:, y0:y0 + 40, x0:x0 + 40].clone() for im in out]
        lit = int((out[2] > 0).sum())
        assert int((out[2] >= 0).sum()) == P
        for k in range(3):
            bg = torch.tensor(sc.background[k], device="cuda")
            assert int((out[0][k * P:(k + 1) * P] == bg).sum()) >= P - lit
        return windows, lit
    ref, lit = render(SIDE - CUT, c - CUT)
    torch.cuda.empty_cache()
    got, lit_got = render(SIDE, c)
    torch.cuda.empty_cache()
    assert lit == lit_got and lit > 100
    for a, b in zip(got, ref):
        # the projected centres are the same, their FP32 hi/lo split is not
        assert float((a - b).abs().max()) <= 1e-5
    for k in (2, 5, 8):
        assert float(got[k].max()) > 0.1
