"""Compositing over 8 x 8 pixel blocks against the oracle where it can go
wrong: every number of blocks per backward wave (chosen by the tile count),
images that end inside a block or a tile, entries that only graze a block
(thin, rotated Gaussians), lists around the batch of 64 entries, and the
median depth on each path.  Bars: those of the parity tests (lists and stop
positions bit-exact, images 1e-4 absolute on unflagged pixels, gradients 1e-3
relative with the oracle's noise term)."""
import numpy as np
import pytest

from paper_2411_17660_amd import scenes
from test_gpu_parity import check_backward, check_forward

pytestmark = pytest.mark.gpu

# (W, H), tile: a backward wave takes as many blocks (up to 4) as leave 4,096
# waves, so 16x16 tiles take one block below 2,048 of them, two below 4,096
# and four beyond
SHAPES = [((33, 17), (16, 16)), ((8, 8), (8, 8)), ((785, 689), (16, 16)),
          ((1030, 1025), (16, 16)), ((1025, 513), (32, 16)), ((1030, 530), (16, 8)),
          ((1031, 1025), (32, 8)), ((523, 509), (8, 8))]


@pytest.fixture(scope="module")
def rast():
    from paper_2411_17660_amd.raster import Rasterizer
    return Rasterizer(0)


@pytest.mark.parametrize("median", [False, True])
@pytest.mark.parametrize("size,tile", SHAPES)
def test_blocks_match_oracle(rast, size, tile, median):
    W, H = size
    for n, thin in ((63, True), (65, False), (200, True)):
        label = f"blocks {W}x{H}/{tile[0]}x{tile[1]} n{n}"
        sc = scenes.tiny_scene(seed=n, n=n, W=W, H=H, f=0.7 * max(W, H), sh_degree=1,
                               ls_mean=-2.2, ls_sigma=0.5, opacity_sigma=1.5)
        if thin:  # 20 : 1 needles at random angles: most of their box is empty
            ls = np.array(sc.log_scales)
            ls[:, 1:] = ls[:, :1] - 3.0
            sc.log_scales = np.ascontiguousarray(ls, np.float32)
        ref, _, flags = check_forward(rast, sc, tile=tile, label=label, median=median)
        check_backward(rast, sc, ref, flags, n, label=label)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("size", [(40, 30), (785, 689), (1030, 1025)])
def test_nonfinite_upstream_stays_in_its_channel(rast, size, bad):
    """A red upstream gradient that is not finite at some pixels leaves the
    green and blue SH gradients and the gradients of Gaussians that reach none
    of those pixels bitwise as they are without it (the sums over pixels are
    matrix products, whose zeros must not meet it)."""
    from gpu_util import gpu_backward, gpu_forward
    W, H = size
    sc = scenes.tiny_scene(seed=5, n=150, W=W, H=H, f=0.7 * max(W, H), sh_degree=1,
                           ls_mean=-2.6, ls_sigma=0.5)
    G = [np.array(x) for x in scenes.upstream(6, sc)]
    gpu_forward(rast, sc)
    good = gpu_backward(rast, G)
    py, px = H // 2, W // 2
    G[0][py * W + px:py * W + px + 3] = bad
    gpu_forward(rast, sc)
    got = gpu_backward(rast, G)
    assert np.array_equal(good["sh"][:, :, 1:], got["sh"][:, :, 1:])
    hit = ~np.isfinite(got["means"]).all(1)
    assert hit.any() and not hit.all()
    for k in ("means", "log_scales", "quats", "opacity", "sh"):
        assert np.array_equal(good[k][~hit], got[k][~hit]), k


# surfel lists of each backward path (1, 2 and 4 blocks per wave), ragged
# images, and disks seen at a grazing angle (their block test falls back to
# the box)
@pytest.mark.parametrize("tilt", [0.2, 1.5])
@pytest.mark.parametrize("size,tile", [((40, 29), (16, 16)), ((523, 500), (8, 8)),
                                       ((785, 689), (16, 16)), ((1030, 1025), (16, 16)),
                                       ((1025, 513), (32, 16))])
def test_surfel_blocks_do_not_depend_on_the_path(rast, size, tile, tilt):
    """The five images are bitwise those of the 8x8 tiles (one block per tile),
    and the gradients agree to FP32 rounding of their FP64 sums."""
    import torch
    from gpu_util import to_dev
    W, H = size
    sc = scenes.tiny_scene(seed=3, n=150, W=W, H=H, f=0.7 * max(W, H), sh_degree=1,
                           ls_mean=-2.2, ls_sigma=0.5, opacity_sigma=1.5)
    d = to_dev(sc)
    d["log_scales"] = d["log_scales"][:, :2].contiguous()
    q = torch.randn(sc.n, 4, generator=torch.Generator().manual_seed(1)) * tilt
    q[:, 0] = 1.0
    d["quats"] = q.cuda()
    args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")]
    P = W * H
    gen = torch.Generator().manual_seed(2)
    G = [torch.randn(k * P, generator=gen).cuda() for k in (3, 1, 1, 3, 1)]
    out = []
    for t in ((8, 8), tile):
        im = rast.forward_surfel(*args, sc.cams, sc.sh_degree, sc.background, tile=t)
        out.append(([x.clone() for x in im], rast.backward_surfel(*G)))
    torch.cuda.synchronize()
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)
    # a key's sums are FP64 and stored as FP32, then summed over keys in FP64
    # and passed through the (linear) chain rule: 2^-24 of the largest term
    for k, a in out[0][1].items():
        b = out[1][1][k]
        err = float((a.double() - b.double()).norm() / a.double().norm())
        assert err <= 2e-5, (k, err)


# Lists worked on in segments (few tiles, lists of two batches and more) against
# the same image inside a batch of frames, which takes them whole: lists shorter
# and longer than the eight segments' batches, and pixels that stop in each of them.
@pytest.mark.parametrize("surfel", [False, True])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 16)])
@pytest.mark.parametrize("n,ls_mean,sigma", [(400, -1.2, 0.2), (3000, -1.5, 3.0),
                                             (3000, -1.0, -2.5)])
def test_segments_do_not_change_the_gradients(rast, n, ls_mean, sigma, tile, surfel):
    import torch
    from gpu_util import to_dev
    W, H, F = 85, 61, 28
    sc = scenes.tiny_scene(seed=8, n=n, W=W, H=H, f=0.8 * W, sh_degree=0, ls_mean=ls_mean,
                           ls_sigma=0.3, opacity_sigma=0.5)
    d = to_dev(sc)
    d["opacity"] += sigma
    if surfel:
        d["log_scales"] = d["log_scales"][:, :2].contiguous()
    P = W * H
    gen = torch.Generator().manual_seed(5)
    G = [torch.randn(k * P, generator=gen).cuda() for k in ((3, 1, 1, 3, 1) if surfel
                                                            else (3, 1, 1))]
    out = []
    for frames in (1, F):
        poses = d["poses"].expand(frames, 3, 4).contiguous()
        cams = [sc.cams[0]] * frames
        args = [d[k] for k in ("means", "log_scales", "quats", "opacity", "sh")] + [poses, cams]
        # the first frame carries the gradient, the others none
        Gs = [torch.cat([g, g.new_zeros(g.numel() * (frames - 1))]) for g in G]
        if surfel:
            rast.forward_surfel(*args, sc.sh_degree, sc.background, tile=tile)
            g = rast.backward_surfel(*Gs)
        else:
            rast.forward(*args, sc.sh_degree, sc.background, tile=tile)
            g = rast.backward(*Gs)
        st = rast.stats()
        assert st["n_keys"] >= 128 * st["n_tiles"]
        waves = st["n_tiles"] * tile[0] * tile[1] // 64
        assert (waves <= 1536) == (frames == 1)
        out.append(g)
    out[1]["twist"] = out[1]["twist"][:1]
    # T and E reach a segment through FP64 products instead of FP32 steps: 2^-24
    # per entry in front of the stop, which is at most ln(1e-4) / ln(1 - 1/255)
    # = 2350 entries deep, random in sign: 3e-6 of a term; terms cancel tenfold
    for k, a in out[0].items():
        b = out[1][k]
        err = float((a.double() - b.double()).norm() / b.double().norm())
        assert err <= 3e-5, (k, err)
