"""Representative workloads of the rasterizer, for timing and for comparing outputs.

Each case is one call (or one short chain of calls) that a mapping system
makes through the package's public entry points, on a seeded synthetic scene:
means on a piecewise-planar depth map seen from a smooth camera trajectory,
as the mapper initialises them from the tracker's depth.

  render  one no-grad rasterize() of the map (evaluation, preview)
  fit     rasterize() and its backward through torch.autograd
  step    forward + loss + backward in one call at a fixed key capacity, the
          inner loop of the mapper ("l1" or "render" = L1 + SSIM loss);
          `graph` replays it as a captured HIP graph
  surfel  the 2D surfel objective: forward, rendering loss, normal
          consistency, backward
  loss    the rendering loss alone on given images
  update  what follows each backward: densification statistics, the Adam
          step with the pose fold, the MCMC position noise

listed() names the cases, draw() gives more of the same ranges, prepare()
makes what a program holds before the call, run() makes the call, work()
says what it cannot do without, and exact() gives its outputs in 64 bits
from plain torch.
"""
import math

import numpy as np
import torch

from paper_2411_17660_amd.raster import Rasterizer, rasterize

DEV = "cuda"
NEAR = 0.2
PARAMS = ("means", "log_scales", "quats", "opacity", "sh")
LAMBDA1, LAMBDA2 = 0.9, 0.2        # rendering loss: colour share, SSIM share
W_NORMAL, W_DIST = 0.05, 100.0     # surfel objective
LRS = dict(lr_means=1.6e-4, lr_sh=5e-3, lr_pose=1e-3)


def _case(name, op, n, frames, width, height, sh, size=-4.0, tile="16x16", mixed=False,
          heavy=False, median=False, loss="", graph=False):
    return dict(name=name, op=op, n=n, frames=frames, width=width, height=height, sh=sh,
                size=size, tile=tile, mixed=mixed, heavy=heavy, median=median, loss=loss,
                graph=graph)


def listed():
    return [
        # a just-started map shown as a thumbnail: the smallest call, all latency
        _case("view-small", "render", 2000, 1, 128, 96, 0, size=-3.0),
        # two ragged thumbnails fitted through autograd: launches and host work
        _case("fit-small", "fit", 3000, 2, 131, 97, 1, size=-3.0),
        # evaluation of one VGA keyframe
        _case("view-vga", "render", 100_000, 1, 640, 480, 3),
        # evaluation of a large map on two full-HD views, median depth
        _case("view-hd", "render", 1_000_000, 2, 1920, 1080, 3, median=True),
        # pose and map refinement of one VGA keyframe through autograd
        _case("fit-vga", "fit", 100_000, 1, 640, 480, 3),
        # the mapper's inner loop on VGA keyframes, captured as a graph
        _case("map-graph", "step", 150_000, 4, 640, 480, 3, loss="render", graph=True),
        # the mapper's batch: 500k Gaussians, eight 1200x680 keyframes
        _case("map-batch", "step", 500_000, 8, 1200, 680, 3, loss="l1"),
        # mixed resolutions, heavy-tailed Gaussian sizes, the large tile
        _case("map-mixed", "step", 200_000, 6, 1296, 968, 3, tile="32x16", mixed=True,
              heavy=True, loss="render"),
        # a small ragged surfel map, one keyframe
        _case("surfel-small", "surfel", 20_000, 1, 321, 243, 2, size=-3.6),
        # the surfel mapper's batch
        _case("surfel-batch", "surfel", 250_000, 4, 1200, 680, 3),
        # the rendering loss of a keyframe batch
        _case("loss", "loss", 1000, 4, 1296, 968, 0, loss="render"),
        # statistics, optimiser and position noise of one mapping iteration
        _case("update", "update", 500_000, 4, 640, 480, 3),
    ]


def draw(rng):
    """One more case: sizes log-uniform over the listed ranges, every option."""
    def logi(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["render", "render", "fit", "fit", "step", "step", "step", "surfel",
                     "surfel", "loss", "update"])
    frames = rng.choice([1, 1, 2, 3, 4, 5, 6, 8])
    width = logi(96, 1400)
    height = max(64, int(width * rng.uniform(0.5, 0.8)))
    # no draw costs more than the largest listed case
    frames = min(frames, max(1, int((3.0e6 if op == "surfel" else 5.0e6) / (width * height))))
    top = {"render": 700_000, "fit": 300_000, "step": 300_000, "surfel": 120_000, "loss": 1000,
           "update": 500_000}[op]
    n = 1000 if op == "loss" else logi(1500, top)
    # the density of a real map: at most ~0.6 Gaussians per pixel of a frame,
    # and Gaussians that shrink as it gets denser (pruning and splitting)
    if op != "loss":
        n = max(1500, min(n, int(0.6 * width * height)))
    size = -2.6 - 0.25 * math.log(max(1.0, n / height)) + rng.uniform(-0.3, 0.3)
    return dict(op=op, n=n, frames=frames, width=width, height=height,
                sh=rng.choice([0, 1, 2, 3, 3]), size=round(max(-4.5, min(-3.0, size)), 2),
                tile=rng.choice(["16x16", "16x16", "16x16", "32x16", "32x8", "16x8"]),
                mixed=frames > 1 and rng.random() < 0.4,
                heavy=rng.random() < 0.3 and op != "surfel",
                median=op in ("render", "fit", "step") and rng.random() < 0.25,
                loss={"step": rng.choice(["l1", "render"]), "loss": "render"}.get(op, ""),
                graph=op == "step" and rng.random() < 0.4)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _sizes(case):
    out = []
    for i in range(case["frames"]):
        s = (1.0, 0.5, 0.75, 0.25)[i % 4] if case["mixed"] else 1.0
        cut = i % 3 if case["mixed"] else 0  # ragged widths in a mixed batch
        out.append((max(16, int(case["width"] * s) - cut), max(16, int(case["height"] * s))))
    return out


def _turn(axis, ang):
    axis = axis / np.linalg.norm(axis)
    K = np.array([[0, -axis[2], axis[1]], [axis[2], 0, -axis[0]], [-axis[1], axis[0], 0]])
    return np.eye(3) + math.sin(ang) * K + (1 - math.cos(ang)) * (K @ K)


def _scene(case, seed):
    """Gaussians (or surfels), cameras and poses of the case, on the GPU."""
    n, F = case["n"], case["frames"]
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float64)

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device=DEV, dtype=torch.float64)

    sizes = _sizes(case)
    cams = [(w, h, 0.5 * (w + h) * 0.65, 0.5 * (w + h) * 0.65, w / 2.0, h / 2.0, NEAR)
            for w, h in sizes]
    # camera-to-world poses: 0.1 m and 5 degrees between keyframes
    R, C = np.eye(3), np.zeros(3)
    head, axis = rng.normal(size=3), rng.normal(size=3)
    head /= np.linalg.norm(head)
    poses, means = [], []
    for f, (w, h, fx, fy, cx, cy, _) in enumerate(cams):
        poses.append(np.concatenate([R.T, (-R.T @ C)[:, None]], 1))
        # this keyframe's share of the map: pixels of a piecewise-planar depth
        m = n // F + (1 if f < n % F else 0)
        u, v = uniform(m) * w, uniform(m) * h
        sx, sy, z0 = uniform(32) * w, uniform(32) * h, 0.5 + 3.5 * uniform(32)
        ang, mag = 2 * math.pi * uniform(32), 2e-3 * uniform(32)
        k = torch.cat([((a[:, None] - sx) ** 2 + (b[:, None] - sy) ** 2).argmin(1)
                       for a, b in zip(u.split(1 << 18), v.split(1 << 18))])
        z = (z0[k] + mag[k] * (torch.cos(ang)[k] * (u - sx[k]) +
                               torch.sin(ang)[k] * (v - sy[k]))).clamp(0.5, 4.0)
        pc = torch.stack([(u - cx) * z / fx, (v - cy) * z / fy, z], 1)
        means.append(pc @ torch.tensor(R.T, device=DEV) + torch.tensor(C, device=DEV))
        head = head + 0.15 * rng.normal(size=3)
        head /= np.linalg.norm(head)
        axis = axis + 0.2 * rng.normal(size=3)
        C = C + 0.1 * head
        R = R @ _turn(axis, math.radians(5.0))
    dims = 2 if case["op"] == "surfel" else 3
    if case["heavy"]:  # Student-t log-scales: a few Gaussians cover many tiles
        chi = (normal(n, dims) ** 2 + normal(n, dims) ** 2 + normal(n, dims) ** 2) / 3
        ls = (case["size"] + 0.5 * normal(n, dims) / chi.sqrt()).clamp(-9.0, -0.5)
    else:
        ls = case["size"] + 0.6 * normal(n, dims)
        mid = ls.mean(1, keepdim=True)
        spread = (ls.amax(1, keepdim=True) - ls.amin(1, keepdim=True)).clamp(min=1e-9)
        ls = mid + (ls - mid) * (math.log(20.0) / spread).clamp(max=1.0)  # at most 20 : 1
    K = (case["sh"] + 1) ** 2
    sh = 0.1 * normal(n, K, 3)
    sh[:, 0] = 0.5 + 0.2 * normal(n, 3)
    quats = normal(n, 4)
    if case["op"] == "surfel":  # disks roughly face the first camera
        quats = torch.cat([1.0 + 0 * quats[:, :1], 0.25 * quats[:, 1:]], 1)
    f32 = {k: v.float().contiguous() for k, v in dict(
        means=torch.cat(means) + 0.01 * normal(n, 3), log_scales=ls, quats=quats,
        opacity=1.5 * normal(n), sh=sh,
        poses=torch.tensor(np.stack(poses), device=DEV)).items()}
    return f32, cams, gen


def _targets(cams, gen):
    """Keyframe images: smooth colour with texture, depth with holes."""
    rgb, dep = [], []
    for w, h in ((c[0], c[1]) for c in cams):
        y = torch.arange(h, device=DEV, dtype=torch.float32)[:, None]
        x = torch.arange(w, device=DEV, dtype=torch.float32)[None]
        r = torch.rand(4, 4, generator=gen, device=DEV)
        for c in range(4):
            wave = torch.sin((r[c, 0] * x + r[c, 1] * y) * 0.1 + 6.3 * r[c, 2])
            noise = torch.randn(h, w, generator=gen, device=DEV)
            if c < 3:
                rgb.append((0.3 + 0.4 * r[c, 3] + 0.2 * wave + 0.03 * noise).clamp(0, 1).ravel())
            else:
                z = 2.0 + wave + 0.02 * noise
                hole = torch.rand(h, w, generator=gen, device=DEV) < 0.1
                dep.append(torch.where(hole, torch.zeros_like(z), z).ravel())
    return torch.cat(rgb).contiguous(), torch.cat(dep).contiguous()


def _pixels(cams):
    return sum(c[0] * c[1] for c in cams)


def _tile(case):
    return tuple(int(t) for t in case["tile"].split("x"))


def _grad_bufs(case, dims=3):
    n, K, F = case["n"], (case["sh"] + 1) ** 2, case["frames"]
    shapes = dict(means=(n, 3), log_scales=(n, dims), quats=(n, 4), opacity=(n,), sh=(n, K, 3),
                  twist=(F, 6))
    return {k: torch.empty(*s, device=DEV) for k, s in shapes.items()}


def _inputs(case, seed):
    """Everything the case's numbers depend on, made from the seed alone."""
    p, cams, gen = _scene(case, seed)
    P, op = _pixels(cams), case["op"]
    s = dict(p=p, cams=cams)
    if op == "fit":  # upstream gradients as a loss of mean type leaves them
        s["up"] = [torch.randn(k * P, generator=gen, device=DEV) for k in (3, 1, 1)]
    elif op in ("step", "surfel", "loss"):
        s["target"] = _targets(cams, gen)
    if op == "loss":  # images near their targets
        t_rgb, t_dep = s["target"]
        s["image"] = (
            (t_rgb + 0.05 * torch.randn(3 * P, generator=gen, device=DEV)).clamp(0, 1),
            t_dep + 0.05 * torch.randn(P, generator=gen, device=DEV))
    if op == "update":
        s["up"] = [torch.randn(k * P, generator=gen, device=DEV) for k in (3, 1, 1)]
        s["grads"] = {
            "means": 1e-3 * torch.randn(p["means"].shape, generator=gen, device=DEV),
            "sh": 1e-4 * torch.randn(p["sh"].shape, generator=gen, device=DEV),
            "twist": 1e-2 * torch.randn(case["frames"], 6, generator=gen, device=DEV)}
        s["eps"] = torch.randn(p["means"].shape, generator=gen, device=DEV)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    p, cams, op, P = s["p"], s["cams"], case["op"], _pixels(s["cams"])
    s["case"], s["rast"] = case, Rasterizer(0)
    rast, args = s["rast"], [p[k] for k in PARAMS] + [p["poses"], cams, case["sh"]]
    s["args"] = args
    if op == "fit":
        for k in PARAMS:
            p[k].requires_grad_(True)
        s["twist"] = torch.zeros(case["frames"], 6, device=DEV, requires_grad=True)
    elif op == "step":
        rast.forward(*args, tile=_tile(case))
        cap = int(rast.stats()["n_keys"] * 1.1) + 4096
        b = _grad_bufs(case)
        b.update(rgb=torch.empty(3 * P, device=DEV), depth=torch.empty(P, device=DEV),
                 alpha=torch.empty(P, device=DEV), loss=torch.empty(1, device=DEV))
        if case["loss"] == "render":
            b["ssim"] = torch.empty(case["frames"], device=DEV)
        s["bufs"], s["cap"] = b, cap
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _step(s)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                _step(s)
    elif op == "loss":  # the loss reads the frame layout of the last forward
        rast.forward(*args)
    elif op == "update":
        rast.forward(*args, tile=_tile(case))
        rast.backward(*s["up"])
        dims = {"means": p["means"].shape, "sh": p["sh"].shape, "twist": (case["frames"], 6)}
        s["moments"] = {f"{m}_{k}": torch.zeros(*d, device=DEV)
                        for m in "mv" for k, d in dims.items()}
        s["moments"]["step"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["accum"] = torch.zeros(case["n"], device=DEV)
        s["count"] = torch.zeros(case["n"], device=DEV)
    return s


# --------------------------------------------------------------------------
# the calls
# --------------------------------------------------------------------------
def _step(s):
    case, b = s["case"], s["bufs"]
    kw = dict(tile=_tile(case), key_capacity=s["cap"], median=case["median"])
    if case["loss"] == "l1":
        s["rast"].step_l1(*s["args"], *s["target"], 1.0, b, **kw)
    else:
        s["rast"].step_render(*s["args"], *s["target"], b, lambda1=LAMBDA1, lambda2=LAMBDA2,
                              **kw)


def _run_surfel(s):
    case, r, p, cams = s["case"], s["rast"], s["p"], s["cams"]
    rgb, depth, alpha, normal, dist = r.forward_surfel(*s["args"], tile=_tile(case))
    g = r.loss_render(rgb, depth, *s["target"], LAMBDA1, LAMBDA2)
    g_normal = torch.zeros_like(normal)
    l_n = r.normal_consistency(cams, depth, alpha, normal, W_NORMAL, g["g_depth"], g["g_alpha"],
                               g_normal)
    g_dist = torch.cat([torch.full((c[0] * c[1],), W_DIST / (c[0] * c[1]), device=DEV)
                        for c in cams])
    grads = r.backward_surfel(g["g_rgb"], g["g_depth"], g["g_alpha"], g_normal, g_dist)
    return dict(rgb=rgb, depth=depth, alpha=alpha, normal=normal, dist=dist, loss=g["loss"],
                loss_normal=l_n, **{"d_" + k: v for k, v in grads.items()})


def run(state):
    s, op = state, state["case"]["op"]
    case, p = s["case"], s["p"]
    kw = dict(tile=_tile(case), rasterizer=s["rast"], median=case["median"])
    if op == "render":
        with torch.no_grad():
            rgb, depth, alpha = rasterize(*s["args"], **kw)
        return dict(rgb=rgb, depth=depth, alpha=alpha)
    if op == "fit":
        rgb, depth, alpha = rasterize(*s["args"], twist=s["twist"], **kw)
        wrt = [p[k] for k in PARAMS] + [s["twist"]]
        g = torch.autograd.grad([rgb, depth, alpha], wrt, s["up"])
        return dict(rgb=rgb, depth=depth, alpha=alpha,
                    **{"d_" + k: v for k, v in zip(PARAMS + ("twist",), g)})
    if op == "step":
        if case["graph"]:
            s["graph"].replay()
        else:
            _step(s)
        b = s["bufs"]
        out = {k: b[k] for k in ("rgb", "depth", "alpha", "loss")}
        out.update({"d_" + k: b[k] for k in PARAMS + ("twist",)})
        if "ssim" in b:
            out["ssim"] = b["ssim"]
        return out
    if op == "surfel":
        return _run_surfel(s)
    if op == "loss":
        return s["rast"].loss_render(*s["image"], *s["target"], LAMBDA1, LAMBDA2)
    r, m, g = s["rast"], s["moments"], s["grads"]
    r.densify_stats(s["accum"], s["count"])
    r.adam_step(dict(means=p["means"], sh=p["sh"], poses=p["poses"]), g, m, **LRS)
    r.mcmc_noise(p["means"], p["log_scales"], p["quats"], p["opacity"], s["eps"], 1.6)
    return dict(accum=s["accum"], count=s["count"], means=p["means"], sh=p["sh"],
                poses=p["poses"], **m)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Inputs read and outputs written once; the arithmetic of the pairs that
    are blended (a pixel is saturated after about 40 of them), of the
    projection and of the window sums."""
    n, F, K = case["n"], case["frames"], (case["sh"] + 1) ** 2
    P = sum(w * h for w, h in _sizes(case))
    surf = case["op"] == "surfel"
    dims = 2 if surf else 3
    params = 4 * n * (3 + dims + 4 + 1 + 3 * K)
    images = 4 * P * (9 if surf else 5)
    # blended entries per pixel from the Gaussians' mean footprint
    f = 0.65 * 0.5 * (case["width"] + case["height"])
    foot = 8.0 * (math.exp(case["size"]) * f / 2.2) ** 2 + 3.0
    deep = min(40.0, n * foot / (case["width"] * case["height"]))
    pairs = P * deep
    ssim = 3 * P * 8 * 22 * 2
    op = case["op"]
    if op == "render":
        return {"bytes": params + images, "flops": 27 * pairs + 400 * n * F}
    if op == "fit":
        return {"bytes": 2 * params + 2 * images, "flops": 90 * pairs + 1500 * n * F}
    if op == "step":
        return {"bytes": 2 * params + images + 16 * P,
                "flops": 90 * pairs + 1500 * n * F + (ssim if case["loss"] == "render" else 0)}
    if op == "surfel":
        return {"bytes": 2 * params + images + 16 * P,
                "flops": 245 * pairs + 1500 * n * F + ssim}
    if op == "loss":
        return {"bytes": 52 * P, "flops": ssim}
    ngrad = n * (3 + 3 * K)
    return {"bytes": 4 * (7 * ngrad + n * (3 + 3 + 4 + 1 + 4) + 2 * n * F),
            "flops": 12 * ngrad + 80 * n}


# --------------------------------------------------------------------------
# the same numbers in 64 bits, in plain torch
# --------------------------------------------------------------------------
A_MIN, A_MAX, T_MIN = (float(np.float32(v)) for v in (1.0 / 255.0, 0.99, 1e-4))
BLOCK = 32  # pixels are taken in BLOCK x BLOCK windows
EXACT_PIXELS, EXACT_N = 7_000_000, 1_000_000  # larger cases take too long


def _sh_colour(d, sh):
    """max(0, sum_k sh_k Y_k(d) + 1/2) with the real spherical harmonics up to
    degree 3, phase (-1)^|m|, from their closed forms."""
    x, y, z = d.unbind(-1)
    c = math.sqrt
    pi = math.pi
    Y = [torch.full_like(x, c(1 / (4 * pi)))]
    if sh.shape[1] > 1:
        k = c(3 / (4 * pi))
        Y += [-k * y, k * z, -k * x]
    if sh.shape[1] > 4:
        k = c(15 / (4 * pi))
        Y += [k * x * y, -k * y * z, c(5 / (16 * pi)) * (3 * z * z - 1), -k * x * z,
              k / 2 * (x * x - y * y)]
    if sh.shape[1] > 9:
        k3, k2, k1 = c(35 / (32 * pi)), c(105 / (4 * pi)), c(21 / (32 * pi))
        Y += [-k3 * y * (3 * x * x - y * y), k2 * x * y * z, -k1 * y * (5 * z * z - 1),
              c(7 / (16 * pi)) * z * (5 * z * z - 3), -k1 * x * (5 * z * z - 1),
              k2 / 2 * z * (x * x - y * y), -k3 * x * (x * x - 3 * y * y)]
    return ((torch.stack(Y, -1)[..., None] * sh).sum(1) + 0.5).clamp(min=0)


def _skew(v):
    o = torch.zeros_like(v[0])
    return torch.stack([torch.stack([o, -v[2], v[1]]), torch.stack([v[2], o, -v[0]]),
                        torch.stack([-v[1], v[0], o])])


def _rotation(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([
        1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)


def _camera(x, twist, pose):
    """Camera of one frame moved by the left twist (first order, at zero)."""
    turn = torch.eye(3, device=DEV, dtype=torch.float64) + _skew(twist[3:])
    W, t = turn @ pose[:, :3], turn @ pose[:, 3] + twist[:3]
    d = x["means"] + W.T @ t
    colour = _sh_colour(d / d.norm(dim=1, keepdim=True), x["sh"])
    return W, t, colour, torch.sigmoid(x["opacity"])


def _project(x, twist, pose, cam):
    """Per-Gaussian screen quantities of one frame (rows), and who is kept
    with which pixel box."""
    w, h, fx, fy, cx, cy, near = cam
    W, t, colour, op = _camera(x, twist, pose)
    M = _rotation(x["quats"]) * x["log_scales"].exp()[:, None, :]
    tc = x["means"] @ W.T + t
    z = torch.where(tc[:, 2] > near, tc[:, 2], torch.ones_like(tc[:, 2]))
    u, v = fx * tc[:, 0] / z + cx, fy * tc[:, 1] / z + cy
    lx, ly = 1.3 * w / (2 * fx), 1.3 * h / (2 * fy)
    rx, ry = (tc[:, 0] / z).clamp(-lx, lx), (tc[:, 1] / z).clamp(-ly, ly)
    o = torch.zeros_like(z)
    J = torch.stack([fx / z, o, -fx * rx / z, o, fy / z, -fy * ry / z], 1).view(-1, 2, 3)
    B = torch.bmm(J, W @ M)
    cov = (B[:, :, None, :] * B[:, None, :, :]).sum(3)
    a, b, c = cov[:, 0, 0] + 0.3, cov[:, 0, 1], cov[:, 1, 1] + 0.3
    with torch.no_grad():
        r = 3 * (0.5 * (a + c) + (0.25 * (a - c) ** 2 + b * b).sqrt()).sqrt()
        box = torch.stack([(u - r).ceil(), (u + r).floor(), (v - r).ceil(), (v + r).floor()], 1)
        qa = 2 * (op / A_MIN).log().clamp(min=0)
        hx, hy = (qa * a).sqrt(), (qa * c).sqrt()
        # the part of the square where alpha can reach 1/255 (only a search aid)
        near_box = torch.stack([torch.maximum(box[:, 0], u - hx - 1),
                                torch.minimum(box[:, 1], u + hx + 1),
                                torch.maximum(box[:, 2], v - hy - 1),
                                torch.minimum(box[:, 3], v + hy + 1)], 1)
        keep = (tc[:, 2] > near) & (op > A_MIN)
    return dict(u=u, v=v, a=a, b=b, c=c, op=op, z=z, colour=colour), keep, box, near_box


def _project_surfel(x, twist, pose, cam):
    w, h, fx, fy, cx, cy, near = cam
    W, t, colour, op = _camera(x, twist, pose)
    T = W @ _rotation(x["quats"])
    mc = x["means"] @ W.T + t
    s = x["log_scales"].exp()
    cols = torch.stack([s[:, :1] * T[:, :, 0], s[:, 1:] * T[:, :, 1], mc], 2)
    K = torch.tensor([[fx, 0, cx], [0, fy, cy], [0, 0, 1]], device=DEV, dtype=torch.float64)
    M = K @ cols
    z = mc[:, 2]
    nrm = T[:, :, 2]
    nrm = torch.where((nrm * mc).sum(1, keepdim=True) < 0, nrm, -nrm)
    zc = torch.where(z > near, z, torch.ones_like(z))
    u, v = M[:, 0, 2] / zc, M[:, 1, 2] / zc
    with torch.no_grad():
        r2 = 2 * (op / A_MIN).log().clamp(min=1e-12)
        keep = (op > A_MIN) & (z > near) & \
            (z - r2.sqrt() * M[:, 2, :2].norm(dim=1) > near)
        D = torch.stack([r2, r2, -torch.ones_like(r2)], 1)[:, None, :]
        Cq = torch.bmm(M * D, M.transpose(1, 2).contiguous())
        rl = (0.5 * r2).sqrt()
        ends = []
        for i, c0 in ((0, u), (1, v)):
            disc = (Cq[:, i, 2] ** 2 - Cq[:, i, i] * Cq[:, 2, 2]).clamp(min=0).sqrt()
            e = [(Cq[:, i, 2] + g * disc) / Cq[:, 2, 2] for g in (1, -1)]
            ends += [torch.minimum(torch.minimum(*e), c0 - rl).ceil(),
                     torch.maximum(torch.maximum(*e), c0 + rl).floor()]
        box = torch.stack(ends, 1)
    return dict(u=u, v=v, M=M.reshape(-1, 9), op=op, z=zc, colour=colour, normal=nrm), keep, \
        box, box


def _block(e, box, px, py, median, surfel):
    """Front-to-back blend of entries e (rows, in depth order) at pixels px, py."""
    inside = (px[:, None] >= box[:, 0]) & (px[:, None] <= box[:, 1]) & \
        (py[:, None] >= box[:, 2]) & (py[:, None] <= box[:, 3])
    dx, dy = px[:, None] - e["u"], py[:, None] - e["v"]
    if surfel:
        M = e["M"].view(-1, 3, 3)
        hu = px[:, None, None] * M[:, 2] - M[:, 0]
        hv = py[:, None, None] * M[:, 2] - M[:, 1]
        p = torch.linalg.cross(hu, hv)
        ok = p[..., 2] != 0
        p2 = torch.where(ok, p[..., 2], torch.ones_like(p[..., 2]))
        s, t = p[..., 0] / p2, p[..., 1] / p2
        G = torch.where(ok, torch.exp(-0.5 * (s * s + t * t)), torch.zeros_like(s))
        low = torch.exp(-(dx * dx + dy * dy))
        disk = G >= low
        z = torch.where(disk, M[:, 2, 0] * s + M[:, 2, 1] * t + M[:, 2, 2], e["z"])
        G = torch.where(disk, G, low)
    else:
        det = e["a"] * e["c"] - e["b"] ** 2
        G = torch.exp(-0.5 * (e["c"] * dx * dx - 2 * e["b"] * dx * dy + e["a"] * dy * dy) / det)
        z = e["z"].expand_as(G)
    alpha = (e["op"] * G).clamp(max=A_MAX)
    alpha = torch.where(inside & (alpha >= A_MIN), alpha, torch.zeros_like(alpha))
    with torch.no_grad():  # stop before an entry that would drop T below T_MIN
        alive = torch.cumprod(1 - alpha, 1) >= T_MIN
    alpha = torch.where(alive, alpha, torch.zeros_like(alpha))
    after = torch.cumprod(1 - alpha, 1)
    before = torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1)
    wgt = alpha * before
    out = [wgt @ e["colour"]]
    if median:
        with torch.no_grad():
            cross = (after < 0.5) & (before >= 0.5)
        out.append((z * cross).sum(1, keepdim=True))
    else:
        out.append((wgt * z).sum(1, keepdim=True))
    out.append(1 - after[:, -1:])
    if surfel:
        out.append(wgt @ e["normal"])
        s0, s1, s2 = (torch.cumsum(wgt * zz, 1) for zz in (torch.ones_like(z), z, z * z))
        out.append((wgt * (s0 * z * z - 2 * z * s1 + s2)).sum(1, keepdim=True))
    return torch.cat(out, 1)


def _windows(cam, keep, order, near_box):
    """(entries in depth order, px, py, pixel ids) of every pixel window."""
    w, h = cam[0], cam[1]
    for y0 in range(0, h, BLOCK):
        y1 = min(h, y0 + BLOCK)
        row = keep & (near_box[:, 2] <= y1 - 1) & (near_box[:, 3] >= y0)
        row = order[row[order]]
        nb = near_box[row]
        for x0 in range(0, w, BLOCK):
            x1 = min(w, x0 + BLOCK)
            idx = row[(nb[:, 0] <= x1 - 1) & (nb[:, 1] >= x0)]
            if idx.numel() == 0:
                continue
            ys, xs = torch.meshgrid(torch.arange(y0, y1, device=DEV),
                                    torch.arange(x0, x1, device=DEV), indexing="ij")
            ys, xs = ys.ravel(), xs.ravel()
            yield idx, xs.double(), ys.double(), ys * w + xs


def _render_exact(case, s, loss):
    """Images [per frame: pixels x channels] and the gradients of the scene for
    the upstream that loss(images) gives (None: images alone)."""
    surfel = case["op"] == "surfel"
    project = _project_surfel if surfel else _project
    x = {k: s["p"][k].detach().double().requires_grad_(loss is not None) for k in PARAMS}
    poses = s["p"]["poses"].double()
    twist = torch.zeros(case["frames"], 6, device=DEV, dtype=torch.float64, requires_grad=True)
    frames, images = [], []
    ch = 9 if surfel else 5
    for f, cam in enumerate(s["cams"]):
        with torch.set_grad_enabled(loss is not None):
            e, keep, box, near_box = project(x, twist[f], poses[f], cam)
        order = torch.argsort(e["z"].detach().float(), stable=True)
        img = torch.zeros(cam[0] * cam[1], ch, device=DEV, dtype=torch.float64)
        with torch.no_grad():
            for idx, px, py, at in _windows(cam, keep, order, near_box):
                img[at] = _block({k: v[idx] for k, v in e.items()}, box[idx], px, py,
                                 case["median"], surfel)
        images.append(img)
        frames.append((e, keep, box, near_box, order))
    if loss is None:
        return images, None, None
    ups, values = loss(images)
    for f, cam in enumerate(s["cams"]):
        e, keep, box, near_box, order = frames[f]
        names = list(e)
        total = {k: torch.zeros_like(e[k]) for k in names}
        for idx, px, py, at in _windows(cam, keep, order, near_box):
            leaf = {k: e[k].detach()[idx].requires_grad_(True) for k in names}
            out = _block(leaf, box[idx], px, py, case["median"], surfel)
            g = torch.autograd.grad(out, [leaf[k] for k in names], ups[f][at],
                                    allow_unused=True)
            for k, v in zip(names, g):
                if v is not None:
                    total[k].index_add_(0, idx, v)
        torch.autograd.backward([e[k] for k in names], [total[k] for k in names],
                                retain_graph=f + 1 < len(frames))
    return images, {**{k: x[k].grad for k in PARAMS}, "twist": twist.grad}, values


def _split(cams, rgb, *flat):
    """Packed images as one [pixels x channels] tensor per frame."""
    out, o = [], 0
    for c in cams:
        k = c[0] * c[1]
        out.append(torch.cat([rgb[3 * o:3 * (o + k)].view(3, k).T] +
                             [v[o:o + k, None] for v in flat], 1).double())
        o += k
    return out


def _packed(images, col, width):
    return torch.cat([i[:, col:col + width].T.reshape(-1) for i in images])


def _blur(x):
    k = torch.exp(-(torch.arange(11, device=DEV, dtype=torch.float64) - 5) ** 2 / 4.5)
    k = k / k.sum()
    x = torch.nn.functional.pad(x, (5, 5, 5, 5))
    x = sum(k[i] * x[..., i:x.shape[-1] - 10 + i] for i in range(11))
    return sum(k[i] * x[..., i:x.shape[-2] - 10 + i, :] for i in range(11))


def _ssim(x, y):
    mx, my = _blur(x), _blur(y)
    vx, vy, cxy = _blur(x * x) - mx * mx, _blur(y * y) - my * my, _blur(x * y) - mx * my
    return (((2 * mx * my + 1e-4) * (2 * cxy + 9e-4)) /
            ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))).mean()


def _loss_frame(kind, cam, img, tgt):
    """One frame's loss of [pixels x (rgb, depth, ...)] images, and its SSIM."""
    valid = tgt[:, 3] > 0
    l1 = (img[:, :3] - tgt[:, :3]).abs().mean()
    ld = (img[valid, 3] - tgt[valid, 3]).abs().mean() if bool(valid.any()) else img.sum() * 0
    if kind == "l1":
        return l1 + ld, None
    ss = _ssim(*(v[:, :3].T.reshape(1, 3, cam[1], cam[0]) for v in (img, tgt)))
    l1w, l2w = (float(np.float32(v)) for v in (LAMBDA1, LAMBDA2))
    return l1w * ((1 - l2w) * l1 + l2w * (1 - ss)) + (1 - l1w) * ld, ss


def _normal_loss(cam, img):
    """Normal consistency of [pixels x (rgb, depth, alpha, normal, dist)]."""
    w, h, fx, fy, cx, cy, _ = cam
    if w < 3 or h < 3:
        return img.sum() * 0
    D = img[:, 3].view(h, w)
    yy, xx = torch.meshgrid(torch.arange(h, device=DEV, dtype=torch.float64),
                            torch.arange(w, device=DEV, dtype=torch.float64), indexing="ij")
    Pt = torch.stack([D * (xx - cx) / fx, D * (yy - cy) / fy, D])
    dX = 0.5 * (Pt[:, 1:-1, 2:] - Pt[:, 1:-1, :-2])
    dY = 0.5 * (Pt[:, 2:, 1:-1] - Pt[:, :-2, 1:-1])
    v = torch.linalg.cross(dY, dX, dim=0)
    sq = (v * v).sum(0)
    N = torch.where(sq > 0, v / torch.where(sq > 0, sq, torch.ones_like(sq)).sqrt(),
                    torch.zeros_like(v))
    nm, al = img[:, 5:8].T.view(3, h, w)[:, 1:-1, 1:-1], img[:, 4].view(h, w)[1:-1, 1:-1]
    term = al - (nm * N).sum(0)
    return torch.where(sq > 0, term, torch.zeros_like(term)).sum() / ((w - 2) * (h - 2))


def _objective(case, s, images):
    """Upstream gradients per frame and the loss values."""
    cams = s["cams"]
    if case["op"] == "fit":
        return _split(cams, s["up"][0], s["up"][1], s["up"][2]), {}
    tgt = _split(cams, s["target"][0], s["target"][1])
    ups, total, normal, ssims = [], 0.0, 0.0, []
    for cam, img, t in zip(cams, images, tgt):
        img = img.detach().requires_grad_(True)
        kind = case["loss"] or "render"
        loss, ss = _loss_frame(kind, cam, img, t)
        full = loss
        if case["op"] == "surfel":
            ln = float(np.float32(W_NORMAL)) * _normal_loss(cam, img)
            normal = normal + ln.detach()
            full = loss + ln + W_DIST * img[:, 8].mean()
        ups.append(torch.autograd.grad(full, img)[0])
        total = total + loss.detach()
        ssims.append(ss.detach() if ss is not None else None)
    values = dict(loss=total.reshape(1))
    if case["op"] == "surfel":
        values["loss_normal"] = normal.reshape(1)
    if ssims[0] is not None:
        values["ssim"] = torch.stack(ssims)
    return ups, values


def _exact_update(case, s):
    """One Adam step from zero moments with the pose fold, then the noise."""
    p = {k: v.double() for k, v in s["p"].items()}
    b1, b2, eps = (float(np.float32(v)) for v in (0.9, 0.999, 1e-15))
    out = dict(accum=None, count=None, step=None)
    delta = {}
    for k, lr in (("means", "lr_means"), ("sh", "lr_sh"), ("twist", "lr_pose")):
        g = s["grads"][k].double()
        m, v = (1 - b1) * g, (1 - b2) * g * g
        out["m_" + k], out["v_" + k] = m, v
        delta[k] = -float(np.float32(LRS[lr])) * (m / (1 - b1)) / ((v / (1 - b2)).sqrt() + eps)
    mu, out["sh"] = p["means"] + delta["means"], p["sh"] + delta["sh"]
    poses = []
    for xi, pose in zip(delta["twist"], p["poses"]):
        A = torch.zeros(4, 4, device=DEV, dtype=torch.float64)
        A[:3, :3], A[:3, 3] = _skew(xi[3:]), xi[:3]
        poses.append((torch.linalg.matrix_exp(A) @
                      torch.cat([pose, torch.eye(4, device=DEV, dtype=torch.float64)[3:]]))[:3])
    out["poses"] = torch.stack(poses)
    M = _rotation(p["quats"]) * p["log_scales"].exp()[:, None, :]
    gate = 1 / (1 + torch.exp(100 * (torch.sigmoid(p["opacity"]) - 0.995)))
    e = (M * (M * s["eps"].double()[:, :, None]).sum(1)[:, None, :]).sum(2)
    out["means"] = mu + float(np.float32(1.6)) * gate[:, None] * e
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    op, cams = case["op"], s["cams"]
    if op == "update":
        return _exact_update(case, s)
    if op == "loss":
        images = _split(cams, *s["image"])
        ups, values = _objective(case, s, images)
        return dict(values, g_rgb=_packed(ups, 0, 3), g_depth=_packed(ups, 3, 1),
                    g_alpha=torch.zeros(_pixels(cams), device=DEV, dtype=torch.float64))
    if _pixels(cams) > EXACT_PIXELS or case["n"] > EXACT_N:
        return None
    loss = None if op == "render" else lambda images: _objective(case, s, images)
    images, grads, values = _render_exact(case, s, loss)
    out = dict(rgb=_packed(images, 0, 3), depth=_packed(images, 3, 1),
               alpha=_packed(images, 4, 1))
    if op == "surfel":
        out.update(normal=_packed(images, 5, 3), dist=_packed(images, 8, 1))
    if grads is not None:
        out.update({"d_" + k: v for k, v in grads.items()})
        out.update({k: v for k, v in values.items() if op == "step" or k != "ssim"})
    return out
