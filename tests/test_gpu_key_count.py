"""The key count that a growing forward waits for belongs to that forward: one
that returns an error (here an earlier call's HIP error, which the forward
reports) does so after its own count has arrived, so that the forward after it,
with more keys, does not take the count for its own."""
import ctypes as C

import numpy as np
import pytest

from paper_2411_17660_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("surfel", [False, True])
def test_count_of_a_failed_forward_is_not_taken_for_the_next(surfel):
    import torch
    from gpu_util import to_dev
    from paper_2411_17660_amd.native import GsrError
    from paper_2411_17660_amd.raster import Rasterizer
    rast, fresh = Rasterizer(0), Rasterizer(0)
    hip_set_device = rast.lib.hipSetDevice
    hip_set_device.argtypes = [C.c_int]
    small, large = (scenes.tiny_scene(seed=4, n=n, W=96, H=72, f=70.0, sh_degree=0, ls_mean=-2.5)
                    for n in (50, 30000))
    dev = {id(s): to_dev(s) for s in (small, large)}
    if surfel:
        for d in dev.values():
            d["log_scales"] = d["log_scales"][:, :2].contiguous()

    def fwd(r, s):
        d = dev[id(s)]
        f = r.forward_surfel if surfel else r.forward
        return f(d["means"], d["log_scales"], d["quats"], d["opacity"], d["sh"], d["poses"],
                 s.cams, s.sh_degree, s.background)
    want = [x.clone() for x in fwd(fresh, large)]
    lists = fresh.debug_lists()
    fwd(rast, small)  # workspaces of the small scene: nothing grows below
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(20):  # the count of the failing forward is some ms away
        a = a @ a
        a /= a.norm()
    assert hip_set_device(1 << 20) != 0
    with pytest.raises(GsrError) as ei:
        fwd(rast, small)
    assert ei.value.status == 4, ei.value
    got = fwd(rast, large)
    for x, y in zip(got, want):
        assert torch.equal(x, y)
    L = rast.debug_lists()
    assert L["K"] == lists["K"]
    for k in ("tile_keys", "tile_vals", "ranges", "n_last"):
        assert np.array_equal(L[k], lists[k]), k


def test_growing_forward_in_a_capture_is_an_error():
    """Its count cannot arrive while the stream is being captured: the call
    fails instead of waiting, and the context works afterwards."""
    import torch
    from gpu_util import to_dev
    from paper_2411_17660_amd.native import GsrError
    from paper_2411_17660_amd.raster import Rasterizer
    rast = Rasterizer(0)
    sc = scenes.tiny_scene(seed=4, n=500, W=96, H=72, f=70.0, sh_degree=0, ls_mean=-2.5)
    d = to_dev(sc)
    P = sc.n_pixels
    out = tuple(torch.empty(k * P, device="cuda") for k in (3, 1, 1))

    def fwd():
        rast.forward(*[d[k] for k in ("means", "log_scales", "quats", "opacity", "sh", "poses")],
                     sc.cams, 0, sc.background, out=out)
    fwd()
    torch.cuda.synchronize()
    want = [x.clone() for x in out]
    hip = {k: getattr(rast.lib, k) for k in ("hipStreamCreate", "hipStreamBeginCapture",
                                             "hipStreamEndCapture", "hipStreamDestroy")}
    hip["hipStreamCreate"].argtypes = [C.POINTER(C.c_void_p)]
    hip["hipStreamBeginCapture"].argtypes = [C.c_void_p, C.c_int]
    hip["hipStreamEndCapture"].argtypes = [C.c_void_p, C.POINTER(C.c_void_p)]
    hip["hipStreamDestroy"].argtypes = [C.c_void_p]
    own, graph = C.c_void_p(), C.c_void_p()  # a stream that nothing uses after its failed capture
    assert hip["hipStreamCreate"](C.byref(own)) == 0
    with torch.cuda.stream(torch.cuda.ExternalStream(own.value)):
        assert hip["hipStreamBeginCapture"](own, 2) == 0  # relaxed
        with pytest.raises(GsrError) as ei:
            fwd()
        assert ei.value.status == 4, ei.value
        assert hip["hipStreamEndCapture"](own, C.byref(graph)) != 0 and not graph.value
    hip["hipStreamDestroy"](own)
    rast.lib.hipGetLastError()
    for x in out:
        x.fill_(0)
    fwd()
    torch.cuda.synchronize()
    for x, y in zip(out, want):
        assert torch.equal(x, y)
