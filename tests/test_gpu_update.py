"""The optimiser step at the ends of its four-element groups, and with arrays
that are not 16-byte aligned: both paths give the same bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,deg", [(1, 0), (2, 1), (3, 0), (5, 2), (341, 3), (4097, 1)])
def test_adam_alignment_changes_nothing(n, deg):
    import torch
    from paper_2411_17660_amd.raster import Rasterizer
    rast = Rasterizer()
    K = (deg + 1) ** 2
    gen = torch.Generator().manual_seed(n)
    shapes = {"means": (n, 3), "sh": (n, K, 3)}
    vals = {(g, k): torch.randn(s, generator=gen).abs() for k, s in shapes.items()
            for g in ("p", "g", "m", "v")}
    out = []
    for shift in (0, 1):
        def place(t):  # `shift` floats past a 16-byte boundary
            buf = torch.zeros(t.numel() + 4, device="cuda")
            v = buf[shift:shift + t.numel()].view(t.shape)
            v.copy_(t)
            return v
        d = {k: place(t) for k, t in vals.items()}
        p = {k: d["p", k] for k in shapes}
        p["poses"] = torch.eye(3, 4, device="cuda")[None].contiguous()
        g = {k: d["g", k] for k in shapes}
        g["twist"] = torch.zeros(1, 6, device="cuda")
        st = {f"{m}_{k}": d[m, k] for k in shapes for m in "mv"}
        st.update(m_twist=torch.zeros(1, 6, device="cuda"),
                  v_twist=torch.zeros(1, 6, device="cuda"),
                  step=torch.zeros(1, dtype=torch.int32, device="cuda"))
        for _ in range(2):
            rast.adam_step(p, g, st)
        assert int(st["step"]) == 2
        out.append([d[k].clone() for k in d])
        assert all(bool((a != b.cuda()).any()) for a, b in
                   ((p[k], vals["p", k]) for k in shapes))
    for a, b in zip(*out):
        assert torch.equal(a, b)
