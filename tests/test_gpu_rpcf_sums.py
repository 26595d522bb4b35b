"""RPCF sums at their extremes against the oracle: boxes in which every term has
a discontinuity and the value 1 or 0, up to the largest radius."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

W, H = 331, 243


@pytest.fixture(scope="module")
def rb():
    import paper_1711_07793_amd as rb
    rb.load_library()
    return rb


def _view(vw, vh, step, x0, y0, z):
    """A screen image of `step` texels a pixel from texel (x0, y0), all of depth z."""
    py, px = np.mgrid[0:vh, 0:vw]
    u = ((x0 + step * (px + 0.3 * py / vh + 0.37)) / W).reshape(-1)
    v = ((y0 + step * (py + 0.21)) / H).reshape(-1)
    return np.stack([u, v, np.full(len(u), z)], 1).astype(np.float32)


VIEWS = {
    "staged": (_view(37, 19, 0.9, 120.0, 90.0, 0.5), 37),           # windows inside the map, texels in LDS
    "border": (_view(37, 19, 0.9, -12.0, -7.0, 0.5), 37),           # over the map's corner
    "spread": (_view(20, 16, 4.0, 110.0, 78.0, 0.5), 20),           # box too large for LDS, inside the map
    "spread border": (_view(40, 30, 9.0, -20.0, -10.0, 0.5), 40),
    "list": (_view(300, 1, 0.3, 100.0, 100.0, 0.5), 0),
}


@pytest.mark.parametrize("r,max_dist", [(5, 16), (14, 8), (15, 16), (31, 8), (32, 1), (32, 8), (32, 64)])
@pytest.mark.parametrize("period,dark", [(5, True), (4, True), (5, False), (4, False)])
def test_every_term_listed(rb, r, max_dist, period, dark):
    """Isolated texels, dark on a lit map or lit on a dark one, on a lattice on which every other texel
    touches one of them: up to 65^2 listed terms, of value 1 (isolated dark) or 0 (isolated lit)."""
    y, x = np.mgrid[0:H, 0:W]
    m = np.where(((x + 2 * y) % period == 0) == dark, np.float32(0.2), np.float32(0.9)).astype(np.float32)
    md = torch.from_numpy(m).cuda()
    rng = np.random.default_rng(10 * r + period)
    for name, (f, vw) in VIEWS.items():
        print(f"listed r={r} maxd={max_dist} period={period} dark={dark} {name}", flush=True)
        p = dict(width=W, height=H, pitch=W, depth_bias=1e-4, max_dist=max_dist, kernel_radius=r, view_width=vw)
        got = rb.rsmss_visibility(md, torch.from_numpy(f).cuda(), p).cpu().numpy()
        idx = np.sort(rng.choice(len(f), 10, replace=False))
        want = oracle.rsmss(m, np.ascontiguousarray(f[idx]), p)
        if name in ("staged", "list"):
            assert np.all(want == (1.0 if dark else 0.0))
        # both are the exact mean rounded to binary32 up to one step, and at most 1
        assert np.max(np.abs(got[idx].astype(np.float64) - want)) <= 2.0 ** -24
