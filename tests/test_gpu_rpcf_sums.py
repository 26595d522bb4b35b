"""RPCF sums at their extremes against the oracle: boxes in which every term has
a discontinuity and the value 1 or 0, up to the largest radius, and boxes whose
few nonzero terms are far below one."""
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


@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 8, 9, 12, 13, 14, 15, 17, 21, 26, 32])
@pytest.mark.parametrize("along_x", [True, False])
@pytest.mark.parametrize("rows", [60, 1500])
def test_small_means(rb, r, along_x, rows):
    """Fragments in the map's first column (or row), at positions down to 2^-90 texels in it: dark but for the
    first texels of one-texel-wide lit corridors, two long and r texels away, which are worth half that position.
    Beside them in every wave, fragments at ordinary positions.  The result is the exact mean rounded, up to one
    step, which is 2^-23 of it.  1500 rows of texels spread every tile over more of them than fit LDS."""
    w = 128
    m = np.full((rows, w), 0.2, np.float32)
    m[:, r + 2:] = 0.9
    m[2::3, r:r + 2] = 0.9
    rng = np.random.default_rng(r)
    n, vw = 40 * 16, 16
    x = 2.0 ** rng.uniform(-90.0, -18.0, n)
    x = np.where(rng.random(n) < 0.3, rng.random(n), x)          # ordinary positions of the same texel
    x = np.where(rng.random(n) < 0.1, x + 1.0, x)                # and of the next one
    y = (np.arange(n) // vw + 0.5 * rng.random(n)) * rows / 40   # the other coordinate is an ordinary one
    f = np.stack([x / w, y / rows, np.full(n, 0.5)], 1).astype(np.float32)
    width, height = w, rows
    if not along_x:
        m, f, width, height = np.ascontiguousarray(m.T), np.ascontiguousarray(f[:, [1, 0, 2]]), rows, w
    md, fd = torch.from_numpy(m).cuda(), torch.from_numpy(f).cuda()
    idx = np.sort(rng.choice(n, 200 if r < 10 else 60, replace=False))
    for view_width in (vw, 0):
        print(f"small r={r} along_x={along_x} rows={rows} vw={view_width}", flush=True)
        p = dict(width=width, height=height, pitch=width, depth_bias=0.0, max_dist=16, kernel_radius=r, view_width=view_width)
        got = rb.rsmss_visibility(md, fd, p).cpu().numpy()[idx].astype(np.float64)
        want = oracle.rsmss(m, np.ascontiguousarray(f[idx]), p).astype(np.float64)
        assert np.sum((want > 0) & (want < 2.0 ** -30)) > 10
        assert np.all(np.abs(got - want) <= 2.0 ** -23 * want)
