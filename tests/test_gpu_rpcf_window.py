"""RPCF against the oracle at every window size, in one part and in several:
radii at the edges of the kernel's word sizes, traversal lengths on both sides
of a word's 32 bits, tiles whose texels fit LDS, that do not but lie inside
the map, and that hang over its borders, and traversals that run out of the
window."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rb():
    import paper_1711_07793_amd as rb
    rb.load_library()
    return rb


def _map(W, H, rng):
    """A receiver tilted enough that every window holds a line where tests
    against a fragment's own depth change, blocks with long straight edges,
    single texels, NaN and both zeros."""
    y, x = np.mgrid[0:H, 0:W]
    m = (0.7 + 0.13 * x / W + 0.08 * y / H).astype(np.float32)
    for _ in range(10):
        x0, y0 = int(rng.integers(0, W)), int(rng.integers(0, H))
        w, h = int(rng.integers(1, W // 2)), int(rng.integers(1, H // 3))
        m[y0:y0 + h, x0:x0 + w] = rng.choice(np.array([0.3, 0.5, -0.0, 0.0], np.float32))
    k = rng.choice(W * H, 60, replace=False)
    m.reshape(-1)[k[:40]] = 0.2
    m.reshape(-1)[k[40:]] = np.nan
    return m


def _view(W, H, vw, vh, step, x0, y0, rng):
    """A screen image of `step` texels a pixel from texel (x0, y0)."""
    py, px = np.mgrid[0:vh, 0:vw]
    u = ((x0 + step * (px + 0.3 * py / vh + 0.37)) / W).reshape(-1)
    v = ((y0 + step * (py + 0.21)) / H).reshape(-1)
    z = 0.7 + 0.13 * u + 0.08 * v + 3e-4
    z = np.where(rng.random(len(z)) < 0.1, rng.choice([0.4, 0.6, 0.0, -0.0], len(z)), z)
    return np.stack([u, v, z], 1).astype(np.float32)


@pytest.mark.parametrize("r,max_dist", [(1, 1), (2, 64), (3, 5), (4, 31), (5, 32), (6, 16), (7, 33), (8, 64), (9, 2),
                                        (10, 16), (11, 40), (12, 16), (13, 64), (14, 16), (14, 64), (15, 16),
                                        (16, 64), (17, 16), (18, 64), (21, 8), (22, 64), (26, 8), (27, 64), (32, 64)])
def test_every_window(rb, r, max_dist):
    rng = np.random.default_rng(100 * r + max_dist)
    W, H = 331, 243
    m = _map(W, H, rng)
    views = {
        "staged": (_view(W, H, 37, 19, 0.9, 120.0, 90.0, rng), 37),     # ragged tiles, windows inside the map
        "border": (_view(W, H, 37, 19, 0.9, -12.0, -7.0, rng), 37),     # clamped band
        "spread": (_view(W, H, 20, 16, 6.0, 110.0, 78.0, rng), 20),     # box too large for LDS
        "spread border": (_view(W, H, 40, 30, 9.0, -20.0, -10.0, rng), 40),
        "flat": (_view(W, H, 300, 1, 0.7, 60.0, 100.0, rng), 0),
    }
    md = torch.from_numpy(m).cuda()
    count = max(12, min(700, 60000 // (2 * r + 1) ** 2))
    for name, (f, vw) in views.items():
        print(f"window r={r} maxd={max_dist} {name}", flush=True)
        p = dict(width=W, height=H, pitch=W, depth_bias=1e-4, max_dist=max_dist, kernel_radius=r, view_width=vw)
        got = rb.rsmss_visibility(md, torch.from_numpy(f).cuda(), p).cpu().numpy()
        idx = np.sort(rng.choice(len(f), min(count, len(f)), replace=False))
        want = oracle.rsmss(m, np.ascontiguousarray(f[idx]), p)
        # both are the exact mean rounded to binary32 up to one step, and at most 1
        assert np.max(np.abs(got[idx].astype(np.float64) - want)) <= 2.0 ** -24
        assert np.all((got >= 0) & (got <= 1))
