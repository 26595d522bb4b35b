"""Rasterizer regions and batches: map sizes on both sides of each region
size's range and off its multiples, primitive counts around a batch of 256 and
around the 64 kept in LDS, polygons, quads and slabs, equal depths and both
zeros across batches.  Bit-equal to the oracle (coverage and depths are exact
on both sides)."""
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


def _prims(n, rng, spread):
    """n primitives around the map's middle (spread: their reach), a fifth of them slabs or quads, many of equal depth."""
    p = np.zeros(n, oracle.PRIM_DTYPE)
    for k in range(n):
        p[k]["depth"] = rng.choice(np.array([0.0, -0.0, 0.25, 0.5, 0.7, np.nan], np.float32))
        kind = rng.random()
        if kind < 0.1:
            a = rng.uniform(0, np.pi)
            p[k]["kind"] = 1
            p[k]["nx"], p[k]["ny"] = np.cos(a), np.sin(a)
            p[k]["o"], p[k]["w"] = rng.uniform(-0.5, 1.0), rng.uniform(0.001, 0.02)
            continue
        c = 0.5 + spread * rng.uniform(-1, 1, 2)
        nv = 4 if kind < 0.2 else 3
        ang = np.sort(rng.uniform(0, 2 * np.pi, nv)) if nv == 3 else np.arange(4) * np.pi / 2 + rng.uniform(0, 1.5)
        rad = spread * np.exp(rng.uniform(np.log(0.01), np.log(1.0)))
        p[k]["nv"] = nv
        p[k]["x"][:nv] = c[0] + rad * np.cos(ang)
        p[k]["y"][:nv] = c[1] + rad * np.sin(ang)
    return p


@pytest.mark.parametrize("W,H", [(1024, 1024), (1025, 1024), (2048, 2048), (2049, 2047), (2051, 2111), (64, 16), (65, 17),
                                 (65536, 3), (5, 65536)])
@pytest.mark.parametrize("n", [1, 64, 65, 256, 257, 600])
def test_regions_and_batches(rb, W, H, n):
    print(f"raster regions {W}x{H} n={n}", flush=True)
    rng = np.random.default_rng(W + 7 * H + n)
    rec = (0.6, 0.05, -0.03)
    # many primitives over a few regions, then spread over the map
    for spread in (0.05, 0.6):
        p = _prims(n, rng, spread)
        d = torch.from_numpy(p.view(np.uint8)).cuda()
        got = rb.rbsm_rasterize(d, rec, W, H).cpu().numpy()
        ti = np.concatenate([rng.integers(0, W, 4000), np.clip(W // 2 + rng.integers(-W // 18 - 2, W // 18 + 2, 4000), 0, W - 1)])
        tj = np.concatenate([rng.integers(0, H, 4000), np.clip(H // 2 + rng.integers(-H // 18 - 2, H // 18 + 2, 4000), 0, H - 1)])
        ti = np.concatenate([ti, [0, W - 1, 0, W - 1]])
        tj = np.concatenate([tj, [0, 0, H - 1, H - 1]])
        want = oracle.raster_texels(p, rec, W, H, ti, tj)
        assert np.array_equal(got[tj, ti].view(np.uint32), want.view(np.uint32))
