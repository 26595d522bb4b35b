"""Composites of the serving engine on both sides of the step size from which a
view's lights are taken one after the other: the bits of the plain entry points
and the compositing call, with ragged tiles and buffers off every alignment."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

GUARD = 5
TILES = 7 * 256  # 32 x 32 tiles of a step


@pytest.fixture(scope="module")
def rb():
    import paper_1711_07793_amd as rb
    rb.load_library()
    return rb


def _off(n, dtype, fill=77):
    """n elements that start off every alignment, and their surroundings."""
    buf = torch.full((n + 2 * GUARD,), fill, dtype=dtype, device="cuda")
    return buf[GUARD:GUARD + n], buf


def _request(rb, md, lid, vw, n, lights, keep, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    fbuf = torch.empty(3 * n + 1, device="cuda")
    f = fbuf[1:].view(n, 3)
    k = torch.arange(n, device="cuda")
    rows = (n + vw - 1) // vw
    f[:, 0] = ((k % vw) + torch.rand(n, generator=g, device="cuda")) / vw * 1.1 - 0.05
    f[:, 1] = ((k // vw) + torch.rand(n, generator=g, device="cuda")) / rows * 1.1 - 0.05
    f[:, 2] = 0.7
    p = dict(width=md.shape[1], height=md.shape[0], depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=vw)
    modes = [(seed + l) % 2 for l in range(lights)]
    weights = [0.75 - 0.4 * l for l in range(lights)]
    vis = [rb.rsmss_visibility(md, f, p) if m else rb.rbsm_visibility(md, f, p) for m in modes]
    want = rb.rbsm_composite(vis, modes, weights)
    outs = [_off(n, torch.float32 if m else torch.uint8) for m in modes]
    comp, cbuf = _off(n, torch.float32)
    spec = [dict(light=lid, mode=m, frags=f, depth_bias=1e-4, max_dist=9, weight=w, out=outs[l][0] if keep else None)
            for l, (m, w) in enumerate(zip(modes, weights))]
    return dict(n=n, lights=spec, view_width=vw, composite=comp), want, vis, outs, cbuf


@pytest.mark.parametrize("vw,n", [(1024, 1024 * 32 * (TILES // 32 - 1)), (1024, 1024 * 32 * (TILES // 32)),
                                  (1023, 1023 * (32 * 55 + 1) + 7), (1025, 1025 * 32 * 54 - 3), (31, 31 * 32 * TILES - 30),
                                  (1, 70)])
@pytest.mark.parametrize("lights,keep", [(1, False), (1, True), (2, True), (4, False), (8, True)])
def test_composites_equal_plain_calls(rb, vw, n, lights, keep):
    rng = np.random.default_rng(n)
    m = np.where(rng.random((211, 300)) < 0.1, np.float32(0.5), np.float32(0.9)).astype(np.float32)
    md = torch.from_numpy(m).cuda()
    eng = rb.Engine(1 << 30, 8)
    lid = eng.add_light(md)
    print(f"views vw={vw} n={n} lights={lights} keep={keep}", flush=True)
    # a small request in the same burst: its own step, or one with the large one
    reqs = [_request(rb, md, lid, vw, n, lights, keep, 3), _request(rb, md, lid, 33, 33 * 40 + 5, lights, keep, 4)]
    torch.cuda.synchronize()
    for t in [eng.submit(**r[0]) for r in reqs]:
        eng.wait(t)
    for r, want, vis, outs, cbuf in reqs:
        assert torch.equal(r["composite"], want)
        assert bool((torch.cat([cbuf[:GUARD], cbuf[-GUARD:]]) == 77).all())
        for v, (out, buf) in zip(vis, outs):
            assert torch.equal(out, v) if keep else bool((buf == 77).all())
            assert bool((torch.cat([buf[:GUARD], buf[-GUARD:]]) == 77).all())
    eng.close()
