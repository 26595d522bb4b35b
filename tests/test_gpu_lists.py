"""Views and lists off every alignment: widths that are no multiple of 4, fewer
fragments than one thread takes, rows that end in the middle of a thread's
four, fragment and result pointers off 16 and 4 bytes, fragments beyond every
side of the map, and maps narrower than the three texels read at once; the
plain entry points, plans and the engine."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

GUARD = 5


@pytest.fixture(scope="module")
def rb():
    import paper_1711_07793_amd as rb
    rb.load_library()
    return rb


def _inputs(W, H, n, vw, seed):
    rng = np.random.default_rng(seed)
    m = np.where(rng.random((H, W)) < 0.4, np.float32(0.5), np.float32(0.9)).astype(np.float32)
    k = np.arange(n)
    w = vw if vw else 40
    u = ((k % w) + rng.random(n)) / w * 1.5 - 0.25
    v = ((k // w) + rng.random(n)) / max(1, (n + w - 1) // w) * 1.5 - 0.25
    return m, np.stack([u, v, rng.choice([0.45, 0.7, 0.95], n)], 1).astype(np.float32)


def _out(n, dtype):
    """A result tensor that starts off every alignment, and its surroundings."""
    buf = torch.full((n + 2 * GUARD,), 77, dtype=dtype, device="cuda")
    return buf[GUARD:GUARD + n], buf


@pytest.mark.parametrize("W,H", [(1, 1), (2, 5), (3, 3), (64, 48)])
@pytest.mark.parametrize("vw", [0, 1, 3, 6, 33, 40])
def test_views_and_lists_off_alignment(rb, W, H, vw):
    md = None
    for n in (1, 2, 3, 4, 5, 7, 130, 255, 1023, 1027, 2051):
        print(f"lists {W}x{H} vw={vw} n={n}", flush=True)
        m, f = _inputs(W, H, n, vw, 1000 * W + 10 * n + vw)
        md = torch.from_numpy(m).cuda()
        fbuf = torch.empty(3 * n + 1, device="cuda")
        fbuf[1:] = torch.from_numpy(f.reshape(-1)).cuda()
        fd = fbuf[1:].view(n, 3)
        p = dict(width=W, height=H, pitch=W, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=vw)
        want = {0: oracle.rbsm_hard(m, f, p), 1: oracle.rsmss(m, f, p), 2: oracle.shadow_map(m, f, p)}
        jobs, bufs = [], []
        for mode, dtype, fn in ((0, torch.uint8, rb.rbsm_visibility), (1, torch.float32, rb.rsmss_visibility)):
            out, buf = _out(n, dtype)
            fn(md, fd, p, out=out)
            bufs.append((mode, out, buf))
            out, buf = _out(n, dtype)
            jobs.append(dict(map=md, frags=fd, params=p, mode=mode, out=out))
            bufs.append((mode, out, buf))
        rb.Plan(jobs).launch()
        out, buf = _out(n, torch.uint8)
        rb.sm_visibility(md, fd, p, out=out)
        bufs.append((2, out, buf))
        torch.cuda.synchronize()
        for mode, out, buf in bufs:
            got = out.cpu().numpy()
            if mode != 1:
                assert np.array_equal(got, want[mode])
            else:  # at most two roundings of values up to 1 apart
                assert np.max(np.abs(got - want[1])) <= 2.0 ** -22
            around = torch.cat([buf[:GUARD], buf[-GUARD:]])
            assert bool((around == 77).all())


@pytest.mark.parametrize("vw,n", [(256, 64 * 256), (256, 64 * 256 - 1), (257, 70 * 257 + 3), (1023, 65 * 1023 - 1), (255, 20000)])
def test_plain_views_in_tiles(rb, vw, n):
    """Plain shadow mapping on both sides of the sizes that go in screen tiles, with ragged tiles."""
    m, f = _inputs(64, 48, n, vw, n)
    p = dict(width=64, height=48, pitch=64, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=vw)
    out, buf = _out(n, torch.uint8)
    rb.sm_visibility(torch.from_numpy(m).cuda(), torch.from_numpy(f).cuda(), p, out=out)
    assert np.array_equal(out.cpu().numpy(), oracle.shadow_map(m, f, p))
    assert bool((torch.cat([buf[:GUARD], buf[-GUARD:]]) == 77).all())


@pytest.mark.parametrize("vw", [0, 6, 33])
@pytest.mark.parametrize("n", [3, 130, 1027])
@pytest.mark.parametrize("keep", [False, True])
def test_engine_composites_off_alignment(rb, n, vw, keep):
    """One pass for a view's lights and its composite: the composite is the weighted sum of the
    per-light results, which are stored only when asked for."""
    W, H = 64, 48
    m, f = _inputs(W, H, n, vw, 5 * n + vw)
    fbuf = torch.empty(3 * n + 1, device="cuda")
    fbuf[1:] = torch.from_numpy(f.reshape(-1)).cuda()
    fd = fbuf[1:].view(n, 3)
    p = dict(width=W, height=H, pitch=W, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=vw)
    vis = [oracle.rbsm_hard(m, f, p), oracle.rsmss(m, f, p), oracle.rsmss(m, f, p)]
    modes, weights = [0, 1, 1], [0.75, 0.3, -1.5]
    eng = rb.Engine(1 << 20, 4)
    lid = eng.add_light(torch.from_numpy(m).cuda())
    comp, cbuf = _out(n, torch.float32)
    outs = [_out(n, torch.float32 if mode else torch.uint8) for mode in modes]
    lights = [dict(light=lid, mode=mode, frags=fd, depth_bias=1e-4, max_dist=9, weight=w, out=outs[k][0] if keep else None)
              for k, (mode, w) in enumerate(zip(modes, weights))]
    eng.wait(eng.submit(n, lights, view_width=vw, composite=comp))
    assert np.max(np.abs(comp.cpu().numpy() - oracle.composite(vis, weights))) <= 2.0 ** -20
    assert bool((torch.cat([cbuf[:GUARD], cbuf[-GUARD:]]) == 77).all())
    for k, (out, buf) in enumerate(outs):
        if keep:
            assert np.max(np.abs(out.cpu().numpy().astype(np.float64) - vis[k])) <= 2.0 ** -22
            assert bool((torch.cat([buf[:GUARD], buf[-GUARD:]]) == 77).all())
        else:
            assert bool((buf == 77).all())
    eng.close()


@pytest.mark.parametrize("tile_w", [16, 32, 64])
@pytest.mark.parametrize("vw,n", [(1, 70), (15, 15 * 65 + 1), (31, 31 * 33 - 1), (64, 64 * 16), (65, 65 * 31 + 64), (130, 130 * 66 + 7)])
def test_tile_edges(rb, tile_w, vw, n):
    """Views that end inside a tile on either side and in the middle of a row, at every tile width, hard and soft."""
    m, f = _inputs(64, 48, n, vw, n)
    p = dict(width=64, height=48, pitch=64, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=vw)
    md, fd = torch.from_numpy(m).cuda(), torch.from_numpy(f).cuda()
    for hard, dtype, fn in ((True, torch.uint8, oracle.rbsm_hard), (False, torch.float32, oracle.rsmss)):
        want = fn(m, f, p)
        for persistent in (0, 1):
            out, buf = _out(n, dtype)
            rb.rbsm_pass_tuned(0 if hard else 1, md, fd, p, (tile_w, 1, 2048, persistent, 0, 0, 3), out=out)
            got = out.cpu().numpy()
            if hard:
                assert np.array_equal(got, want)
            else:  # at most two roundings of values up to 1 apart
                assert np.max(np.abs(got - want)) <= 2.0 ** -22
            assert bool((torch.cat([buf[:GUARD], buf[-GUARD:]]) == 77).all())


@pytest.mark.parametrize("n", [2 ** 28 + 5, 2 ** 31 - 1])
def test_views_past_32_bit_indices(rb, n):
    """A view whose fragment indices need the 64-bit forms: the bits of the same fragments given as a list."""
    m, _ = _inputs(64, 48, 4, 0, 5)
    md = torch.from_numpy(m).cuda()
    f = torch.empty((n, 3), device="cuda").uniform_(-0.02, 1.02, generator=torch.Generator(device="cuda").manual_seed(3))
    p = dict(width=64, height=48, pitch=64, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=0)
    want = rb.rbsm_visibility(md, f, p)
    print(f"views n={n}", flush=True)
    view = dict(p, view_width=4099)
    assert torch.equal(rb.rbsm_visibility(md, f, view), want)
    got = torch.full_like(want, 77)
    plan = rb.Plan([dict(map=md, frags=f, params=view, mode=0, out=got)])
    plan.launch()
    assert torch.equal(got, want)


@pytest.mark.parametrize("pitch,H", [(2 ** 22 - 1, 200), (2 ** 22, 200), (5_000_001, 100), (2 ** 30 - 64, 1), (2 ** 29, 2)])
def test_long_pitch(rb, pitch, H):
    """Narrow maps whose rows lie far apart, below and above the 2^24 bytes a row that 24-bit
    multiplies could take, with fragments spread over them so that their texels do not fit LDS: views, plans and the engine."""
    W, vw, n = 64, 33, 33 * 70
    m, f = _inputs(W, H, n, vw, 11)
    f = f[np.random.default_rng(1).permutation(n)]  # every tile spans the map
    full = torch.full((H, pitch), float("nan"), device="cuda")  # reads beside the map differ from it
    md = full[:, :W]
    md.copy_(torch.from_numpy(m))
    fd = torch.from_numpy(f).cuda()
    eng = rb.Engine(1 << 20, 4)
    lid = eng.add_light(md)
    for view_width in (vw, 0):
        p = dict(width=W, height=H, pitch=pitch, depth_bias=1e-4, max_dist=9, kernel_radius=0, view_width=view_width)
        want = {0: oracle.rbsm_hard(m, f, dict(p, pitch=W)), 1: oracle.rsmss(m, f, dict(p, pitch=W))}
        for mode, dtype, fn in ((0, torch.uint8, rb.rbsm_visibility), (1, torch.float32, rb.rsmss_visibility)):
            print(f"pitch {pitch} vw={view_width} mode={mode}", flush=True)
            got = [fn(md, fd, p), rb.rbsm_pass_tuned(mode, md, fd, p, (32, 1, 0, 0, 0, 0, 3)),
                   rb.rbsm_pass_tuned(mode, md, fd, p, (16, 1, 256, 1, 0, 0, 3))]
            got += [torch.empty(n, dtype=dtype, device="cuda") for _ in range(2)]
            rb.Plan([dict(map=md, frags=fd, params=p, mode=mode, out=got[3])]).launch()
            eng.wait(eng.submit(n, [dict(light=lid, mode=mode, frags=fd, depth_bias=1e-4, max_dist=9, out=got[4])],
                                view_width=view_width))
            torch.cuda.synchronize()
            for g in got:  # at most two roundings of values up to 1 apart
                assert np.max(np.abs(g.cpu().numpy().astype(np.float64) - want[mode])) <= (0 if mode == 0 else 2.0 ** -22)
    eng.close()
