"""Performance cases of the RBSM / RSMSS shadow pass.

Each case is one piece of work that a renderer gives this framework: a shadow
pass over one view, a batched frame of many views and lights, a burst of
serving requests, a shadow-map rasterization, or a composite of several
lights.  Scenes and cameras follow the recipes of the repository's synthetic
workloads (random constant-depth triangles, optionally a fence of thin bars,
over a tilted receiver; a perspective camera ray-cast in light space), made
here in float64 with torch so a 4K frame takes milliseconds.

``listed()`` names the cases, ``draw`` gives more of the same ranges,
``prepare`` makes the inputs on the GPU from a seed, ``run`` is one pass
through the public entry points, ``work`` its least bytes and operations, and
``exact`` the same results in 64 bits from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1711_07793_amd as rb

BIAS = 1e-4
RECEIVER = (0.9, 0.05, 0.03)  # depth at the map's centre and its slopes
PRIM = np.dtype([("kind", "<i4"), ("nv", "<i4"), ("x", "<f8", (4,)), ("y", "<f8", (4,)), ("nx", "<f8"),
                 ("ny", "<f8"), ("o", "<f8"), ("w", "<f8"), ("depth", "<f4"), ("pad", "<i4")])

# views and maps of the batched frame and of the serving pool
BATCH_VIEWS = [(1280, 720), (1280, 720), (1920, 1080), (1920, 1080), (2560, 1440), (2560, 1440), (3840, 2160),
               (3840, 2160)]
CASCADES = [8192, 4096, 2048, 1024]
SPOTS = [1024, 2048, 4096, 1024, 4096, 2048, 2048, 1024, 4096, 2048, 1024, 4096]
SERVE_VIEWS = [(1280, 720), (1920, 1080), (3840, 2160)]


def listed():
    view = dict(kind="view", scene="tris", tris=64, pitch=0, flat=False, radius=0)
    return [
        # the smallest call: scattered probe points against a small map, bound by latency and launch cost
        dict(name="hard_64k_points", kind="view", entry="hard", scene="quad", tris=1, map_w=512, map_h=512, pitch=0,
             view_w=65536, view_h=1, flat=True, max_dist=16, radius=0),
        # one light of a full-HD frame, the paper's hard-shadow setting
        dict(view, name="hard_1080p", entry="hard", map_w=2048, map_h=2048, view_w=1920, view_h=1080, max_dist=32),
        # a laptop panel's view (rows that are no multiple of 4) over a non-square padded map
        dict(view, name="hard_768p_ragged", entry="hard", map_w=1500, map_h=1100, pitch=1536, view_w=1366, view_h=768,
             max_dist=16),
        # a 4K frame's filtered penumbra over thin bars: the largest single view
        dict(view, name="rsmss_4k_fence", entry="rsmss", scene="fence", tris=256, map_w=4096, map_h=4096, view_w=3840,
             view_h=2160, max_dist=16),
        # the visible fragments of a view as a compacted list of odd length, no screen layout
        dict(view, name="rsmss_visible_list", entry="rsmss", map_w=2048, map_h=2048, view_w=1921, view_h=1081,
             flat=True, max_dist=16),
        # a wide filtered penumbra (box of 11 x 11 texels) on the 4K frame
        dict(view, name="rpcf_4k_r5", entry="rsmss", scene="fence", tris=256, map_w=4096, map_h=4096, view_w=3840,
             view_h=2160, max_dist=16, radius=5),
        # the widest lights' penumbra (27 x 27 texels) at full HD
        dict(view, name="rpcf_1080p_r13", entry="rsmss", map_w=2048, map_h=2048, view_w=1920, view_h=1080, max_dist=16,
             radius=13),
        # plain shadow mapping of a full-HD frame: the unfiltered baseline a renderer falls back to
        dict(view, name="sm_1080p", entry="sm", map_w=2048, map_h=2048, view_w=1920, view_h=1080, max_dist=16),
        # a whole frame: 8 views, a directional light's cascades and spot lights, one captured plan
        dict(name="batch_8views", kind="batch", views=8, shrink=1.0, form="graph"),
        # a burst of 32 requests to the serving engine, 1-4 lights each, composited
        dict(name="serve_32", kind="serve", requests=32, lights=8, shrink=1.0),
        # a spot light's map, drawn anew each frame
        dict(name="raster_1024", kind="raster", tris=64, fence=False, map_w=1024, map_h=1024, pitch=0),
        # a directional light's finest cascade
        dict(name="raster_8192", kind="raster", tris=64, fence=False, map_w=8192, map_h=8192, pitch=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["points", "sm", "hard", "rsmss", "rsmss", "rpcf", "rpcf", "batch", "serve", "raster", "raster",
                       "composite"])
    map_w = _log_int(rng, 300, 8192)
    map_h = map_w if rng.random() < 0.5 else max(256, min(8192, int(map_w * rng.uniform(0.6, 1.6))))
    pitch = (map_w + 63) // 64 * 64 if rng.random() < 0.3 else 0
    if kind == "points":
        return dict(kind="view", entry=rng.choice(["hard", "rsmss"]), scene="quad", tris=1, map_w=map_w, map_h=map_h,
                    pitch=pitch, view_w=_log_int(rng, 1000, 500000), view_h=1, flat=True,
                    max_dist=rng.choice([8, 16, 32]), radius=0)
    if kind in ("sm", "hard", "rsmss", "rpcf"):
        view_w = _log_int(rng, 320, 3840)
        view_h = max(90, min(2160, int(view_w * rng.uniform(0.5, 0.75))))
        radius = 0
        if kind == "rpcf":
            radius = rng.randint(1, 15)
            while view_w * view_h * (2 * radius + 3) ** 2 > 1.4e9:
                view_w, view_h = view_w * 7 // 8, view_h * 7 // 8
        scene = rng.choice(["tris", "tris", "fence"])
        return dict(kind="view", entry="rsmss" if kind == "rpcf" else kind, scene=scene, tris=rng.choice([64, 128, 256]),
                    map_w=map_w, map_h=map_h, pitch=pitch, view_w=view_w, view_h=view_h, flat=rng.random() < 0.2,
                    max_dist=rng.choice([8, 16, 24, 32]), radius=radius)
    if kind == "batch":
        return dict(kind="batch", views=rng.randint(1, 7), shrink=round(rng.uniform(1.0, 6.0), 3),
                    form=rng.choice(["graph", "graph", "launch", "noalloc"]))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(4, 31), lights=rng.randint(4, 8),
                    shrink=round(rng.uniform(1.0, 4.0), 3))
    if kind == "raster":
        return dict(kind="raster", tris=rng.choice([16, 64, 256]), fence=rng.random() < 0.3, map_w=map_w, map_h=map_h,
                    pitch=pitch)
    return dict(kind="composite", n=_log_int(rng, 20000, 8294400), lights=rng.randint(1, 8), seed=rng.randint(0, 999))


# ---------------------------------------------------------------------------
# scenes, maps and fragments
# ---------------------------------------------------------------------------

class Scene:
    """Triangles (sorted by depth) and, when asked for, a fence of 32 bars of one depth."""

    def __init__(self, rng, width, height, tris, fence=False, quad=False):
        self.w, self.h = width, height
        self.receiver = (0.9, 0.0, 0.0) if quad else RECEIVER
        self.polys, self.bars = [], None
        if quad:
            side, rot = rng.uniform(0.3, 0.6), rng.uniform(0.0, math.pi / 2)
            cx, cy = rng.uniform(0.3, 0.7, 2)
            c, s = math.cos(rot) * side / 2, math.sin(rot) * side / 2
            corners = [(-1, -1), (1, -1), (1, 1), (-1, 1)]
            self.polys.append(([(cx + x * c - y * s, cy + x * s + y * c) for x, y in corners],
                               float(np.float32(rng.uniform(0.2, 0.5)))))
            return
        while len(self.polys) < tris:
            x0, y0 = rng.random(2)
            length = np.exp(rng.uniform(math.log(8.0), math.log(512.0), 2))
            ang = rng.uniform(0.0, 2 * math.pi, 2)
            x = x0 + length * np.cos(ang) / width
            y = y0 + length * np.sin(ang) / height
            if min(x.min(), y.min()) < 0.0 or max(x.max(), y.max()) > 1.0:
                continue
            pts = [(float(x0), float(y0)), (float(x[0]), float(y[0])), (float(x[1]), float(y[1]))]
            area = sum(a[0] * b[1] - b[0] * a[1] for a, b in zip(pts, pts[1:] + pts[:1]))
            self.polys.append((pts if area > 0 else pts[::-1], float(np.float32(rng.uniform(0.1, 0.8)))))
        self.polys.sort(key=lambda p: p[1])
        if fence:
            ang = rng.uniform(0.0, math.pi)
            nx, ny = math.cos(ang), math.sin(ang)
            depth = float(np.float32(rng.uniform(0.1, 0.8)))
            widths = rng.integers(1, 4, 32) / max(width, height)
            gaps = rng.integers(8, 33, 32) / max(width, height)
            ends = [nx * x + ny * y for x in (0, 1) for y in (0, 1)]
            slack = max(0.0, max(ends) - min(ends) - float((widths + gaps).sum()))
            start = min(ends) + slack * rng.random()
            starts = start + np.concatenate([[0.0], np.cumsum(widths + gaps)[:-1]])
            self.bars = (nx, ny, starts, widths, depth)

    def records(self):
        """The primitives as rbsm_prim records."""
        out = np.zeros(len(self.polys) + (32 if self.bars else 0), dtype=PRIM)
        for r, (pts, depth) in zip(out, self.polys):
            r["kind"], r["nv"], r["depth"] = 0, len(pts), depth
            for e, (x, y) in enumerate(pts):
                r["x"][e], r["y"][e] = x, y
        if self.bars:
            nx, ny, starts, widths, depth = self.bars
            for r, o, w in zip(out[len(self.polys):], starts, widths):
                r["kind"], r["nx"], r["ny"], r["o"], r["w"], r["depth"] = 1, nx, ny, o, w, depth
        return out

    def in_bars(self, u, v):
        nx, ny, starts, widths, _ = self.bars
        t = nx * u + ny * v
        lo = torch.from_numpy(starts).to(t.device)
        hi = torch.from_numpy(starts + widths).to(t.device)
        b = torch.searchsorted(lo, t, right=True) - 1
        return (b >= 0) & (t < hi[b.clamp(min=0)])

    def map64(self):
        """The depth map in float64: the nearest surface at every texel centre."""
        r0, ru, rv = self.receiver
        px = (torch.arange(self.w, dtype=torch.float64, device="cuda") + 0.5) / self.w
        py = (torch.arange(self.h, dtype=torch.float64, device="cuda") + 0.5) / self.h
        m = (r0 + ru * (px - 0.5))[None, :] + (rv * (py - 0.5))[:, None]
        for pts, depth in self.polys:
            x, y = [p[0] for p in pts], [p[1] for p in pts]
            i0, i1 = max(int(min(x) * self.w) - 1, 0), min(int(max(x) * self.w) + 2, self.w)
            j0, j1 = max(int(min(y) * self.h) - 1, 0), min(int(max(y) * self.h) + 2, self.h)
            if i0 >= i1 or j0 >= j1:
                continue
            inside = _in_poly(pts, px[None, i0:i1], py[j0:j1, None])
            part = m[j0:j1, i0:i1]
            part.copy_(torch.where(inside, part.clamp(max=depth), part))
        if self.bars:
            for j in range(0, self.h, 1024):
                part = m[j:j + 1024]
                inside = self.in_bars(px[None, :], py[j:j + 1024, None])
                part.copy_(torch.where(inside, part.clamp(max=self.bars[4]), part))
        return m

    def map(self, pitch=0):
        m = torch.zeros((self.h, pitch or self.w), dtype=torch.float32, device="cuda")[:, :self.w]
        m.copy_(self.map64())
        return m

    def camera(self, rng, view_w, view_h, rows=None):
        """Fragments [n, 3] of rows [r0, r1) of a perspective view: the first surface each pixel's ray meets."""
        r0, r1 = rows or (0, view_h)
        yaw = rng.integers(0, 4) * math.pi / 2 + math.radians(rng.uniform(-8.0, 8.0))
        sp, cp, ty = math.sin(math.radians(35.0)), math.cos(math.radians(35.0)), math.tan(math.radians(20.0))
        sy, cy, tx, zc = math.sin(yaw), math.cos(yaw), ty * view_w / view_h, 0.55
        fwd, up, right = (sp * cy, sp * sy, cp), (cp * cy, cp * sy, -sp), (sy, -cy, 0.0)
        d0, ru, rv = self.receiver
        back = (d0 - zc) / cp
        c = (0.5 - back * fwd[0], 0.5 - back * fwd[1])
        x = ((torch.arange(view_w, dtype=torch.float64, device="cuda") + 0.5) / view_w * 2 - 1)[None, :] * tx
        y = (1 - (torch.arange(r0, r1, dtype=torch.float64, device="cuda") + 0.5) / view_h * 2)[:, None] * ty
        dz = fwd[2] + x * right[2] + y * up[2]  # > 0: every ray leaves the light
        au = (fwd[0] + x * right[0] + y * up[0]) / dz
        av = (fwd[1] + x * right[1] + y * up[1]) / dz
        z = d0 + ru * (c[0] - 0.5) + rv * (c[1] - 0.5) - zc
        z = zc + z / (1.0 - ru * au - rv * av)  # the receiver's depth along the ray
        hits = [(depth, pts) for pts, depth in self.polys if depth > zc]
        if self.bars and self.bars[4] > zc:
            hits.append((self.bars[4], None))
        for depth, pts in sorted(hits, key=lambda h: -h[0]):
            u, v = c[0] + (depth - zc) * au, c[1] + (depth - zc) * av
            inside = _in_poly(pts, u, v) if pts is not None else self.in_bars(u, v)
            z = torch.where(inside, torch.full_like(z, depth), z)
        f = torch.stack([c[0] + (z - zc) * au, c[1] + (z - zc) * av, z], dim=-1)
        return f.to(torch.float32).reshape(-1, 3).contiguous()


def _in_poly(pts, u, v):
    """Counter-clockwise polygon, top-left rule."""
    inside = None
    for (ax, ay), (bx, by) in zip(pts, pts[1:] + pts[:1]):
        e = (bx - ax) * (v - ay) - (by - ay) * (u - ax)
        owns = by < ay or (by == ay and bx < ax)
        ok = e >= 0.0 if owns else e > 0.0
        inside = ok if inside is None else inside & ok
    return inside


def _view_inputs(case, seed):
    rng = np.random.default_rng([seed, 1])
    scene = Scene(rng, case["map_w"], case["map_h"], case["tris"], case["scene"] == "fence", case["scene"] == "quad")
    m = scene.map(case["pitch"])
    if case["scene"] == "quad":  # scattered points on the receiver
        g = torch.Generator(device="cuda").manual_seed(seed)
        f = torch.rand((case["view_w"] * case["view_h"], 3), generator=g, device="cuda")
        f[:, 2] = 0.9
        return m, f
    f = scene.camera(rng, case["view_w"], case["view_h"])
    if case["flat"]:  # the visible fragments: runs of each row, the rest of the view is background
        k = torch.arange(f.shape[0], device="cuda")
        x, y = k % case["view_w"], k // case["view_w"]
        edge = 0.1 + 0.1 * torch.sin(y * 0.02)
        f = f[(x > edge * case["view_w"]) & (x % 97 < 83)].contiguous()
        f = f[:f.shape[0] - (1 - f.shape[0] % 2)]  # an odd count
    return m, f


def _params(case):
    return rb.Params(width=case["map_w"], height=case["map_h"], depth_bias=BIAS, max_dist=case["max_dist"],
                     kernel_radius=case["radius"], view_width=0 if case["flat"] else case["view_w"])


def _batch_jobs(case, seed):
    """The jobs of a frame: every view's rows split over the cascades (hard), two spot lights each over a band (RSMSS).
    The layout is the case's own, scenes and cameras the seed's."""
    rng = np.random.default_rng([seed, 2])
    scenes = [Scene(rng, s, s, 64) for s in CASCADES + SPOTS]
    layout = np.random.default_rng(4001)
    jobs = []
    views = BATCH_VIEWS[len(BATCH_VIEWS) - case["views"]:] if case["shrink"] > 1 else BATCH_VIEWS[:case["views"]]
    for w, h in views:
        w, h = int(w / case["shrink"]), int(h / case["shrink"])
        cam = int(rng.integers(1 << 30))
        cuts = np.concatenate([[0], np.round(np.cumsum(layout.dirichlet([2.0] * 4)) * h).astype(int)])
        cuts[-1] = h
        for c in range(4):
            r0, r1 = h - int(cuts[c + 1]), h - int(cuts[c])
            if r1 > r0:
                jobs.append((c, 0, 32 if c < 2 else 16, cam, w, h, r0, r1))
        for s in layout.choice(12, size=2, replace=False):
            rows = max(1, int(round(layout.uniform(0.3, 1.0) * h)))
            r0 = int(layout.integers(0, h - rows + 1))
            jobs.append((4 + int(s), 1, 16, cam, w, h, r0, r0 + rows))
    used = sorted({j[0] for j in jobs})
    maps = {k: scenes[k].map() for k in used}
    out = []
    for k, mode, maxd, cam, w, h, r0, r1 in jobs:
        f = scenes[k].camera(np.random.default_rng(cam), w, h, (r0, r1))
        side = scenes[k].w
        out.append(dict(map=maps[k], frags=f, mode=mode,
                        params=rb.Params(width=side, height=side, depth_bias=BIAS, max_dist=maxd, view_width=w),
                        out=torch.empty(f.shape[0], dtype=torch.float32 if mode else torch.uint8, device="cuda")))
    return out


def _serve_inputs(case, seed):
    """A pool of lights, each view's fragments for each light, and the burst's requests (view, lights, modes)."""
    rng = np.random.default_rng([seed, 3])
    burst = np.random.default_rng(5001)
    lights = [Scene(rng, s, s, 64) for s in ([1024, 2048, 4096, 8192] * 2)[:case["lights"]]]
    views = [(int(w / case["shrink"]), int(h / case["shrink"])) for w, h in SERVE_VIEWS]
    frags = {(l, v): sc.camera(np.random.default_rng([seed, v]), *views[v])
             for l, sc in enumerate(lights) for v in range(len(views))}
    reqs = []
    for q in range(case["requests"]):
        n = int(burst.integers(1, 5))
        reqs.append((q % 3, [int(x) for x in burst.choice(len(lights), size=n, replace=False)],
                     [int(x) for x in burst.integers(0, 2, n)]))
    return [sc.map() for sc in lights], views, frags, reqs


def _composite_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng([case["seed"], 4])
    modes = [int(x) for x in rng.integers(0, 2, case["lights"])]
    weights = [float(np.float32(x)) for x in rng.uniform(0.05, 1.0, case["lights"])]
    vis = [torch.rand(case["n"], generator=g, device="cuda") for _ in modes]
    return [v if m else (v > 0.4).to(torch.uint8) for v, m in zip(vis, modes)], modes, weights


def _raster_scene(case, seed):
    return Scene(np.random.default_rng([seed, 5]), case["map_w"], case["map_h"], case["tris"], case["fence"])


# ---------------------------------------------------------------------------
# preparing and running
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "view":
        m, f = _view_inputs(case, seed)
        out = torch.empty(f.shape[0], dtype=torch.float32 if case["entry"] == "rsmss" else torch.uint8, device="cuda")
        fn = dict(sm=rb.sm_visibility, hard=rb.rbsm_visibility, rsmss=rb.rsmss_visibility)[case["entry"]]
        return dict(kind=kind, fn=fn, map=m, frags=f, params=_params(case), out=out)
    if kind == "batch":
        jobs = _batch_jobs(case, seed)
        state = dict(kind="noalloc" if case["form"] == "noalloc" else "plan", jobs=jobs,
                     out=[j["out"] for j in jobs])
        if case["form"] != "noalloc":
            state["plan"] = rb.Plan(jobs)
            if case["form"] == "graph":
                state["plan"].capture(torch.cuda.Stream())
        return state
    if kind == "serve":
        maps, views, frags, reqs = _serve_inputs(case, seed)
        engine = rb.Engine(4 << 30, 32)
        ids = [engine.add_light(m) for m in maps]
        torch.cuda.synchronize()
        built, out = [], []
        for v, ls, modes in reqs:
            w, h = views[v]
            out.append(torch.empty(w * h, dtype=torch.float32, device="cuda"))
            lights = [dict(light=ids[l], mode=m, frags=frags[(l, v)], depth_bias=BIAS, max_dist=16,
                           weight=1.0 / len(ls)) for l, m in zip(ls, modes)]
            built.append(engine.build_request(w * h, lights, view_width=w, composite=out[-1]))
        return dict(kind=kind, engine=engine, built=built, out=out)
    if kind == "raster":
        scene = _raster_scene(case, seed)
        prims = torch.from_numpy(scene.records().view(np.uint8)).cuda()
        out = torch.zeros((case["map_h"], case["pitch"] or case["map_w"]), device="cuda")[:, :case["map_w"]]
        return dict(kind=kind, prims=prims, receiver=scene.receiver, w=case["map_w"], h=case["map_h"], out=out)
    vis, modes, weights = _composite_inputs(case, seed)
    return dict(kind=kind, vis=vis, modes=modes, weights=weights, out=torch.empty(case["n"], device="cuda"))


def run(state):
    kind = state["kind"]
    if kind == "view":
        return state["fn"](state["map"], state["frags"], state["params"], out=state["out"])
    if kind == "plan":
        state["plan"].launch()
    elif kind == "noalloc":
        rb.batch_launch_noalloc(state["jobs"])
    elif kind == "serve":
        tickets = [state["engine"].submit_built(*b) for b in state["built"]]
        for t in tickets:
            state["engine"].wait(t)
    elif kind == "raster":
        rb.rbsm_rasterize(state["prims"], state["receiver"], state["w"], state["h"], out=state["out"])
    else:
        rb.rbsm_composite(state["vis"], state["modes"], state["weights"], out=state["out"])
    return state["out"]


# ---------------------------------------------------------------------------
# least work
# ---------------------------------------------------------------------------

def _view_work(n, map_w, map_h, out_bytes, radius=0):
    # every fragment read, every result written, every texel that the view meets read once (a camera sees about a
    # quarter of its map); a few operations per fragment, with a radius one test per texel and one term per offset
    texels = min(n, map_w * map_h // 4)
    ops = 12 * n if radius == 0 else n * ((2 * radius + 3) ** 2 + (2 * radius + 1) ** 2)
    return 12 * n + out_bytes * n + 4 * texels, ops


def work(case):
    kind = case["kind"]
    if kind == "view":
        n = case["view_w"] * case["view_h"]
        if case["flat"] and case["scene"] != "quad":
            n = int(n * 0.9 * 83 / 97)
        b, f = _view_work(n, case["map_w"], case["map_h"], 4 if case["entry"] == "rsmss" else 1, case["radius"])
        return dict(bytes=b, flops=f)
    if kind == "batch":
        views = BATCH_VIEWS[len(BATCH_VIEWS) - case["views"]:] if case["shrink"] > 1 else BATCH_VIEWS[:case["views"]]
        pixels = sum(int(w / case["shrink"]) * int(h / case["shrink"]) for w, h in views)
        n = 2.3 * pixels  # the cascades cover a view once, its two spot lights 0.65 of it each on average
        return dict(bytes=int(12 * n + pixels + 1.3 * pixels * 4 + n), flops=int(12 * n))
    if kind == "serve":
        views = [int(w / case["shrink"]) * int(h / case["shrink"]) for w, h in SERVE_VIEWS]
        n = sum(views[q % 3] for q in range(case["requests"]))
        return dict(bytes=int(n * (2.5 * (12 + 2.5) + 4 + 2.5)), flops=int(2.5 * 12 * n))
    if kind == "raster":
        n = case["map_w"] * case["map_h"]
        return dict(bytes=4 * n + 112 * case["tris"], flops=4 * n)
    n, lights = case["n"], case["lights"]
    return dict(bytes=int(n * (4 + 2.5 * lights)), flops=2 * n * lights)


# ---------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------

def _texel(m, i, j):
    h, w = m.shape
    return m[j.clamp(0, h - 1), i.clamp(0, w - 1)]


def _walk(m, i, j, zb, s, dx, dy, bits, max_dist):
    """Bounded traversal: +k where texel k ends the edge, -k where it leaves it, -(max_dist + 1) where it runs out."""
    a, b = ((0, 1), (0, -1)) if dx else ((-1, 0), (1, 0))
    chk_a, chk_b = (bits[2], bits[3]) if dx else (bits[0], bits[1])
    rd = torch.full_like(i, -(max_dist + 1))
    live = torch.arange(i.numel(), device=i.device)
    for k in range(1, max_dist + 1):
        li, lj, lz, ls = i[live] + k * dx, j[live] + k * dy, zb[live], s[live]
        end = (lz > _texel(m, li, lj)) == ls
        share = chk_a[live] & ((lz > _texel(m, li + a[0], lj + a[1])) == ls)
        share |= chk_b[live] & ((lz > _texel(m, li + b[0], lj + b[1])) == ls)
        rd[live] = torch.where(end, k, torch.where(share, rd[live], -k))
        live = live[~end & share]
        if live.numel() == 0:
            break
    return rd


def _axis(rn, rp, f):
    ends = (rn > 0).int() + (rp > 0).int()
    an, ap = rn.abs().double(), rp.abs().double()
    q = torch.where(rp > 0, ap - f, an - 1 + f) / (an + ap - 1)
    t = torch.where(ends == 1, q, torch.where(ends == 0, 1.0, 0.0))
    return ends, t


def _filtered(m, i, j, fx, fy, zb, max_dist):
    """RSMSS values (float64) of fragments in texels (i, j): tests and traversals as defined, then 64-bit arithmetic."""
    s = ~(zb > _texel(m, i, j))
    bits = [(zb > _texel(m, i + dx, j + dy)) == s for dx, dy in ((-1, 0), (1, 0), (0, 1), (0, -1))]
    v = s.double()
    e = torch.nonzero(bits[0] | bits[1] | bits[2] | bits[3]).flatten()
    if e.numel():
        ei, ej, ez, es, eb = i[e], j[e], zb[e], s[e], [b[e] for b in bits]
        rd = [_walk(m, ei, ej, ez, es, dx, dy, eb, max_dist) for dx, dy in ((-1, 0), (1, 0), (0, 1), (0, -1))]
        _, tx = _axis(rd[0], rd[1], fx[e])
        _, ty = _axis(rd[3], rd[2], fy[e])
        v[e] = torch.where(es, tx + ty, 1 - ty - tx).clamp(0.0, 1.0)
    return v


def _rsmss64(m, f, max_dist, radius=0):
    h, w = m.shape
    x, y = f[:, 0] * torch.tensor(float(w), device="cuda"), f[:, 1] * torch.tensor(float(h), device="cuda")
    i, j = torch.floor(x).long(), torch.floor(y).long()
    fx, fy = (x - torch.floor(x)).double(), (y - torch.floor(y)).double()
    zb = f[:, 2] - torch.tensor(BIAS, dtype=torch.float32, device="cuda")
    acc = torch.zeros(f.shape[0], dtype=torch.float64, device="cuda")
    for a in range(-radius, radius + 1):
        for b in range(-radius, radius + 1):
            acc += _filtered(m, i + a, j + b, fx, fy, zb, max_dist)
    return acc / (2 * radius + 1) ** 2


def _hard64(m, f, max_dist):
    """Hard visibility as 0.0 / 1.0 (decisions in binary32, as defined)."""
    h, w = m.shape
    x, y = f[:, 0] * torch.tensor(float(w), device="cuda"), f[:, 1] * torch.tensor(float(h), device="cuda")
    i, j = torch.floor(x).long(), torch.floor(y).long()
    fx, fy = x - torch.floor(x), y - torch.floor(y)
    zb = f[:, 2] - torch.tensor(BIAS, dtype=torch.float32, device="cuda")
    s = ~(zb > _texel(m, i, j))
    bits = [(zb > _texel(m, i + dx, j + dy)) == s for dx, dy in ((-1, 0), (1, 0), (0, 1), (0, -1))]
    v = s.double()
    e = torch.nonzero(s & (bits[0] | bits[1] | bits[2] | bits[3])).flatten()
    if e.numel():
        ei, ej, ez, es, eb = i[e], j[e], zb[e], s[e], [b[e] for b in bits]
        rd = [_walk(m, ei, ej, ez, es, dx, dy, eb, max_dist) for dx, dy in ((-1, 0), (1, 0), (0, 1), (0, -1))]
        nx, tx = _axis(rd[0], rd[1], fx[e].double())
        ny, ty = _axis(rd[3], rd[2], fy[e].double())
        tx, ty = tx.float(), ty.float()
        v[e] = ((nx != 2) & (ny != 2) & ~(ty < 1 - tx)).double()
    return v


def exact(case, seed):
    kind = case["kind"]
    if kind == "view":
        n = case["view_w"] * case["view_h"]
        if case["entry"] != "rsmss" or n * (2 * case["radius"] + 1) ** 2 > 1.7e9:
            return None
        m, f = _view_inputs(case, seed)
        return _rsmss64(m, f, case["max_dist"], case["radius"])
    if kind == "batch":
        return [_rsmss64(j["map"], j["frags"], j["params"].max_dist) if j["mode"] else None
                for j in _batch_jobs(case, seed)]
    if kind == "serve":
        maps, _, frags, reqs = _serve_inputs(case, seed)
        out = []
        for v, ls, modes in reqs:
            w = float(np.float32(1.0 / len(ls)))
            out.append(sum(w * (_rsmss64 if m else _hard64)(maps[l], frags[(l, v)], 16) for l, m in zip(ls, modes)))
        return out
    if kind == "raster":
        return _raster_scene(case, seed).map64()
    vis, _, weights = _composite_inputs(case, seed)
    return sum(w * v.double() for v, w in zip(vis, weights))
