"""Performance cases of the radar-scan library, through its Python entry points.

Each case is the work a program has this library do: polar images of resident
scenes one at a time, as a batch, as a replayed graph or through the scan
server; the image epilogue; frames of a moving scene (refit, then scan); and
a rebuild of the tree on the GPU.  The scenes are the synthetic ones of
``workloads`` (a 60-triangle room, a 200 k-triangle urban block, a
2 M-triangle city).  Meshes and their trees stay resident for the life of the
process, as they do in a simulator; poses, ray seeds, vertex positions and
images come from a case's seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2310_03505_amd as R
import workloads as W

NOISE = dict(blur_sigma_bins=2.0, uniform_amp=1e-7, perlin_amp=1e-6, perlin_cell_az=16.0,
             perlin_cell_bins=64.0)


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: a cheap sensor in a room, one image per control step
        dict(name="room_scan", kind="scan", scene="room", mode="single", scans=1, azimuths=400, rays=64,
             bounces=3, bins=1024, beam_deg=2.0, air=False, cook_torrance=False),
        # 64 poses of the room replayed as a captured graph (many small robots)
        dict(name="room_graph_64", kind="scan", scene="room", mode="graph", scans=64, azimuths=400, rays=64,
             bounces=3, bins=1024, beam_deg=2.0, air=False, cook_torrance=False),
        # an ordinary scan: street scene at a navigation radar's resolution
        dict(name="urban_scan", kind="scan", scene="urban", mode="single", scans=1, azimuths=400, rays=1024,
             bounces=4, bins=3776, beam_deg=2.0, air=False, cook_torrance=False),
        # the same with multipath returns along the air path
        dict(name="urban_air", kind="scan", scene="urban", mode="single", scans=1, azimuths=400, rays=1024,
             bounces=4, bins=3776, beam_deg=2.0, air=True, cook_torrance=False),
        # microfacet materials, and the 8-bit image with noise from the same call
        dict(name="urban_post", kind="scan", scene="urban", mode="post", scans=1, azimuths=400, rays=1024,
             bounces=4, bins=3776, beam_deg=2.0, air=False, cook_torrance=True),
        # twelve requests of mixed shape through the continuous-batching server
        dict(name="urban_server", kind="scan", scene="urban", mode="server", scans=12, azimuths=331, rays=555,
             bounces=4, bins=3776, beam_deg=2.0, air=False, cook_torrance=False),
        # the largest single image: two million triangles, five interactions
        dict(name="city_scan", kind="scan", scene="city", mode="single", scans=1, azimuths=400, rays=4096,
             bounces=5, bins=3776, beam_deg=2.0, air=False, cook_torrance=False),
        # few rays per azimuth in a wide cone: the real-time setting on the same mesh
        dict(name="city_realtime", kind="scan", scene="city", mode="single", scans=1, azimuths=400, rays=200,
             bounces=4, bins=3776, beam_deg=10.0, air=False, cook_torrance=False),
        # a stretch of trajectory, the poses traced together; shapes vary
        dict(name="city_batch", kind="scan", scene="city", mode="batch", scans=6, azimuths=267, rays=777,
             bounces=5, bins=3776, beam_deg=2.0, air=False, cook_torrance=False),
        # the epilogue of a stored set of images, all noise terms on
        dict(name="post_64", kind="post", images=64, azimuths=400, bins=3776, sigma=2.0, uniform=True,
             perlin=True, db=True),
        # one frame of a scene whose objects move: refit, then a quick scan
        dict(name="city_frame", kind="frame", scene="city", builder="gpu", azimuths=100, rays=64, bounces=2,
             bins=3776),
        # a new mesh: the tree built on the GPU from the host copy, then a quick scan
        dict(name="city_build", kind="build", scene="city", azimuths=100, rays=64, bounces=2, bins=3776),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choices(["scan", "post", "frame", "build"], [8, 3, 1, 1])[0]
    if kind == "post":
        az, bins = _log_int(rng, 1, 800), _log_int(rng, 17, 5000)
        n = max(1, min(_log_int(rng, 1, 64), 96_000_000 // (az * bins)))
        return dict(kind="post", images=n, azimuths=az, bins=bins,
                    sigma=rng.choice([0.0, 0.5, 1.3, 2.0, 4.0, 8.0]), uniform=rng.random() < 0.7,
                    perlin=rng.random() < 0.7, db=rng.random() < 0.7)
    if kind != "scan":
        scene = rng.choice(["room", "urban", "city"])
        c = dict(kind=kind, scene=scene, azimuths=_log_int(rng, 16, 400), rays=_log_int(rng, 8, 128),
                 bounces=rng.randint(1, 3), bins=1024 if scene == "room" else 3776)
        if kind == "frame":
            c["builder"] = rng.choice(["gpu", "host"]) if scene != "city" else "gpu"
        return c
    scene = rng.choice(["room", "urban", "urban", "city"])
    mode = rng.choice(["single", "single", "post", "batch", "graph", "server"])
    scans = 1 if mode in ("single", "post") else _log_int(rng, 2, 64 if scene == "room" else 12)
    azimuths = _log_int(rng, 16, 800)
    bounces = rng.randint(1, 5)
    top = 64 if scene == "room" else 4096
    # at most half the listed largest scan's primaries in one case
    rays = _log_int(rng, 1 if scene == "room" else 16, top)
    rays = max(1, min(rays, 800_000 // (azimuths * scans)))
    return dict(kind="scan", scene=scene, mode=mode, scans=scans, azimuths=azimuths, rays=rays, bounces=bounces,
                bins=rng.choice([257, 1024]) if scene == "room" else rng.choice([1001, 2048, 3776]),
                beam_deg=rng.choice([2.0, 2.0, 10.0]), air=rng.random() < 0.2, cook_torrance=rng.random() < 0.2)


# ------------------------------------------------------------------ resident scenes
_meshes: dict = {}
_resident: dict = {}


def _mesh(name):
    if name not in _meshes:
        _meshes[name] = dict(room=W.tiny_room, urban=W.urban_block, city=W.large_scene)[name]()
    return _meshes[name]


class _Resident:
    """A context and a scene with the default tree, kept by the program."""

    def __init__(self, name):
        m = _mesh(name)
        self.ctx = R.Context(0)
        self.scene = R.Scene(self.ctx, m.vertices, m.indices, m.tri_material)


def _scene(name, role=""):
    if (name, role) not in _resident:
        _resident[name, role] = _Resident(name)
    return _resident[name, role]


class _Own(R.Scene):
    """A scene that lives as long as the state that holds it."""

    def __del__(self):
        torch.cuda.synchronize()
        self.release()


class _Graph:
    def __init__(self, res, scans, materials, images):
        self.handle, _ = R.rr_graph_create(res.ctx.handle, res.scene.handle, scans, materials, images)

    def __del__(self):
        R.rr_graph_destroy(self.handle)


class _Server:
    """A server owns its context; one per scene and material table."""

    def __init__(self, name, materials):
        self.res = _scene(name, "server")
        self.handle = R.rr_server_create(self.res.ctx.handle, self.res.scene.handle, materials)


_servers: dict = {}


def _materials(c):
    m = _mesh(c["scene"])
    if c.get("cook_torrance"):
        return [W.material_cook_torrance(0.2, 0.5, 100.0, 0.1) for _ in m.materials]
    return m.materials


def _scans(c, seed):
    """The case's (pose, params) list; with several scans their azimuth and ray counts vary
    around the case's, except in a graph, whose scans share the sensor."""
    rng = np.random.default_rng(seed)
    n = c.get("scans", 1)
    if c["scene"] == "room":
        poses = [p for p, _ in W.room_poses(_mesh("room"), seed=seed, n_poses=n)]
    else:
        tiles = 3 if c["scene"] == "city" else 1
        pts = W.street_points(rng, n, tiles)
        poses = [W.yaw_pose(p, rng.uniform(-math.pi, math.pi)) for p in pts]
    flags = W.FLAG_BEAM_GAIN | (W.FLAG_AIR_PATH if c.get("air") else 0)
    # the shapes are the case's own: the same for every seed
    vary = c.get("mode") in ("batch", "server")
    shape = random.Random(17)
    out = []
    for i, pose in enumerate(poses):
        f = (shape.uniform(0.5, 1.5), shape.uniform(0.5, 1.5)) if vary else (1.0, 1.0)
        out.append((pose, W.sensor_params(max(1, round(c["azimuths"] * f[0])), max(1, round(c["rays"] * f[1])),
                                          c["bounces"], c["bins"], beam_width_deg=c.get("beam_deg", 2.0),
                                          seed=int(rng.integers(1, 1 << 40)), scan_id=i, flags=flags)))
    return out


def _images(scans):
    return [torch.empty((p["n_azimuth"], p["n_bins"]), dtype=torch.float32, device="cuda") for _, p in scans]


# ------------------------------------------------------------------ prepare and run
def prepare(case, seed):
    c = case
    if c["kind"] == "post":
        return dict(c=c, ctx=_scene("room").ctx, images=_polar_images(c, seed), post=_post(c, seed))
    scans, mats = _scans(c, seed), _materials(c)
    s = dict(c=c, scans=scans, mats=mats)
    if c["kind"] in ("frame", "build"):
        m = _mesh(c["scene"])
        moved = _moved(m.vertices, seed)
        s["ctx"] = _scene("room").ctx
        if c["kind"] == "build":
            s["scene"] = _Own(s["ctx"], moved, m.indices, m.tri_material, build=False)
        else:
            opts = dict(builder=1) if c["builder"] == "gpu" else dict(spatial_pct=-1)
            s["scene"] = _Own(s["ctx"], m.vertices, m.indices, m.tri_material, **opts)
            s["vertices"] = torch.from_numpy(moved).cuda()
        s["images"] = _images(scans)
        return s
    if c["mode"] == "server":
        key = (c["scene"], bool(c["cook_torrance"]))
        if _servers and key not in _servers:  # one server at a time
            for k in list(_servers):
                R.rr_server_destroy(_servers.pop(k).handle)
        if key not in _servers:
            _servers[key] = _Server(c["scene"], mats)
        s["server"] = _servers[key]
        s["images"] = _images(scans)
        return s
    s["res"] = res = _scene(c["scene"])
    if c["mode"] == "graph":
        p = scans[0][1]
        s["stack"] = torch.empty((len(scans), p["n_azimuth"], p["n_bins"]), dtype=torch.float32, device="cuda")
        s["images"] = list(s["stack"])
        s["graph"] = _Graph(res, scans, mats, s["images"])
    elif c["mode"] == "post":
        p = scans[0][1]
        s["post"] = dict(NOISE, seed=seed)
        s["images"] = _images(scans)
        s["db"] = torch.empty((p["n_azimuth"], p["n_bins"]), dtype=torch.float32, device="cuda")
        s["u8"] = torch.empty((p["n_azimuth"], p["n_bins"]), dtype=torch.uint8, device="cuda")
    else:
        s["images"] = _images(scans)
    return s


def run(s):
    c = s["c"]
    if c["kind"] == "post":
        return list(R.rr_postprocess(s["ctx"].handle, s["images"], s["post"], want_db=c["db"]))
    if c["kind"] in ("frame", "build"):
        (pose, prm), ctx, scene, img = s["scans"][0], s["ctx"].handle, s["scene"], s["images"][0]
        if c["kind"] == "frame":
            scene.refit(s["vertices"])
            return R.scan(scene, pose, prm, s["mats"], image=img)
        R.rr_bvh_build(ctx, scene.handle, builder=1)
        # with the statistics the call waits: the next build replaces the tree
        _, st = R.rr_radar_scan(ctx, scene.handle, pose, prm, s["mats"], image=img, stats=True)
        return [img, st["segments"]]
    if c["mode"] == "server":
        srv = s["server"].handle
        tickets = [R.rr_server_submit(srv, pose, prm, img) for (pose, prm), img in zip(s["scans"], s["images"])]
        for t in tickets:
            R.rr_server_wait(srv, t)
        return s["images"]
    ctx, scene = s["res"].ctx.handle, s["res"].scene
    if c["mode"] == "graph":
        R.rr_graph_launch(s["graph"].handle, s["scans"], s["images"])
        return s["stack"]
    if c["mode"] == "batch":
        return R.rr_radar_scan_batch(ctx, scene.handle, s["scans"], s["mats"], images=s["images"])[0]
    pose, prm = s["scans"][0]
    if c["mode"] == "post":
        return list(R.rr_radar_scan_post(ctx, scene.handle, pose, prm, s["mats"], s["post"], image=s["images"][0],
                                         db=s["db"], u8=s["u8"])[:3])
    return R.scan(scene, pose, prm, s["mats"], image=s["images"][0])


def _post(c, seed):
    return dict(blur_sigma_bins=c["sigma"], uniform_amp=1e-7 if c["uniform"] else 0.0,
                perlin_amp=1e-6 if c["perlin"] else 0.0, perlin_cell_az=16.0, perlin_cell_bins=64.0,
                seed=seed, scan_id=3)


def _moved(vertices, seed):
    """The mesh with a smooth seeded displacement of up to a decimetre."""
    rng = np.random.default_rng(seed)
    k, ph = rng.uniform(0.02, 0.2, (3, 3)), rng.uniform(0, 2 * math.pi, 3)
    d = np.sin(vertices.astype(np.float32) @ k.T.astype(np.float32) + ph.astype(np.float32))
    return np.ascontiguousarray(vertices + np.float32(0.1) * d, dtype=np.float32)


def _polar_images(c, seed):
    """Polar images with the values of radar scans: a few clusters of returns per azimuth
    with energies log-uniform over 1e-8..1, sparse weak returns, zeros elsewhere, rare
    values above 1 (the recipe of workloads.polar_images, made on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    n, az, nb = c["images"], c["azimuths"], c["bins"]
    img = torch.zeros((n * az, nb), dtype=torch.float32, device="cuda")

    def u(*shape):
        return torch.rand(shape, generator=g, device="cuda")

    rows = torch.arange(n * az, device="cuda")[:, None].expand(-1, 11)
    for k in range(6):
        keep = (u(n * az, 1) < (6 - k) / 7.0).float()
        centre = (u(n * az, 1) * nb).long()
        width = 1 + (u(n * az, 1) * 5).long()
        off = torch.arange(-5, 6, device="cuda")[None, :]
        peak = 10.0 ** (-8.0 * u(n * az, 1)) * keep
        fall = torch.exp(-0.5 * (off / (width * 0.5).clamp(min=0.5)) ** 2) * (off.abs() <= width)
        col = centre + off
        ok = (col >= 0) & (col < nb)
        img.index_put_((rows[ok], col[ok]), (peak * fall)[ok])
    weak = u(n * az, nb)
    img += torch.where(weak < 0.02, 10.0 ** (-12.0 + 400.0 * weak), 0.0)
    hot = u(n * az, nb)
    img = torch.where(hot < 1e-4, 1.0 + 1e4 * hot, img)
    return img.view(n, az, nb)


# ------------------------------------------------------------------ work
# closest-hit queries per primary grow by about this factor per bounce level, and each visits this many
# nodes (76 flops a visit) and tests this many triangles (46 flops a test)
_GROWTH = dict(room=1.14, urban=1.83, city=1.83)
_VISITS = dict(room=(4.2, 2.0), urban=(22.7, 5.5), city=(23.4, 5.0))


def work(case):
    c = case
    if c["kind"] == "post":
        n = c["images"] * c["azimuths"] * c["bins"]
        taps = 2 * math.ceil(3 * c["sigma"]) + 1 if c["sigma"] else 0
        return dict(bytes=n * (4 + 1 + (4 if c["db"] else 0)),
                    flops=n * (2 * taps + 30 + 20 * c["uniform"] + 40 * c["perlin"]))
    m = _mesh(c["scene"])
    geometry = m.vertices.nbytes + m.indices.nbytes + m.tri_material.nbytes
    v, t = _VISITS[c["scene"]]
    n_bytes = flops = 0.0
    for _, p in _scans(c, 0):
        prim = p["n_azimuth"] * p["rays_per_beam"]
        seg = prim * sum(_GROWTH[c["scene"]] ** d for d in range(p["max_bounces"]))
        n_bytes += 4.0 * p["n_azimuth"] * p["n_bins"]
        flops += seg * (76.0 * v + 46.0 * t + 300.0)
    if c["kind"] in ("frame", "build"):
        n_bytes += geometry + 64.0 * 0.28 * m.n_tris + 64.0 * m.n_tris  # tree and leaf triangles written
    return dict(bytes=n_bytes, flops=flops)


# ------------------------------------------------------------------ the same in 64 bits
def exact(case, seed):
    c = case
    if c["kind"] == "post":
        imgs, post = _polar_images(c, seed), _post(c, seed)
        db = torch.empty(imgs.shape, dtype=torch.float64, device="cuda") if c["db"] else None
        if c["db"]:
            for i in range(c["images"]):
                db[i] = _epilogue64(imgs[i].double(), post, post["scan_id"] + i)
        return [db, None]
    if c["kind"] == "scan" and c["scene"] == "room" and not c["air"] and not c["cook_torrance"] and c["mode"] != "post":
        scans, mats, m = _scans(c, seed), _materials(c), _mesh("room")
        out = [_trace64(m, mats, pose, prm) for pose, prm in scans]
        return torch.stack(out) if c["mode"] == "graph" else out if c["mode"] in ("batch", "server") else out[0]
    return None  # brute force over a city mesh takes far too long


def _mul128(a, b):
    """(high, low) 64-bit words of a * b, int64 tensors holding unsigned words."""
    lo32 = 0xFFFFFFFF

    def split(x):
        return (x >> 32) & lo32, x & lo32

    a1, a0 = split(a)
    b1, b0 = split(b)
    p00, p01, p10, p11 = a0 * b0, a0 * b1, a1 * b0, a1 * b1
    mid = ((p00 >> 32) & lo32) + (p01 & lo32) + (p10 & lo32)
    high = p11 + ((p01 >> 32) & lo32) + ((p10 >> 32) & lo32) + ((mid >> 32) & lo32)
    return high, a * b


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _philox(seed, scan_id, c0, c1, c2, c3):
    """Philox4x64-10 (Salmon et al., SC'11) over int64 counter tensors."""
    x = [torch.as_tensor(v, dtype=torch.int64, device="cuda").expand(c0.shape) for v in (c0, c1, c2, c3)]
    m0 = torch.tensor(_signed(0xD2E7470EE14C6C93), device="cuda")
    m1 = torch.tensor(_signed(0xCA5A826395121157), device="cuda")
    k0, k1 = seed, scan_id
    for r in range(10):
        if r:
            k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
        h0, l0 = _mul128(m0, x[0])
        h1, l1 = _mul128(m1, x[2])
        x = [h1 ^ x[1] ^ _signed(k0), l1, h0 ^ x[3] ^ _signed(k1), l0]
    return x


def _u53(x):
    return ((x >> 11) & ((1 << 53) - 1)).double() * 2.0 ** -53


def _epilogue64(e, post, scan_id):
    """Range blur, uniform and gradient noise and dB of one float64 image [azimuth, bin]."""
    az, nb = e.shape
    sigma = float(np.float32(post["blur_sigma_bins"]))
    if sigma > 0:
        r = math.ceil(3 * sigma)
        w = [math.exp(-m * m / (2 * sigma * sigma)) for m in range(-r, r + 1)]
        pad = torch.nn.functional.pad(e, (r, r))
        e = sum(wm / sum(w) * pad[:, i:i + nb] for i, wm in enumerate(w))
    k = torch.arange(az, device="cuda")
    b = torch.arange(nb, device="cuda")
    if post["uniform_amp"] > 0:
        nq = (nb + 3) // 4
        kk, qq = torch.meshgrid(k, torch.arange(nq, device="cuda"), indexing="ij")
        words = torch.stack(_philox(post["seed"], scan_id, kk, qq, 1, 0), dim=-1).reshape(az, 4 * nq)[:, :nb]
        e = e + float(np.float32(post["uniform_amp"])) * _u53(words)
    if post["perlin_amp"] > 0:
        x = k.double() / post["perlin_cell_az"]
        y = b.double() / post["perlin_cell_bins"]
        i0, j0 = x.floor().long(), y.floor().long()
        li, lj = torch.meshgrid(torch.arange(int(i0[-1]) + 2, device="cuda"),
                                torch.arange(int(j0[-1]) + 2, device="cuda"), indexing="ij")
        g = (_philox(post["seed"], scan_id, li, lj, 2, 0)[0] >> 61) & 7
        vec = torch.tensor([[1, 1], [-1, 1], [1, -1], [-1, -1], [1, 0], [-1, 0], [0, 1], [0, -1]],
                           dtype=torch.float64, device="cuda")[g]
        fx, fy = (x - i0)[:, None], (y - j0)[None, :]

        def corner(di, dj):
            v = vec[i0 + di][:, j0 + dj]
            return v[..., 0] * (fx - di) + v[..., 1] * (fy - dj)

        def fade(t):
            return t * t * t * (t * (t * 6 - 15) + 10)

        nx0 = corner(0, 0) + fade(fx) * (corner(1, 0) - corner(0, 0))
        nx1 = corner(0, 1) + fade(fx) * (corner(1, 1) - corner(0, 1))
        e = e + float(np.float32(post["perlin_amp"])) * (0.5 + 0.5 * (nx0 + fade(fy) * (nx1 - nx0)))
    return 10.0 * torch.log10(e)


def _trace64(mesh, mats, pose, prm):
    """The polar image of a small mesh by brute force, one bounce level after another."""
    def d64(x):
        return torch.as_tensor(np.asarray(x, dtype=np.float64), device="cuda")

    tri = d64(mesh.vertices.astype(np.float32))[torch.from_numpy(mesh.indices.astype(np.int64)).cuda()]
    v0, e1, e2 = tri[:, 0], tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0]
    nrm = torch.nn.functional.normalize(torch.linalg.cross(e1, e2), dim=1)
    tmat = torch.from_numpy(mesh.tri_material.astype(np.int64)).cuda()
    b = float(np.float32(prm["beam_width_rad"]))
    f32 = np.float32
    kind = torch.tensor([m["kind"] for m in mats], device="cuda")
    idx = d64([f32(m["n"]) for m in mats])
    refl = d64([f32(m["reflectance"]) for m in mats])
    expo = d64([f32(m["C"]) for m in mats])
    wa, wb, ws = [], [], []
    for m in mats:
        a_, b_, c_ = float(f32(m["A"])), float(f32(m["B"])), float(f32(m["C"]))
        s_ = 1 - a_ - b_
        z = a_ * math.pi + 2 * b_ + s_ * math.sqrt(math.pi) * math.exp(math.lgamma((c_ + 1) / 2) - math.lgamma(c_ / 2 + 1))
        wa.append(a_ * b / z)
        wb.append(2 * b_ * math.sin(b / 2) / z)
        ws.append(s_ * b / z)
    wa, wb, ws = d64(wa), d64(wb), d64(ws)
    # primaries: a Gaussian cone around each azimuth
    na, ns, nb = prm["n_azimuth"], prm["rays_per_beam"], prm["n_bins"]
    kk, ii = torch.meshgrid(torch.arange(na, device="cuda"), torch.arange(ns, device="cuda"), indexing="ij")
    kk, ii = kk.reshape(-1), ii.reshape(-1)
    u = _philox(prm["seed"], prm["scan_id"], kk, ii, 0, 0)
    z = torch.sqrt(-2 * torch.log(_u53(u[0]) + 2.0 ** -53)) * torch.cos(2 * math.pi * _u53(u[1]))
    om = -math.pi + 2 * math.pi * _u53(u[2])
    p = torch.tensor(float(f32(prm["beam_prob"])), dtype=torch.float64)
    r = z * (b / 2 / (math.sqrt(2) * float(torch.special.erfinv(p))))
    phi, th = 2 * math.pi * kk.double() / na + r * torch.cos(om), r * torch.sin(om)
    ds = torch.stack([torch.cos(th) * torch.cos(phi), torch.cos(th) * torch.sin(phi), torch.sin(th)], dim=1)
    w, x, y, q = (float(f32(t)) for t in pose["quat_wxyz"])
    n = math.sqrt(w * w + x * x + y * y + q * q)
    w, x, y, q = w / n, x / n, y / n, q / n
    rot = d64([[1 - 2 * (y * y + q * q), 2 * (x * y - w * q), 2 * (x * q + w * y)],
               [2 * (x * y + w * q), 1 - 2 * (x * x + q * q), 2 * (y * q - w * x)],
               [2 * (x * q - w * y), 2 * (y * q + w * x), 1 - 2 * (x * x + y * y)]])
    d = torch.nn.functional.normalize(ds @ rot.T, dim=1)
    o = d64([f32(t) for t in pose["position"]]).expand_as(d)
    g = torch.exp(-0.5 * z * z) if prm["flags"] & 1 else torch.ones_like(z)
    E = torch.full_like(z, 1.0 / ns)
    L, col = torch.zeros_like(z), kk
    med = torch.full_like(kk, -1)
    ex = torch.full_like(kk, -1)
    img = torch.zeros(na * nb, dtype=torch.float64, device="cuda")
    dr, cut = float(f32(prm["bin_size_m"])), float(f32(prm["energy_cutoff"]))
    ids = torch.arange(len(v0), device="cuda")
    for depth in range(prm["max_bounces"]):
        if not len(o):
            break
        # Moller-Trumbore against every triangle
        pv = torch.linalg.cross(d[:, None], e2[None])
        det = (e1 * pv).sum(-1)
        inv = torch.where(det == 0, math.nan, 1 / det)
        sv = o[:, None] - v0
        bu = (sv * pv).sum(-1) * inv
        qv = torch.linalg.cross(sv, e1[None].expand_as(sv))
        bv = (d[:, None] * qv).sum(-1) * inv
        t = (e2 * qv).sum(-1) * inv
        ok = (bu >= 0) & (bv >= 0) & (bu + bv <= 1) & (t > 0) & (ids != ex[:, None])
        n_cur = torch.where(med < 0, 1.0, idx[med.clamp(min=0)])
        t, hit = torch.where(ok, t, math.inf).min(1)
        on = t <= (nb * dr - L) / n_cur
        o, d, g, E, L, col, med, n_cur, t, hit = (v[on] for v in (o, d, g, E, L, col, med, n_cur, t, hit))
        mat, nv = tmat[hit], nrm[hit]
        enter = (d * nv).sum(1) < 0
        nf = torch.where(enter[:, None], nv, -nv)
        ci = -(d * nf).sum(1)
        diel = kind[mat] == 0
        n2 = torch.where(enter, idx[mat], 1.0)
        eta = n_cur / n2
        k = 1 - eta ** 2 * (1 - ci ** 2)
        refr = diel & (k >= 0)
        ct = torch.sqrt(k.clamp(min=0))
        rs = (n_cur * ci - n2 * ct) / (n_cur * ci + n2 * ct)
        rp = (n2 * ci - n_cur * ct) / (n2 * ci + n_cur * ct)
        Rf = torch.where(diel, torch.where(refr, 0.5 * (rs ** 2 + rp ** 2), 1.0), refl[mat])
        cw = (2 * ci ** 2 - 1).clamp(min=0)
        wr = (wa[mat] + wb[mat] * cw + ws[mat] * cw ** expo[mat]).clamp(0, 1)
        e_ret = E * Rf * wr
        rng = L + n_cur * t
        bin_ = (rng / dr).long()
        inb = bin_ < nb
        img.index_add_(0, (col * nb + bin_)[inb], (e_ret * g)[inb])
        pt = o + t[:, None] * d
        rd = torch.nn.functional.normalize(d + 2 * ci[:, None] * nf, dim=1)
        td = torch.nn.functional.normalize(eta[:, None] * d + (eta * ci - ct)[:, None] * nf, dim=1)
        er, et = E * Rf - e_ret, torch.where(refr, E * (1 - Rf), 0.0)
        kr, kt = er > cut, et > cut
        tmed = torch.where(enter, mat, -1)
        o, d = torch.cat([pt[kr], pt[kt]]), torch.cat([rd[kr], td[kt]])
        E, L, g = torch.cat([er[kr], et[kt]]), torch.cat([rng[kr], rng[kt]]), torch.cat([g[kr], g[kt]])
        col, ex = torch.cat([col[kr], col[kt]]), torch.cat([hit[kr], hit[kt]])
        med = torch.cat([med[kr], tmed[kt]])
    return img.view(na, nb)
