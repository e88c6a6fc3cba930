"""Performance cases of the point rasterizer: the work its users have it do, through the public entry points.

A case is a plain dict (see `_case`); `prepare` makes what a program holds before the call (points, built clouds,
cameras, output buffers), `run` is one pass. Five operations:

  frame   pr_render + pr_resolve, once per camera (an interactive viewer; a stereo pair is two of them)
  views   pr_render_views over all cameras in one launch, then one pr_resolve each (VR pairs, camera arrays, the groups
          a render server forms)
  hqs     pr_render_hqs, once per camera (high-quality shading)
  lod     pr_render + pr_resolve over a layered (level-of-detail) cloud with node culling
  build   a cloud from positions and colours in device memory: load, order, boxes, Eq. 1 words

The clouds are synthetic: `terrain` is a square kilometre with relief, box buildings and poles, like an aerial scan
(`strips`: the points come tile by tile, as a scanner delivers them; otherwise in random order), `primitives` is eight
planes and spheres in a 100 m cube, one after the other. Every output is a whole number (keys, indices, packed words,
colours, the bits of boxes and positions) and has to stay the same bit for bit.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2204_01287_amd as pr

ORDERS = {"input": pr.PR_ORDER_INPUT, "morton": pr.PR_ORDER_MORTON, "spread": pr.PR_ORDER_MORTON_SPREAD}
CHUNK = 1 << 25  # points generated at a time
SIDE = 1000.0    # metres of a terrain's side


def _case(op, n, *, source="terrain", order="spread", batch=10240, camera="orbit", views=1, w=1920, h=1080, precision=0,
          lod_px=0.0, window=1.01, name=None):
    c = {"op": op, "n": n, "source": source, "order": order, "batch": batch, "camera": camera, "views": views, "w": w,
         "h": h, "precision": precision, "lod_px": lod_px, "window": window}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # a small scanned object in a small, odd-sized window: launches and latency
        _case("frame", 20011, source="primitives", order="input", camera="fixed", w=641, h=479, name="frame_20k"),
        # one million points as they come, 720p: the first thing a viewer is tried with
        _case("frame", 1_000_000, source="primitives", order="input", camera="fixed", w=1280, h=720, name="frame_1m"),
        # an aerial scan seen from around it, every batch in view, full HD
        _case("frame", 100_000_000, source="strips", name="orbit_100m"),
        # the same with full-precision coordinates (12 bytes a point), plain Morton order
        _case("frame", 100_000_000, source="strips", order="morton", precision=30, name="orbit_100m_30bit"),
        # a billion points from inside the scene: a stereo pair, one frame per eye
        _case("frame", 1_000_000_000, camera="stereo", views=2, w=2016, h=2240, name="stereo_1g"),
        # two billion points, both eyes of a headset in one launch
        _case("views", 2_000_000_000, camera="stereo", views=2, w=2016, h=2240, name="stereo_views_2g"),
        # a camera array over one cloud in one launch
        _case("views", 500_000_000, camera="aerial", views=64, w=1024, h=1024, name="array_64_500m"),
        # high-quality shading of one eye
        _case("hqs", 500_000_000, camera="stereo", views=1, w=2016, h=2240, name="hqs_500m"),
        # a layered cloud with the paper's 100-pixel node culling, a stereo pair
        _case("lod", 100_000_000, order="input", camera="stereo", views=2, w=2016, h=2240, lod_px=100.0, name="lod_100m"),
        # loading a small cloud in the order it has
        _case("build", 1_000_000, source="primitives", order="input", name="build_1m"),
        # loading an ordinary scan, sorted
        _case("build", 20_000_003, source="strips", name="build_20m"),
        # loading a large cloud whose points come in no order
        _case("build", 500_000_000, name="build_500m"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["frame", "frame", "frame", "views", "views", "hqs", "lod", "build", "build", "build"])
    order = rng.choice(["spread", "spread", "morton", "input"])
    source = "primitives" if order == "input" and rng.random() < 0.5 else rng.choice(["strips", "terrain"])
    if order == "input" and source == "terrain":
        source = "strips"  # batches of points in no order at all are nobody's layout
    batch = rng.choice([10240, 10240, 10240, 5120, 20480, 4 * rng.randint(300, 3000)])
    precision = rng.choice([0, 0, 0, 0, 0, 0, 10, 20, 30])
    w = _log(rng, 320, 3840)
    h = max(200, min(2240, int(w * rng.uniform(0.5, 1.1))))
    top = 5_000_000 if source == "primitives" else 200_000_000
    n = _log(rng, 20_000, top)
    if op == "build":
        return _case("build", _log(rng, 50_000, top), source=source, order=order, batch=batch)
    if op == "lod":
        return _case("lod", _log(rng, 200_000, 50_000_000), order="input", camera=rng.choice(["stereo", "orbit"]), w=w, h=h,
                     lod_px=rng.choice([0.0, 50.0, 100.0, 200.0]))
    if source == "primitives":
        camera = "fixed"
    else:
        camera = rng.choice(["orbit", "stereo", "aerial"])
    if op == "views":
        views = _log(rng, 1, 64) if camera == "aerial" else 2 if camera == "stereo" else rng.randint(1, 4)
        w, h = (w, h) if views <= 4 else (min(w, 1024), min(h, 1024))
        return _case("views", n, source=source, order=order, batch=batch, camera=camera, views=views, w=w, h=h,
                     precision=precision)
    if op == "hqs":
        return _case("hqs", n, source=source, order=order, batch=batch, camera=camera, w=w, h=h, precision=precision,
                     window=rng.choice([1.0, 1.01, 1.05]))
    return _case("frame", n, source=source, order=order, batch=batch, camera=camera, views=2 if camera == "stereo" else 1,
                 w=w, h=h, precision=precision)


# ------------------------------------------------------------------- points
def _colours(n, g):
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _primitives(n, g):
    """Eight planes and spheres in [0, 100]^3 metres with a centimetre of noise, one after the other."""
    xyz = torch.empty(n, 3, device="cuda")
    cut = [n * i // 8 for i in range(9)]
    for i in range(8):
        m = cut[i + 1] - cut[i]
        u = torch.rand(m, 3, generator=g, device="cuda")
        at = 20.0 + 60.0 * torch.rand(3, generator=g, device="cuda")
        if i % 2:
            d = torch.randn(m, 3, generator=g, device="cuda")
            p = at + (5.0 + 15.0 * float(u[0, 0])) * d / d.norm(dim=1, keepdim=True)
        else:
            axes = torch.linalg.qr(torch.randn(3, 3, generator=g, device="cuda"))[0]
            side = 20.0 + 60.0 * torch.rand(2, generator=g, device="cuda")
            p = at + (u[:, :1] - 0.5) * side[0] * axes[0] + (u[:, 1:2] - 0.5) * side[1] * axes[1]
        xyz[cut[i]:cut[i + 1]] = p.clamp_(0.0, 100.0)
    xyz += 0.01 * torch.randn(n, 3, generator=g, device="cuda")
    return xyz


def _relief(g):
    """A height map of the square kilometre at half a metre: five octaves of relief and 300 box buildings."""
    m = 2048
    z = torch.zeros(1, 1, m, m, device="cuda")
    for o in range(5):
        r = torch.randn(1, 1, 5 * 2 ** o, 5 * 2 ** o, generator=g, device="cuda")
        z += 15.0 * 0.5 ** o * torch.nn.functional.interpolate(r, size=(m, m), mode="bicubic", align_corners=True)
    z = z[0, 0]
    box = torch.rand(300, 5, generator=g, device="cuda").cpu().numpy()
    for bx, by, bw, bh, up in box:
        x0, y0, bw, bh = int(bx * (m - 90)), int(by * (m - 90)), int(16 + 64 * bw), int(16 + 64 * bh)
        z[y0:y0 + bh, x0:x0 + bw] = z[y0, x0] + 5.0 + 55.0 * float(up)
    return z.contiguous()


def _terrain(n, g, strips):
    """Points over the relief: mostly surface, some walls and plants above it, 4 % on 5,000 poles; a centimetre of
    noise. strips: tile after 10 m tile in serpentine order."""
    z = _relief(g)
    m = z.shape[0]
    poles = torch.rand(5000, 2, generator=g, device="cuda") * SIDE
    xyz = torch.empty(n, 3, device="cuda")
    for lo in range(0, n, CHUNK):
        k = min(CHUNK, n - lo)
        u = torch.rand(4, k, generator=g, device="cuda")
        if strips:
            t = (torch.arange(lo, lo + k, device="cuda", dtype=torch.int64) * 10000).div_(n, rounding_mode="floor")
            row, col = t // 100, t % 100
            col = torch.where(row % 2 == 0, col, 99 - col)
            x, y = (col + u[0]) * 10.0, (row + u[1]) * 10.0
        else:
            x, y = u[0] * SIDE, u[1] * SIDE
            at = (u[3] * 25.0 * 5000).to(torch.int64).clamp_(max=4999)
            pole = u[3] < 0.04
            x = torch.where(pole, poles[at, 0] + 0.1 * u[1], x)
            y = torch.where(pole, poles[at, 1] + 0.1 * u[0], y)
        fx, fy = x * ((m - 1) / SIDE), y * ((m - 1) / SIDE)
        ix, iy = fx.to(torch.int64).clamp_(0, m - 2), fy.to(torch.int64).clamp_(0, m - 2)
        fx, fy = fx - ix, fy - iy
        at = iy * m + ix
        f = z.view(-1)
        ground = torch.lerp(torch.lerp(f[at], f[at + 1], fx), torch.lerp(f[at + m], f[at + m + 1], fx), fy)
        up = torch.where(u[3] < 0.1, 12.0 * u[2], torch.zeros_like(x))
        out = xyz[lo:lo + k]
        out[:, 0], out[:, 1], out[:, 2] = x, y, ground + up
        out += 0.01 * torch.randn(k, 3, generator=g, device="cuda")
    return xyz


def _points(case, g):
    n = case["n"]
    xyz = _primitives(n, g) if case["source"] == "primitives" else _terrain(n, g, case["source"] == "strips")
    return xyz, _colours(n, g)


def _spread_bits(q):
    for s, mask in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F), (4, 0x10C30C30C30C30C3),
                    (2, 0x1249249249249249)):
        q = (q | (q << s)) & mask
    return q


def _layers(xyz, rgba, g, cap=10240):
    """A layered point cloud: every point on one level of the octree (four times the points per level), the nodes level
    by level, each cut into batches of at most cap points that start at multiples of four."""
    n = xyz.shape[0]
    depth = 0
    while depth < 15 and 0.75 * n / 4 ** depth > cap:
        depth += 1
    weight = torch.tensor([4.0 ** i for i in range(depth + 1)], dtype=torch.float64)
    edge = (weight.cumsum(0) / weight.sum()).to("cuda", torch.float32)
    level = torch.bucketize(torch.rand(n, generator=g, device="cuda"), edge).clamp_(max=depth)
    lo, hi = xyz.min(0).values, xyz.max(0).values
    size = float((hi - lo).max())
    cell = ((xyz - lo) * (2 ** depth / size)).to(torch.int64).clamp_(0, 2 ** depth - 1) >> (depth - level)[:, None]
    key = (level << 48) | _spread_bits(cell[:, 0]) | (_spread_bits(cell[:, 1]) << 1) | (_spread_bits(cell[:, 2]) << 2)
    key, by = torch.sort(key, stable=True)
    _, count = torch.unique_consecutive(key, return_counts=True)
    first = (count.cumsum(0) - count)
    head = by[first]
    where = torch.cat([lo.double() + cell[head].double() * (size / 2.0 ** level[head].double())[:, None],
                       (size / 2.0 ** level[head].double())[:, None], level[head].double()[:, None]], dim=1).cpu().numpy()
    count, first = count.cpu().numpy(), first.cpu().numpy()
    parts = (count + cap - 1) // cap
    node = np.repeat(np.arange(len(count)), parts)
    part = np.arange(len(node)) - np.repeat(np.cumsum(parts) - parts, parts)
    length = np.minimum(count[node] - part * cap, cap)
    room = (length + 3) // 4 * 4
    start = np.cumsum(room) - room
    spans = np.stack([start, length], axis=1).astype(np.uint32)
    rank = torch.arange(n, device="cuda")
    old = torch.from_numpy(first[node] + part * cap).cuda()
    to = rank + torch.repeat_interleave(torch.from_numpy(start).cuda() - old, torch.from_numpy(length).cuda())
    total = int(room.sum())
    xyz_out, rgba_out = torch.zeros(total, 3, device="cuda"), torch.zeros(total, dtype=torch.int32, device="cuda")
    xyz_out[to], rgba_out[to] = xyz[by], rgba[by]
    return xyz_out, rgba_out, spans, where[node]


# ------------------------------------------------------------------ cameras
def _look(eye, target, fovy, w, h, near, far):
    eye, target = np.asarray(eye, float), np.asarray(target, float)
    f = (target - eye) / np.linalg.norm(target - eye)
    s = np.cross(f, (0.0, 0.0, 1.0))
    s /= np.linalg.norm(s)
    u = np.cross(s, f)
    v = np.eye(4)
    v[0, :3], v[1, :3], v[2, :3] = s, u, -f
    v[:3, 3] = -s @ eye, -u @ eye, f @ eye
    p = np.zeros((4, 4))
    c = 1.0 / math.tan(math.radians(fovy) / 2.0)
    p[0, 0], p[1, 1], p[2, 2], p[2, 3], p[3, 2] = c * h / w, c, (far + near) / (near - far), 2 * far * near / (near - far), -1.0
    return v.astype(np.float32), p.astype(np.float32)


def _cameras(case, seed):
    rng = np.random.default_rng(seed)
    w, h, out = case["w"], case["h"], []
    if case["camera"] == "fixed":
        return [_look((50 + rng.uniform(-5, 5), -90.0, 120.0), (50, 50, 50), 60.0, w, h, 0.5, 1000.0)]
    if case["camera"] == "orbit":
        for _ in range(case["views"]):
            a = rng.uniform(0.0, 2.0 * math.pi)
            out.append(_look((500 + 800 * math.cos(a), 500 + 800 * math.sin(a), 450.0), (500, 500, 0), 60.0, w, h, 0.5, 5000.0))
    elif case["camera"] == "stereo":
        at = np.array([500.0 + rng.uniform(-5, 5), 500.0 + rng.uniform(-5, 5), 70.0])
        ahead = np.array([math.cos(math.radians(-15.0)), 0.0, math.sin(math.radians(-15.0))])
        for s in (-0.032, 0.032)[:case["views"]]:
            eye = at + np.array([0.0, -s, 0.0])
            out.append(_look(eye, eye + ahead, 100.0, w, h, 0.05, 3000.0))
    else:
        for _ in range(case["views"]):
            yaw, pitch = rng.uniform(0.0, 2.0 * math.pi), math.radians(rng.uniform(-60.0, -10.0))
            eye = np.array([rng.uniform(0, SIDE), rng.uniform(0, SIDE), rng.uniform(50.0, 430.0)])
            out.append(_look(eye, eye + [math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)],
                             60.0, w, h, 0.5, 5000.0))
    return out


# --------------------------------------------------------------------- pass
class _State:
    pass


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    s = _State()
    s.case, s.op = case, case["op"]
    s.ctx = pr.Context(0)
    xyz, rgba = _points(case, g)
    if s.op == "build":
        s.xyz, s.rgba = xyz, rgba
        return s
    if s.op == "lod":
        xyz, rgba, spans, nodes = _layers(xyz, rgba, g)
        s.cloud = pr.DeviceCloud(s.ctx, xyz, rgba, spans=spans, nodes=nodes)
    else:
        s.cloud = pr.DeviceCloud(s.ctx, xyz, rgba, case["batch"], ORDERS[case["order"]])
    del xyz, rgba
    w, h = case["w"], case["h"]
    cams = _cameras(case, seed)
    room = (w * h + 3) // 4 * 4  # every view's buffers start at a multiple of 16 bytes
    s.vb = torch.zeros(len(cams), room, dtype=torch.int64, device="cuda")
    s.fb = torch.zeros(len(cams), room, dtype=torch.int32, device="cuda")
    s.views = [(v, p, w, h, s.vb[i]) for i, (v, p) in enumerate(cams)]
    s.out = {"keys": s.vb[:, :w * h], "colours": s.fb[:, :w * h]}
    s.opts = pr.RenderOpts.make(precision=case["precision"], lod_px=case["lod_px"])
    if s.op == "views":
        s.cloud.drop_load_buffers()
        s.work_bytes = pr.pr_views_work_bytes(s.cloud.handle, len(cams))
        s.work = torch.empty(s.work_bytes, dtype=torch.uint8, device="cuda")
    if s.op == "hqs":
        s.sums = torch.zeros(len(cams), 2 * room, dtype=torch.int64, device="cuda")
        s.out["sums"] = s.sums[:, :2 * w * h]
    return s


def run(s):
    if s.op == "build":
        c = pr.DeviceCloud(s.ctx, s.xyz, s.rgba, s.case["batch"], ORDERS[s.case["order"]])
        out = {f: c.view(f, torch.int32, c.n) for f in ("low", "med", "high", "colors", "perm")}
        out["positions"], out["batches"] = c.view("xyz", torch.int32, 3 * c.n), c.view("batches", torch.int32, 8 * c.nb)
        return out
    ctx, cloud = s.ctx.handle, s.cloud.handle
    if s.op == "views":
        pr.pr_render_views(ctx, cloud, s.views, s.opts, s.work, s.work_bytes)
    for i, (v, p, w, h, vb) in enumerate(s.views):
        if s.op == "hqs":
            pr.pr_render_hqs(ctx, cloud, v, p, w, h, s.opts, s.case["window"], vb, s.sums[i], 0xFF000000, s.fb[i])
            continue
        if s.op != "views":
            pr.pr_render(ctx, cloud, v, p, w, h, s.opts, vb)
        pr.pr_resolve(ctx, cloud, vb, w, h, 0xFF000000, s.fb[i])
    return s.out


def work(case):
    """Bytes and operations of one pass. A frame reads the words of the points in view (4, 8 or 12 bytes each) and every
    batch record once, writes each pixel's key and colour and reads a colour a pixel; a build reads positions and colours
    and writes positions, colours, permutation, words and batch records. 20 operations a point and view: unpack and
    convert 6, project 9, floor 2, bounds 2, compare 1."""
    n, op, batches = case["n"], case["op"], -(-case["n"] // case["batch"])
    if op == "build":
        sorted_ = case["order"] != "input"
        return {"bytes": 16 * n + 20 * n + (12 * n if sorted_ else 0) + 32 * batches, "flops": 15 * n}
    views = case["views"]
    # share of the points in view, as these cameras see the terrain
    seen = {"fixed": 1.0, "orbit": 0.97, "stereo": 0.28, "aerial": 0.14}[case["camera"]]
    if op == "lod":
        seen *= 0.06 if case["lod_px"] else 1.0
    once = min(1.0, seen * (1 if case["camera"] == "stereo" else views)) if op == "views" else seen * views
    words = 4 * max(1, case["precision"] // 10)
    pixels = case["w"] * case["h"] * views
    moved = words * once * n + 32 * batches + 24 * pixels
    if op == "hqs":
        moved += (words + 4) * seen * views * n + 32 * pixels
    return {"bytes": moved, "flops": 20.0 * seen * views * n * (2 if op == "hqs" else 1)}


def exact(case, seed):
    """Every output is a whole number that has to be equal bit for bit: there is nothing that 64 bits would say better."""
    return None
