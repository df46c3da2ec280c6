"""Performance cases of the renderer: the calls that a program which trains or
evaluates embodied agents makes, through the package's public entry points.

A case is a dict of plain values.  Its `kind` names the entry point:

  plain    Context.render_plain   frames of one scene, written to two tensors
  noalloc  Context.render_noalloc the same call on the library's static scratch
  render   Context.render         frames of one scene, any output set
  batch    Context.render_batch   one view per environment over several scenes
  stepper  Stepper.step           the same, captured once as a graph
  env      Context.actuate + Stepper.step_device: a whole environment step
  actuate  Context.actuate        agents moved against their scenes' obstacles
  free     Context.nav_free       free-space queries of one scene
  serve    Server.submit / wait   single-view requests from independent clients

Scenes are generated apartments: a grid of rooms with doorways and furniture
boxes, every surface tessellated to one cell size, the vertices displaced by
about a centimetre as in a scan.  Cameras stand 1.5 m high at free places of
the rooms and look level, with a 90 degree field of view unless the case says
otherwise.  A scene belongs to its case (a dataset's scene does not change
between runs); poses, agents, actions, query points and noise seeds come from
the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1904_01201_amd as hab

NEAR = 0.01
CAMERA_HEIGHT = 1.5
AGENT_RADIUS = 0.1
BODY_HEIGHTS = (0.1, 1.5)     # obstacles: the mesh cut just above the floor and at the agent's top
ROOM_HEIGHT = 2.8
ACTION_SETS = 16              # action tensors an environment loop cycles through

OUTPUTS = {"d": hab.OUT_DEPTH, "rgb": hab.OUT_RGB, "rgbd": hab.OUT_RGB | hab.OUT_DEPTH,
           "rgbds": hab.OUT_RGB | hab.OUT_DEPTH | hab.OUT_SEMANTIC,
           "rgbdt": hab.OUT_RGB | hab.OUT_DEPTH | hab.OUT_TRI}


def listed():
    return [
        # one agent in one small room, a frame at a time: the smallest call, all latency
        dict(name="room_frame_128", kind="plain", scenes=1, tri_lo=2_000, tri_hi=2_000, views=1,
             width=128, height=128, hfov=90.0, outputs="rgbd"),
        # one agent in a scanned apartment at the paper's sensor, a frame at a time
        dict(name="apartment_frame_256", kind="plain", scenes=1, tri_lo=200_000, tri_hi=200_000, views=1,
             width=256, height=256, hfov=90.0, outputs="rgbd"),
        # a depth-only robot sensor of an odd size inside a loop that must not allocate
        dict(name="depth_frame_noalloc", kind="noalloc", scenes=1, tri_lo=60_000, tri_hi=60_000, views=1,
             width=203, height=117, hfov=70.0, outputs="d"),
        # evaluation footage: a few larger frames of a detailed scene with the visible triangle
        dict(name="eval_frames_512", kind="render", scenes=1, tri_lo=1_000_000, tri_hi=1_000_000, views=8,
             width=512, height=384, hfov=90.0, outputs="rgbdt"),
        # a depth dataset rendered in bulk: many small frames of one coarse scene
        dict(name="dataset_depth_64", kind="render", scenes=1, tri_lo=20_000, tri_hi=20_000, views=1024,
             width=64, height=64, hfov=90.0, outputs="d"),
        # reinforcement learning: 64 environments over 4 scenes, the paper's sensor
        dict(name="batch64_4scenes_256", kind="batch", scenes=4, tri_lo=100_000, tri_hi=1_000_000, views=64,
             width=256, height=256, hfov=90.0, outputs="rgbd"),
        # every sensor at once: textured colour, noisy depth and the semantic mask
        dict(name="batch32_all_sensors_256", kind="batch", scenes=2, tri_lo=150_000, tri_hi=400_000, views=32,
             width=256, height=256, hfov=90.0, outputs="rgbds", textured=True, sigma=0.1),
        # a large mixed batch (128 / 256 / 512 px, depth / colour / both) as a captured step
        dict(name="stepper256_16scenes_mixed", kind="stepper", scenes=16, tri_lo=50_000, tri_hi=800_000, views=256,
             width=256, height=256, hfov=90.0, outputs="mixed"),
        # the whole environment step on the device: 64 agents move, 64 views are rendered
        dict(name="env_loop_64", kind="env", scenes=4, tri_lo=100_000, tri_hi=1_000_000, views=64,
             width=256, height=256, hfov=90.0, outputs="rgbd"),
        # agents moved in bulk against the rendered meshes (episode generation, blind agents)
        dict(name="actuate_65536", kind="actuate", scenes=4, tri_lo=100_000, tri_hi=1_000_000, views=65_536),
        # sampling start and goal positions: a map of a scene's free floor
        dict(name="free_space_1m", kind="free", scenes=1, tri_lo=500_000, tri_hi=500_000, views=1 << 20),
        # 64 independent clients' requests, mixed sensors, through the serving loop
        dict(name="serve_64_mixed", kind="serve", scenes=4, tri_lo=100_000, tri_hi=1_000_000, views=64,
             width=256, height=256, hfov=90.0, outputs="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "noalloc", "render", "batch", "stepper", "env", "actuate", "free", "serve"])
    if kind in ("actuate", "free"):
        c = dict(kind=kind, scenes=1 if kind == "free" else rng.randint(1, 4), tri_lo=_log_int(rng, 20_000, 200_000))
        c["tri_hi"] = c["tri_lo"] if kind == "free" else _log_int(rng, c["tri_lo"], 1_000_000)
        c["views"] = _log_int(rng, 64, 65_536 if kind == "actuate" else 1 << 20)
        return c
    if kind in ("plain", "noalloc", "render"):
        tri = _log_int(rng, 2_000, 300_000 if kind == "noalloc" else 1_000_000)
        w = _log_int(rng, 48, 256 if kind == "noalloc" else 512)
        h = max(32, int(w * rng.uniform(0.6, 1.1)))
        # as many frames as 4 Mpixel and 16 M triangle fetches hold (one frame on the static scratch)
        most = 1 if kind == "noalloc" else max(1, min(1024, (1 << 22) // (w * h), 16_000_000 // tri))
        return dict(kind=kind, scenes=1, tri_lo=tri, tri_hi=tri, views=_log_int(rng, 1, most), width=w, height=h,
                    hfov=round(rng.uniform(60.0, 100.0), 1),
                    outputs=rng.choice(["d", "rgb", "rgbd"] + (["rgbdt"] if kind == "render" else [])))
    scenes = rng.randint(1, 8)
    c = dict(kind=kind, scenes=scenes, tri_lo=_log_int(rng, 50_000, 200_000))
    c["tri_hi"] = _log_int(rng, c["tri_lo"], 800_000)
    c["views"] = max(scenes, _log_int(rng, 8, 128))
    c["width"] = _log_int(rng, 96, 256)
    c["height"] = max(64, int(c["width"] * rng.uniform(0.7, 1.0)))
    c["hfov"] = round(rng.uniform(70.0, 100.0), 1)
    c["outputs"] = "rgbd" if kind == "env" else rng.choice(["d", "rgbd", "mixed"])
    if kind == "batch" and rng.random() < 0.4:
        c.update(outputs="rgbds", textured=True, sigma=round(rng.uniform(0.01, 0.4), 3))
    return c


# ---------------------------------------------------------------- scenes
class _Mesh:
    """Host arrays of one scene, its free floor and its boxes."""


def _layout(tri, rng):
    """Rectangles (origin, u edge, v edge, instance) of the rooms, walls and boxes, and the rooms' extents."""
    rooms_x, rooms_z, per_room = (1, 1, 16) if tri < 10_000 else (2, 4, 24) if tri < 100_000 else (2, 4, 50)
    xs = np.concatenate([[0.0], np.cumsum(rng.uniform(3.5, 5.5, rooms_x))])
    zs = np.concatenate([[0.0], np.cumsum(rng.uniform(3.5, 5.5, rooms_z))])
    H, rects, rooms, boxes = ROOM_HEIGHT, [], [], []

    def rect(o, u, v, inst=None):
        rects.append((o, u, v, len(rects) if inst is None else inst))

    def wall(axis, at, lo, hi, door):
        spans = [(lo, hi, 0.0)]
        if door:
            d = float(rng.uniform(lo + 0.3, hi - 1.2))
            spans = [(lo, d, 0.0), (d + 0.9, hi, 0.0), (d, d + 0.9, 2.1)]
        for a, b, y in spans:
            if axis == 0:
                rect((at, y, a), (0.0, 0.0, b - a), (0.0, H - y, 0.0))
            else:
                rect((a, y, at), (b - a, 0.0, 0.0), (0.0, H - y, 0.0))

    for i in range(rooms_x):
        for k in range(rooms_z):
            x0, x1, z0, z1 = xs[i], xs[i + 1], zs[k], zs[k + 1]
            rooms.append((x0, z0, x1, z1))
            for y in (0.0, H):
                rect((x0, y, z0), (x1 - x0, 0.0, 0.0), (0.0, 0.0, z1 - z0))
            wall(0, x0, z0, z1, i > 0)
            wall(1, z0, x0, x1, k > 0)
            if i == rooms_x - 1:
                wall(0, x1, z0, z1, False)
            if k == rooms_z - 1:
                wall(1, z1, x0, x1, False)
    nstruct = len(rects)
    for r, (x0, z0, x1, z1) in enumerate(rooms):
        for _ in range(per_room):
            for _try in range(50):
                sx, sy, sz = rng.uniform(0.2, 1.2, 3)
                bx, bz = rng.uniform(x0 + 0.05, x1 - 0.05 - sx), rng.uniform(z0 + 0.05, z1 - 0.05 - sz)
                cx, cz = (x0 + x1) / 2, (z0 + z1) / 2
                if math.hypot(min(max(cx, bx), bx + sx) - cx, min(max(cz, bz), bz + sz) - cz) > 1.0:
                    break
            else:
                continue
            inst = nstruct + len(boxes)
            boxes.append((bx, bz, bx + sx, bz + sz))
            rect((bx, sy, bz), (sx, 0.0, 0.0), (0.0, 0.0, sz), inst)
            for at in (bx, bx + sx):
                rect((at, 0.0, bz), (0.0, 0.0, sz), (0.0, sy, 0.0), inst)
            for at in (bz, bz + sz):
                rect((bx, 0.0, at), (sx, 0.0, 0.0), (0.0, sy, 0.0), inst)
    return rects, rooms, boxes


@functools.lru_cache(maxsize=64)
def _mesh(tri, index, textured=False):
    """About `tri` triangles of apartment `index`."""
    rng = np.random.default_rng([tri, index, 1])
    rects, rooms, boxes = _layout(tri, rng)
    o, u, v = (np.array([r[k] for r in rects]) for k in range(3))
    lu, lv = np.abs(u).sum(1), np.abs(v).sum(1)
    cell = math.sqrt(2.0 * float((lu * lv).sum()) / tri)
    nu, nv = np.maximum(1, np.rint(lu / cell)).astype(np.int64), np.maximum(1, np.rint(lv / cell)).astype(np.int64)

    def spread(counts):
        own = np.repeat(np.arange(len(rects)), counts)
        return own, np.arange(own.size) - np.repeat(np.cumsum(counts) - counts, counts)

    own, at = spread((nu + 1) * (nv + 1))
    fi, fj = (at // (nv[own] + 1)) / nu[own], (at % (nv[own] + 1)) / nv[own]
    pos = o[own] + u[own] * fi[:, None] + v[own] * fj[:, None]
    # displacement by a hash of the place, so that coincident vertices move together
    q = np.rint(pos * 1e4) @ np.array([[12.9898, 39.3461, 73.1561], [78.2331, 11.1351, 52.2352], [37.7191, 83.1553, 9.1517]])
    wave = np.sin(q) * 43758.5453
    m = _Mesh()
    m.positions = (pos + ((wave - np.floor(wave)) - 0.5) * 0.03).astype(np.float32)
    base = rng.integers(32, 225, (len(rects), 3))
    m.colors = np.clip(base[own] + rng.integers(-31, 32, (own.size, 3)), 0, 255).astype(np.uint8)
    first = np.cumsum((nu + 1) * (nv + 1)) - (nu + 1) * (nv + 1)
    qown, qat = spread(nu * nv)
    a = first[qown] + (qat // nv[qown]) * (nv[qown] + 1) + qat % nv[qown]
    b = a + nv[qown] + 1
    m.indices = np.stack([a, b, b + 1, a, b + 1, a + 1], 1).reshape(-1, 3).astype(np.uint32)
    m.instances = np.repeat(np.array([r[3] for r in rects], np.uint32)[qown], 2)
    m.uvs = m.texture = None
    if textured:
        m.uvs = (rng.random((len(rects), 2))[own] + np.stack([fi * lu[own], fj * lv[own]], 1) / 4.0).astype(np.float32)
        n = 1024
        fine, coarse = rng.integers(-24, 25, (n, n, 3)), rng.integers(40, 216, (n // 32, n // 32, 3))
        m.texture = np.clip(np.kron(coarse, np.ones((32, 32, 1), np.int64)) + fine, 0, 255).astype(np.uint8)
    m.rooms, m.boxes = np.array(rooms), np.array(boxes).reshape(-1, 4)
    return m


def _meshes(case):
    """The case's scenes: triangle counts spread over [tri_lo, tri_hi] in their logarithm."""
    n = case["scenes"]
    tri = [int(case["tri_lo"] * (case["tri_hi"] / case["tri_lo"]) ** (k / max(1, n - 1))) for k in range(n)]
    return [_mesh(t, k, bool(case.get("textured"))) for k, t in enumerate(tri)]


def _free_states(mesh, n, rng):
    """x, z, yaw of n agents at free places of the rooms."""
    x, z = np.empty(0), np.empty(0)
    while x.size < n:
        r = mesh.rooms[rng.integers(0, len(mesh.rooms), 2 * n + 16)]
        px = rng.uniform(r[:, 0] + 0.3, r[:, 2] - 0.3)
        pz = rng.uniform(r[:, 1] + 0.3, r[:, 3] - 0.3)
        ok = np.ones(px.size, bool)
        for x0, z0, x1, z1 in mesh.boxes:
            ok &= (px < x0 - 0.2) | (px > x1 + 0.2) | (pz < z0 - 0.2) | (pz > z1 + 0.2)
        x, z = np.concatenate([x, px[ok]]), np.concatenate([z, pz[ok]])
    return x[:n], z[:n], rng.uniform(0.0, 2.0 * math.pi, n)


def _poses(x, z, yaw):
    c, s, o, i = np.cos(yaw), np.sin(yaw), np.zeros_like(yaw), np.ones_like(yaw)
    return np.stack([x, i * CAMERA_HEIGHT, z, c, o, s, o, i, o, -s, o, c], 1).astype(np.float32)


def _views(case, seed):
    """Scene and pose of every view: an equal share of the views per scene, in order."""
    meshes, rng = _meshes(case), np.random.default_rng([seed, 7])
    owner = np.arange(case["views"]) * len(meshes) // case["views"]
    states = [np.stack(_free_states(m, int((owner == k).sum()), rng), 1) for k, m in enumerate(meshes)]
    return meshes, owner, np.concatenate(states)


def _sensors(case):
    """(width, height, outputs) of every view."""
    n, w, h = case["views"], case["width"], case["height"]
    if case["outputs"] != "mixed":
        return [(w, h, case["outputs"])] * n
    sizes, outs = [(w // 2, h // 2), (w, h), (2 * w, 2 * h)], ["d", "rgb", "rgbd"]
    return [(*sizes[(k * 7 // 3) % 3], outs[(k * 5 // 7) % 3]) for k in range(n)]


# ---------------------------------------------------------------- the program's own state
class _State:
    """What a program keeps between calls; its library objects go with it."""

    def __init__(self):
        self.ctx = hab.Context(0)
        self.owned = []

    def __del__(self):
        torch.cuda.synchronize()
        for o in self.owned:
            o.close()
        self.ctx.close()


def _start_states(s, meshes, owner, states, rng):
    """Agents on the device, their obstacle sets and the action tensors of the coming steps."""
    navs = [s.ctx.nav_from_scene(h, BODY_HEIGHTS) for h in s.handles]
    s.nav_of = s.ctx.nav_array([navs[k] for k in owner])
    x, z, yaw = states.T
    s.agents = torch.from_numpy(np.stack([x, z, -np.sin(yaw), -np.cos(yaw)], 1)).cuda()
    n = len(owner)
    s.actions = torch.from_numpy(rng.choice([1, 1, 2, 3], (ACTION_SETS, n)).astype(np.uint8)).cuda()
    s.collided = torch.empty(n, dtype=torch.uint8, device="cuda")
    s.poses = torch.empty((n, 12), dtype=torch.float32, device="cuda")
    s.params, s.step = s.ctx.actuation(), 0


def prepare(case, seed):
    kind = case["kind"]
    s = _State()
    s.kind = kind
    meshes, owner, states = _views(case, seed) if kind != "free" else (_meshes(case), None, None)
    rng = np.random.default_rng([seed, 8])
    s.handles = [s.ctx.upload_scene(m) for m in meshes]
    if kind == "free":
        s.nav = s.ctx.nav_from_scene(s.handles[0], BODY_HEIGHTS)
        lo, hi = meshes[0].positions.min(0), meshes[0].positions.max(0)
        s.points = torch.from_numpy(np.stack([rng.uniform(lo[0], hi[0], case["views"]),
                                              rng.uniform(lo[2], hi[2], case["views"])], 1)).cuda()
        s.out = torch.empty(case["views"], dtype=torch.uint8, device="cuda")
        return s
    if kind == "actuate":
        _start_states(s, meshes, owner, states, rng)
        return s
    s.host_poses = _poses(*states.T)
    specs = _sensors(case)
    # one tensor per output of each kind of sensor, one slice of it per view
    s.out, s.slices, made = {}, [None] * len(specs), {}
    for spec in sorted(set(specs)):
        made[spec] = s.ctx.sensor(spec[0], spec[1], case["hfov"], NEAR, OUTPUTS[spec[2]], case.get("sigma", 0.0))
        at = [k for k, x in enumerate(specs) if x == spec]
        tensors = s.ctx.alloc(made[spec], len(at))
        s.out["%dx%d_%s" % spec] = tensors
        for i, k in enumerate(at):
            s.slices[k] = {name: t[i] for name, t in tensors.items()}
    s.sensors = [made[spec] for spec in specs]
    seeds = rng.integers(0, 1 << 31, len(specs))
    items = [(s.handles[owner[k]], s.sensors[k], s.host_poses[k], *[s.slices[k].get(n) for n in ("rgb", "depth", "tri", "semantic")],
              int(seeds[k])) for k in range(len(specs))]
    if kind in ("batch", "stepper", "env"):
        s.ctx.autotune(items)
    if kind == "batch":
        s.views = s.ctx.make_views(items)
    elif kind in ("stepper", "env"):
        s.stepper = s.ctx.stepper(items)
        s.owned.append(s.stepper)
        if kind == "env":
            _start_states(s, meshes, owner, states, rng)
    elif kind == "serve":
        s.server = hab.Server(s.ctx, num_streams=2, max_batch=64, memory_budget=2 << 30)
        s.owned.append(s.server)
        s.requests = [it[:3] for it in items]
    return s


def _actuate(s):
    s.ctx.actuate(s.nav_of, s.agents, s.actions[s.step % ACTION_SETS], s.collided, s.poses, CAMERA_HEIGHT, s.params)
    s.step += 1
    return {"agents": s.agents, "collided": s.collided, "poses": s.poses}


def run(s):
    if s.kind in ("plain", "noalloc"):
        out = next(iter(s.out.values()))
        call = s.ctx.render_plain if s.kind == "plain" else s.ctx.render_noalloc
        call(s.handles[0], s.sensors[0], s.host_poses, out.get("rgb"), out.get("depth"))
    elif s.kind == "render":
        s.ctx.render(s.handles[0], s.sensors[0], s.host_poses, out=next(iter(s.out.values())))
    elif s.kind == "batch":
        s.ctx.set_poses(s.views, s.host_poses)
        s.ctx.render_batch(None, views=s.views)
    elif s.kind == "stepper":
        s.stepper.step(s.host_poses)
    elif s.kind == "env":
        moved = _actuate(s)
        s.stepper.step_device(s.poses)
        return {"frames": s.out, **moved}
    elif s.kind == "actuate":
        return _actuate(s)
    elif s.kind == "free":
        return s.ctx.nav_free(s.nav, s.points, AGENT_RADIUS, s.out)
    elif s.kind == "serve":
        tickets = [s.server.submit(scene, sensor, pose, o.get("rgb"), o.get("depth"))
                   for (scene, sensor, pose), o in zip(s.requests, s.slices)]
        for t in tickets:
            s.server.wait(t)
    return s.out if s.kind in ("batch", "stepper", "serve") else {"frames": s.out}


def work(case):
    """Bytes: every output once, poses or agents once, and the geometry: all of a scene for a few views of it, the
    quarter that one view can see for a single one (15 bytes a vertex, 12 a triangle).  Operations: the transform
    and setup of the triangles in sight of each view, the edge tests and interpolation of one triangle per pixel."""
    kind, n = case["kind"], case["views"]
    meshes = _meshes(case)
    if kind in ("actuate", "free"):
        # an agent's state twice, its action, pose and flag; a query's point and answer; a contact test or two each
        return {"bytes": n * (114 if kind == "actuate" else 17), "flops": n * (120 if kind == "actuate" else 30)}
    per = {"d": 4, "rgb": 3, "rgbd": 7, "rgbds": 11, "rgbdt": 11}
    pixels = sum(w * h for w, h, _ in _sensors(case))
    bytes_ = sum(w * h * per[o] for w, h, o in _sensors(case)) + 48 * n
    seen = min(1.0, 0.25 * n / len(meshes))
    bytes_ += sum(seen * (15 * m.positions.shape[0] + 12 * m.indices.shape[0]) for m in meshes)
    in_sight = 0.25 * n / len(meshes) * sum(m.indices.shape[0] for m in meshes)
    return {"bytes": int(bytes_), "flops": int(100 * in_sight + 40 * pixels)}


# ---------------------------------------------------------------- the same in 64 bits
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _depth(corners, pose, W, H, hfov):
    """Planar depth of one view [H, W]: at each pixel centre the nearest of the triangles `corners` [T, 3, 3], found
    with homogeneous edge functions (no clipping, no snapping)."""
    dev = corners.device
    p = torch.as_tensor(pose[:3].astype(np.float64), device=dev)
    R = torch.as_tensor(pose[3:].astype(np.float64).reshape(3, 3), device=dev)
    f = W / (2.0 * math.tan(math.radians(hfov) / 2.0))
    c = (corners - p) @ R
    w = -c[..., 2]
    h = torch.stack([f * c[..., 0] + 0.5 * W * w, -f * c[..., 1] + 0.5 * H * w, w], -1)
    x, y = h[..., 0], h[..., 1]
    outside = ((x < 0).all(1) | (x > W * w).all(1) | (y < 0).all(1) | (y > H * w).all(1) | (w < NEAR).all(1))
    h, w = h[~outside], w[~outside]
    det = (h[:, 0] * torch.linalg.cross(h[:, 1], h[:, 2])).sum(1)
    h, w, det = h[det != 0], w[det != 0], det[det != 0]
    edges = torch.stack([torch.linalg.cross(h[:, (k + 1) % 3], h[:, (k + 2) % 3]) for k in range(3)], 1) / det[:, None, None]
    px = h[..., :2] / w[..., None]
    crossing = (w < NEAR).any(1)
    size = torch.tensor([W - 1, H - 1], dtype=torch.float64, device=dev)
    lo = torch.where(crossing[:, None], torch.zeros_like(size), torch.ceil(px.amin(1) - 0.5).clamp(min=0)).minimum(size + 1).long()
    hi = torch.where(crossing[:, None], size, torch.floor(px.amax(1) - 0.5).minimum(size).clamp(min=-1)).long()
    ext = (hi - lo + 1).clamp(min=0)
    count = ext[:, 0] * ext[:, 1]
    rho = torch.zeros(W * H, dtype=torch.float64, device=dev)
    some = torch.nonzero(count).flatten()
    ends = torch.cumsum(count[some], 0)
    begin = 0
    while begin < some.numel():
        done = int(ends[begin - 1]) if begin else 0
        stop = max(begin + 1, int(torch.searchsorted(ends, torch.tensor(done + 16_000_000, device=dev))))
        t = some[begin:stop]
        own = torch.repeat_interleave(torch.arange(t.numel(), device=dev), count[t])
        at = torch.arange(own.numel(), device=dev) - (torch.cumsum(count[t], 0) - count[t])[own]
        wide = ext[t, 0][own]
        i, j = lo[t, 0][own] + at % wide, lo[t, 1][own] + at // wide
        e = edges[t][own]
        b = e[..., 0] * (i + 0.5)[:, None] + e[..., 1] * (j + 0.5)[:, None] + e[..., 2]
        r = b.sum(1)
        hit = (b >= 0).all(1) & (r > 0) & (r <= 1.0 / NEAR)
        rho.scatter_reduce_(0, (j * W + i)[hit], r[hit], "amax")
        begin = stop
    return torch.where(rho > 0, 1.0 / rho, torch.zeros_like(rho)).reshape(H, W)


def _exact_frames(case, meshes, owner, poses):
    """The layout of prepare()'s outputs with the depth images in 64 bits."""
    specs = _sensors(case)
    out = {}
    for spec in sorted(set(specs)):
        out["%dx%d_%s" % spec] = {"depth": None}
    if case.get("sigma") or not any("d" in s[2] for s in specs):
        return None
    corners = [torch.as_tensor(m.positions.astype(np.float64)[m.indices.astype(np.int64)], device=_device()) for m in meshes]
    for spec in sorted(set(specs)):
        if "d" in spec[2]:
            out["%dx%d_%s" % spec]["depth"] = torch.stack(
                [_depth(corners[owner[k]], poses[k], spec[0], spec[1], case["hfov"]) for k, x in enumerate(specs) if x == spec])
    return out


def _segments(mesh):
    """The mesh's cross-sections at BODY_HEIGHTS, [n, 4] in (triangle, height) order."""
    P = mesh.positions.astype(np.float64)[mesh.indices.astype(np.int64)]
    parts, order = [], []
    for k, y in enumerate(BODY_HEIGHTS):
        up = P[..., 1] >= y
        t = np.nonzero(up.any(1) & ~up.all(1))[0]
        ends = []
        for e in range(3):
            a, b, ua, ub = P[t, e], P[t, (e + 1) % 3], up[t, e], up[t, (e + 1) % 3]
            lo, hi = np.where(ua[:, None], b, a), np.where(ua[:, None], a, b)
            with np.errstate(divide="ignore", invalid="ignore"):
                s = (y - lo[:, 1]) / (hi[:, 1] - lo[:, 1])
            ends.append((ua != ub, lo[:, [0, 2]] + s[:, None] * (hi[:, [0, 2]] - lo[:, [0, 2]])))
        first = np.where(ends[0][0][:, None], ends[0][1], ends[1][1])
        last = np.where(ends[2][0][:, None], ends[2][1], ends[1][1])
        parts.append(np.concatenate([first, last], 1))
        order.append(t * len(BODY_HEIGHTS) + k)
    return np.concatenate(parts).astype(np.float32).astype(np.float64)[np.argsort(np.concatenate(order), kind="stable")]


def _first_contact(seg, p, d, r):
    """Earliest contact (time, normal) of discs at p [n, 2] moving by d with the segments [m, 4]; time inf: none."""
    a, b = seg[None, :, :2], seg[None, :, 2:]
    e = b - a
    L2 = (e * e).sum(-1)
    nrm = torch.stack([-e[..., 1], e[..., 0]], -1) / L2.sqrt()[..., None]
    p_, d_ = p[:, None], d[:, None]
    inf = torch.full((), math.inf, dtype=torch.float64, device=p.device)
    d0, rate = ((p_ - a) * nrm).sum(-1), (d_ * nrm).sum(-1)
    sign = torch.where(d0 < 0, -1.0, 1.0)
    d0, rate = d0 * sign, rate * sign
    t = ((d0 - r) / -rate).clamp(min=0)
    s = ((p_ + t[..., None] * d_ - a) * e).sum(-1) / L2
    times = [torch.where((L2 > 0) & (rate < 0) & (t <= 1) & (s >= 0) & (s <= 1), t, inf)]
    dd = (d_ * d_).sum(-1)
    for q in (a, b):
        g = p_ - q
        bq, c = (g * d_).sum(-1), (g * g).sum(-1) - r * r
        disc = bq * bq - dd * c
        t = torch.where(c <= 0, torch.zeros_like(c), (-bq - disc.clamp(min=0).sqrt()) / dd)
        times.append(torch.where((bq < 0) & ((c <= 0) | (disc >= 0)) & (t <= 1), t, inf))
    times = torch.stack(times, -1).flatten(1)
    at = times.argmin(1)
    best, j, kind = times.gather(1, at[:, None])[:, 0], at // 3, at % 3
    row = torch.arange(p.shape[0], device=p.device)
    end = torch.where((kind == 1)[:, None], seg[j, :2], seg[j, 2:])
    off = p + best.clamp(max=1.0)[:, None] * d - end
    side = nrm[0, j] * sign[row, j][:, None]
    return best, torch.where((kind == 0)[:, None], side, off / off.norm(dim=1, keepdim=True))


def _move(seg, p, d, r):
    """Collide-and-slide of discs at p by d, at most four passes."""
    p, d = p.clone(), d.clone()
    going = torch.ones(p.shape[0], dtype=torch.bool, device=p.device)
    for _ in range(4):
        going &= (d * d).sum(1) > 0
        for part in torch.nonzero(going).flatten().split(max(1, 6_000_000 // max(1, seg.shape[0]))):
            if not part.numel():
                continue
            q, m = p[part], d[part]
            near = ((seg[:, 0::2].amin(1) <= q[:, 0].max() + 0.6) & (seg[:, 0::2].amax(1) >= q[:, 0].min() - 0.6)
                    & (seg[:, 1::2].amin(1) <= q[:, 1].max() + 0.6) & (seg[:, 1::2].amax(1) >= q[:, 1].min() - 0.6))
            t, nrm = _first_contact(seg[near], q, m, r) if near.any() else (torch.full_like(q[:, 0], math.inf), m)
            hit = torch.isfinite(t)
            go = torch.where(hit, (t.clamp(max=1.0) - 1e-6 / m.norm(dim=1)).clamp(min=0), torch.ones_like(t))
            p[part] = q + go[:, None] * m
            rest = (1 - go)[:, None] * m
            rest = rest - (rest * nrm).sum(1, keepdim=True) * nrm
            d[part] = torch.where(hit[:, None], rest, torch.zeros_like(rest))
    return p


def _exact_agents(meshes, owner, states, actions):
    """Agent states and camera poses after one action each."""
    dev = _device()
    x, z, yaw = states.T
    agents = torch.as_tensor(np.stack([x, z, -np.sin(yaw), -np.cos(yaw)], 1), device=dev)
    act = torch.as_tensor(actions.astype(np.int64), device=dev)
    turn = math.radians(10.0)
    s = torch.where(act == 2, math.sin(turn), -math.sin(turn))
    fx, fz = agents[:, 2].clone(), agents[:, 3].clone()
    turns = (act == 2) | (act == 3)
    agents[:, 2] = torch.where(turns, fx * math.cos(turn) + fz * s, fx)
    agents[:, 3] = torch.where(turns, fz * math.cos(turn) - fx * s, fz)
    own = torch.as_tensor(owner, device=dev)
    for k, m in enumerate(meshes):
        seg = torch.as_tensor(_segments(m), device=dev)
        at = torch.nonzero((own == k) & (act == 1)).flatten()
        at = at[torch.argsort(torch.floor(agents[at, 0]) * 1000 + agents[at, 1])]     # neighbours share their segments
        for part in at.split(256):
            agents[part, :2] = _move(seg, agents[part, :2], 0.25 * agents[part, 2:], AGENT_RADIUS)
    o, i = torch.zeros_like(fx), torch.ones_like(fx)
    px, pz, fx, fz = agents.T
    poses = torch.stack([px, i * CAMERA_HEIGHT, pz, -fz, o, -fx, o, i, o, fx, o, -fz], 1)
    return {"agents": agents, "collided": None, "poses": poses}


def exact(case, seed):
    kind = case["kind"]
    if kind == "free":
        return None
    meshes, owner, states = _views(case, seed)
    if kind in ("actuate", "env"):
        rng = np.random.default_rng([seed, 8])
        if kind == "env":
            rng.integers(0, 1 << 31, case["views"])
        moved = _exact_agents(meshes, owner, states, rng.choice([1, 1, 2, 3], (ACTION_SETS, case["views"])).astype(np.uint8)[0])
        if kind == "actuate":
            return moved
        poses = moved["poses"].cpu().numpy().astype(np.float32)
        return {"frames": _exact_frames(case, meshes, owner, poses), **moved}
    frames = _exact_frames(case, meshes, owner, _poses(*states.T))
    if frames is None:
        return None
    return frames if kind in ("batch", "stepper", "serve") else {"frames": frames}
