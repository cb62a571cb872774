"""Timed work of the stereo ray tracer, as a program that uses it would have it done.

Four kinds of pass, each through the public entry points:

  frame    one stereo frame of a resident scene (render_stereo, or rt_render_stereo_noalloc), outputs and workspace
           kept from frame to frame as a viewer keeps them
  batch    many small and large pairs over several scenes at once (render_batch), or a captured batch replayed
           (BatchGraph.launch), as a server does
  rebuild  an animated scene: its triangles are on the device and have moved, so the tree is built again
           (rt_scene_build) and a frame is rendered from it
  display  the 8-bit display image of a rendered pair (compose)

Scenes are triangle soups of the kind the paper measures, scaled up: a height field with spheres standing on it, a few
polyhedra, or analytic spheres over a plane; 30% of a terrain's triangles are mirrors.  Everything is made from the
seed.  exact() is the plain definition in 64 bits: every ray against every primitive.
"""
import ctypes
import functools
import math
import types

import numpy as np
import torch

from paper_1702_01530_amd import rt, stereo

# ---------------------------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------------------------


def _frame(name, scene, width, height, depth, lights, grid=0, spheres=0, level=0, accel="ploc", entry="stereo",
           host=False):
    return {"name": name, "path": "frame", "scene": scene, "grid": grid, "spheres": spheres, "level": level,
            "lights": lights, "depth": depth, "width": width, "height": height, "accel": accel, "entry": entry,
            "host": host}


def listed():
    return [
        # the smallest call there is: analytic spheres over a plane, the size of the paper's own images; launches count
        _frame("spheres_256", "spheres", 256, 256, 1, 1),
        # the paper's five polyhedra (100 triangles), the images read back into pinned host memory as its program does
        _frame("solids_256_readback", "solids", 256, 256, 1, 1, host=True),
        # the paper's prototype had no tree: a few thousand polygons, every ray against every triangle
        _frame("brute_2k_256", "terrain", 256, 256, 1, 1, grid=24, spheres=4, level=2, accel="none"),
        # a request of a small server, rendered without allocating; odd image size
        _frame("noalloc_13k_641x479", "terrain", 641, 479, 4, 2, grid=65, spheres=16, level=2, entry="noalloc"),
        # a viewer's frame of an ordinary scene
        _frame("frame_212k_1080p", "terrain", 1920, 1080, 3, 2, grid=256, spheres=64, level=3),
        # the throughput frame of this repository's benchmark, and the same scene at 4K
        _frame("frame_3.4M_1080p", "terrain", 1920, 1080, 4, 4, grid=1024, spheres=256, level=4),
        _frame("frame_3.4M_4k", "terrain", 3840, 2160, 4, 4, grid=1024, spheres=256, level=4),
        # 16 pairs of mixed sizes and depths over scenes of 1k to 500k triangles, as one batch
        {"name": "batch_16_mixed", "path": "batch", "pairs": 16, "scenes": 4, "tris_lo": 1000, "tris_hi": 500000,
         "largest": 3, "lights": 2, "graph": False},
        # a server's tick: 8 small pairs replayed from a captured graph, poses new each time
        {"name": "batch_8_small_graph", "path": "batch", "pairs": 8, "scenes": 3, "tris_lo": 1000, "tris_hi": 20000,
         "largest": 1, "lights": 2, "graph": True},
        # a small animated scene, built and shown at preview size
        {"name": "rebuild_10k_320x240", "path": "rebuild", "grid": 65, "spheres": 6, "level": 2, "lights": 2, "depth": 2,
         "width": 320, "height": 240, "accel": "ploc"},
        # the benchmark's scene with moving geometry
        {"name": "rebuild_3.4M_640x480", "path": "rebuild", "grid": 1024, "spheres": 256, "level": 4, "lights": 4,
         "depth": 2, "width": 640, "height": 480, "accel": "ploc"},
        # a 4K pair for a red-cyan display
        {"name": "anaglyph_4k", "path": "display", "width": 3840, "height": 2160, "mode": "anaglyph"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _terrain_size(rng, lo, hi):
    """Grid, spheres and level of a terrain of about lo .. hi triangles, a third of them in spheres."""
    t = _log_int(rng, lo, hi)
    level = 1 if t < 5000 else (2 if t < 50000 else (3 if t < 1000000 else 4))
    spheres = max(1, min(256, round(t / 3 / (20 * 4 ** level))))
    grid = max(6, round(math.sqrt(max(t - spheres * 20 * 4 ** level, 50) / 2)) + 1)
    return {"grid": grid, "spheres": spheres, "level": level}


def _image_size(rng, lo, hi):
    """Width and height of about lo .. hi pixels in an ordinary aspect ratio, odd ones among them."""
    px, ratio = _log_int(rng, lo, hi), rng.choice([1.0, 4 / 3, 16 / 10, 16 / 9, 21 / 9])
    return {"width": max(16, round(math.sqrt(px * ratio))), "height": max(16, round(math.sqrt(px / ratio)))}


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "small", "brute", "batch", "rebuild", "rebuild", "display"])
    if kind == "frame":
        c = _frame("", "terrain", 0, 0, rng.randint(0, 4), rng.randint(1, 4), accel=rng.choice(["ploc", "ploc", "karras"]),
                   entry=rng.choice(["stereo", "stereo", "noalloc"]), host=rng.random() < 0.2)
        c.update(_terrain_size(rng, 1000, 3300000))
        # without a workspace a large image takes many passes: callers of that entry point render small ones
        c.update(_image_size(rng, 60000, 600000 if c["entry"] == "noalloc" else 5000000))
    elif kind == "small":
        c = _frame("", rng.choice(["spheres", "solids"]), 0, 0, rng.randint(0, 3), 1,
                   entry=rng.choice(["stereo", "noalloc"]), host=rng.random() < 0.3)
        c.update(_image_size(rng, 4000, 300000))
    elif kind == "brute":
        c = _frame("", "terrain", 0, 0, rng.randint(0, 1), 1, accel="none")
        c.update(_terrain_size(rng, 300, 3000))
        c.update(_image_size(rng, 20000, 80000))
    elif kind == "batch":
        lo = _log_int(rng, 1000, 20000)
        c = {"path": "batch", "pairs": rng.randint(3, 12), "scenes": rng.randint(1, 4), "tris_lo": lo,
             "tris_hi": _log_int(rng, lo, 500000), "largest": rng.randint(0, 3), "lights": rng.randint(1, 2),
             "graph": rng.random() < 0.5}
    elif kind == "rebuild":
        c = {"path": "rebuild", "lights": rng.randint(1, 4), "depth": rng.randint(0, 3),
             "accel": rng.choice(["ploc", "ploc", "karras"])}
        c.update(_terrain_size(rng, 1000, 3300000))
        c.update(_image_size(rng, 30000, 640 * 480))
    else:
        c = {"path": "display", "mode": rng.choice(["anaglyph", "side_by_side"])}
        c.update(_image_size(rng, 60000, 3840 * 2160))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------------------------
# Scenes and cameras
# ---------------------------------------------------------------------------------------------

DEV = "cuda"
EXTENT = 16.0
LIGHTS = [[-6, 8, 2], [6, 6, 12], [-5, 7, 14], [5, 8, 1]]


def _lights(n):
    return np.asarray([p + [1.4 / (n + 1)] * 3 for p in LIGHTS[:n]], np.float32)


@functools.lru_cache(maxsize=8)
def _icosphere(level):
    """The unit icosahedron after `level` midpoint subdivisions, as [20 * 4^level, 3, 3] corners on the GPU."""
    phi = (1 + math.sqrt(5)) / 2
    v = np.asarray([p for a in (-1, 1) for b in (-phi, phi) for p in ((0, a, b), (a, b, 0), (b, 0, a))])
    f = [(i, j, k) for i in range(12) for j in range(i) for k in range(j)
         if all(abs(np.linalg.norm(v[a] - v[b]) - 2) < 1e-9 for a, b in ((i, j), (j, k), (i, k)))]
    t = torch.tensor(v[np.asarray(f)] / math.sqrt(1 + phi * phi), dtype=torch.float64, device=DEV)
    for _ in range(level):
        a, b, c = t.unbind(1)
        ab, bc, ca = (torch.nn.functional.normalize(x + y, dim=-1) for x, y in ((a, b), (b, c), (c, a)))
        t = torch.stack([torch.stack(x, 1) for x in ((a, ab, ca), (b, bc, ab), (c, ca, bc), (ab, bc, ca))], 1).reshape(-1, 3, 3)
    return t


def _rotation(rng):
    q = rng.normal(size=4)
    w, x, y, z = q / np.linalg.norm(q)
    return np.asarray([[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                       [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                       [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]])


def _heights(rng):
    """A seeded fractal height function (value noise on a wrapped 256 x 256 lattice, 6 octaves), |h| <= 1."""
    lattice = torch.tensor(rng.uniform(-1, 1, (256, 256)), device=DEV)
    shift = rng.uniform(0, 256, (6, 2))

    def h(x, z):
        total = 0.0
        for o in range(6):
            s, a = 0.25 * 2 ** o, 0.5 ** o
            u, v = x * s + shift[o, 0], z * s + shift[o, 1]
            i, j = u.floor(), v.floor()
            fu, fv = u - i, v - j
            fu, fv = (f * f * f * (f * (f * 6 - 15) + 10) for f in (fu, fv))
            i, j = i.long() % 256, j.long() % 256
            i1, j1 = (i + 1) % 256, (j + 1) % 256
            lo = lattice[i, j] * (1 - fu) + lattice[i1, j] * fu
            hi = lattice[i, j1] * (1 - fu) + lattice[i1, j1] * fu
            total = total + a * (lo * (1 - fv) + hi * fv)
        return total / (2 - 0.5 ** 5)

    return h


def _material(kd, ks, kr, n=32.0):
    return [*kd, *([ks] * 3), *([kr] * 3), n]


def _terrain(grid, spheres, level, lights, seed):
    """Triangles [T,3,3] float32 and material indices [T] int32 on the GPU, and the scene's small arrays."""
    rng = np.random.default_rng([seed, grid, spheres, level])
    h = _heights(rng)
    x = torch.linspace(-EXTENT / 2, EXTENT / 2, grid, dtype=torch.float64, device=DEV)[:, None].expand(grid, grid)
    z = torch.linspace(0, EXTENT, grid, dtype=torch.float64, device=DEV)[None].expand(grid, grid)
    p = torch.stack([x, h(x, z), z], -1)
    a, b, c, d = p[:-1, :-1], p[1:, :-1], p[1:, 1:], p[:-1, 1:]
    ground = torch.stack([torch.stack([a, c, b], -2), torch.stack([a, d, c], -2)], 2).reshape(-1, 3, 3)
    ball = _icosphere(level)
    at = torch.tensor(np.stack([rng.uniform(1 - EXTENT / 2, EXTENT / 2 - 1, spheres), rng.uniform(1, EXTENT - 1, spheres)], 1),
                      device=DEV)
    r = torch.tensor(rng.uniform(0.3, 0.8, spheres) * min(1.0, 8 / math.sqrt(spheres)), device=DEV)
    lift = torch.tensor(rng.uniform(0.2, 1.2, spheres), device=DEV)
    turn = torch.tensor(np.stack([_rotation(rng) for _ in range(spheres)]), device=DEV)
    centre = torch.stack([at[:, 0], h(at[:, 0], at[:, 1]) + r * lift, at[:, 1]], -1)
    balls = torch.matmul(ball.reshape(1, -1, 3), turn) * r[:, None, None] + centre[:, None]
    tris = torch.cat([ground, balls.reshape(-1, 3, 3)]).float()
    owner = torch.cat([torch.zeros(len(ground), dtype=torch.int32, device=DEV),
                       torch.arange(1, spheres + 1, dtype=torch.int32, device=DEV).repeat_interleave(len(ball))])
    mirror = torch.tensor(rng.random(len(tris)) < 0.3, device=DEV)
    mats = []
    for kd in np.concatenate([[[0.45, 0.5, 0.35]], rng.uniform(0.1, 0.9, (spheres, 3))]):
        mats += [_material(kd, 0.3, 0.0), _material(kd, 0.3, 0.8)]
    return tris, owner * 2 + mirror.int(), np.asarray(mats, np.float32), _lights(lights)


def _scene(tris=None, tri_material=None, spheres=(), planes=(), materials=(), lights=()):
    tris = np.zeros((0, 3, 3), np.float32) if tris is None else tris
    spheres, planes = np.asarray(spheres, np.float32).reshape(-1, 4), np.asarray(planes, np.float32).reshape(-1, 4)
    return types.SimpleNamespace(
        triangles=tris, tri_material=np.zeros(0, np.uint32) if tri_material is None else tri_material,
        spheres=spheres, sphere_material=np.arange(len(spheres), dtype=np.uint32),
        planes=planes, plane_material=np.full(len(planes), len(spheres), np.uint32),
        materials=np.asarray(materials, np.float32), lights=lights, ambient=np.full(3, 0.05, np.float32),
        background=np.asarray([0.2, 0.3, 0.5], np.float32))


@functools.lru_cache(maxsize=1)
def _solids():
    """The outward-wound faces of a cube, an icosahedron and a dodecahedron (12, 20 and 36 triangles)."""
    phi = (1 + math.sqrt(5)) / 2
    cube = np.asarray([(x, y, z) for x in (-1, 1) for y in (-1, 1) for z in (-1, 1)], float)
    ring = [p for a in (-1, 1) for b in (-1, 1) for p in ((0, a, b * phi), (a, b * phi, 0), (b * phi, 0, a))]
    ico = np.asarray(ring)
    dodeca = np.concatenate([cube, [p for a in (-1, 1) for b in (-1, 1)
                                    for p in ((0, a / phi, b * phi), (a / phi, b * phi, 0), (b * phi, 0, a / phi))]])
    faces = {"cube": np.concatenate([np.eye(3), -np.eye(3)]),
             "ico": np.concatenate([cube, [p for a in (-1, 1) for b in (-1, 1) for p in
                                           ((0, a * phi, b / phi), (a * phi, b / phi, 0), (b / phi, 0, a * phi))]]),
             "dodeca": np.asarray([p for a in (-1, 1) for b in (-1, 1)
                                   for p in ((0, a * phi, b), (a * phi, b, 0), (b, 0, a * phi))])}
    out = []
    for verts, normals in ((cube, faces["cube"]), (ico, faces["ico"]), (dodeca, faces["dodeca"])):
        verts, tris = verts / np.linalg.norm(verts[0]), []
        for n in normals / np.linalg.norm(normals, axis=1, keepdims=True):
            at = np.nonzero(verts @ n > (verts @ n).max() - 1e-9)[0]
            c = verts[at].mean(0)
            e = verts[at[0]] - c
            angle = np.arctan2((verts[at] - c) @ np.cross(n, e) / np.linalg.norm(e), (verts[at] - c) @ e)
            v = verts[at[np.argsort(angle, kind="stable")]]
            tris += [(v[0], v[k], v[k + 1]) for k in range(1, len(v) - 1)]
        out.append(np.asarray(tris))
    return out


def _host_scene(case, seed):
    """The scene of a frame case, as the host arrays that GpuScene takes."""
    if case["scene"] == "terrain":
        tris, mat, mats, lights = _terrain(case["grid"], case["spheres"], case["level"], case["lights"], seed)
        return _scene(tris.cpu().numpy(), mat.cpu().numpy().view(np.uint32), materials=mats, lights=lights)
    rng = np.random.default_rng([seed, 77])
    light = np.asarray([[rng.uniform(-3, 3), rng.uniform(4, 6), rng.uniform(0, 2), 1, 1, 1]], np.float32)
    if case["scene"] == "spheres":
        balls = np.stack([rng.uniform(-2, 2, 8), rng.uniform(0, 2, 8), rng.uniform(3, 7, 8), rng.uniform(0.2, 0.6, 8)], 1)
        mats = [_material(rng.uniform(0.1, 0.9, 3), s, s) for s in rng.uniform(0, 0.6, 8)] + [_material([0.5] * 3, 0, 0)]
        return _scene(spheres=balls, planes=[[0, 1, 0, 0]], materials=mats, lights=light)
    cube, ico, dodeca = _solids()
    tris, mat, mats = [], [], []
    for k, solid in enumerate((cube, cube, ico, ico, dodeca)):
        centre = [rng.uniform(-2, 2), rng.uniform(0.5, 2), rng.uniform(3, 7)]
        tris.append(solid @ _rotation(rng).T * rng.uniform(0.3, 0.6) + centre)
        mat.append(np.full(len(solid), k, np.uint32))
        mats.append(_material(rng.uniform(0.1, 0.9, 3), rng.uniform(0, 0.5), rng.uniform(0, 0.5)))
    return _scene(np.concatenate(tris).astype(np.float32), np.concatenate(mat), materials=mats, lights=light)


def _camera(center, target, width, height, depth, baseline=0.065):
    """Values as the FP32 camera holds them."""
    c, t = np.asarray(center, np.float32), np.asarray(target, np.float32)
    return types.SimpleNamespace(center=c, forward=t - c, up=np.asarray([0, 1, 0], np.float32), hfov_deg=60.0,
                                 baseline=float(np.float32(baseline)), convergence=float(np.linalg.norm(t - c).astype(np.float32)),
                                 width=width, height=height, max_depth=depth)


def _case_camera(case, seed):
    w, h, d = case["width"], case["height"], case["depth"]
    if case["path"] == "frame" and case["scene"] != "terrain":
        return _camera((0, 1, 0), (0, 1, 5), w, h, d)
    j = np.random.default_rng([seed, 5]).uniform(-0.5, 0.5, 2)  # where the viewer stands just now
    return _camera((j[0], 2.5 + 0.5 * j[1], -4), (0, 0, 8), w, h, d)


SIZES = [(320, 240), (640, 480), (1280, 720), (1920, 1080)]


def _batch(case, seed):
    """The scenes of a batch, as (grid, spheres, level), and its pairs (scene index, camera)."""
    targets = np.exp(np.linspace(math.log(case["tris_lo"]), math.log(case["tris_hi"]), case["scenes"]))
    scenes = []
    for t in targets:
        level = 1 if t < 5000 else (2 if t < 50000 else 3)
        n = int(max(2, min(64, round(0.35 * t / (20 * 4 ** level)))))
        scenes.append((int(max(6, round(math.sqrt(max(t - n * 20 * 4 ** level, 50) / 2)) + 1)), n, level))
    shape = np.random.default_rng([case["pairs"], case["scenes"], case["largest"]])  # sizes and depths are the case's
    pose = np.random.default_rng([seed, 9])
    pairs = []
    for i in range(case["pairs"]):
        w, h = SIZES[int(shape.integers(case["largest"] + 1))]
        depth, k = int(shape.integers(1, 4)), int(shape.integers(case["scenes"]))
        angle, r = pose.uniform(0, 2 * math.pi), pose.uniform(7, 11)
        eye = [r * math.sin(angle), pose.uniform(2, 4), 8 - r * math.cos(angle)]
        pairs.append((k, _camera(eye, (0, 0, 8), w, h, depth, pose.uniform(0.03, 0.1))))
    return scenes, pairs


# ---------------------------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------------------------


class _Rebuilt:
    """An animated scene: device arrays, a descriptor over them, and storage and scratch kept between builds."""

    def __init__(self, case, seed):
        self.tris, self.mat, mats, lights = _terrain(case["grid"], case["spheres"], case["level"], case["lights"], seed)
        self.mats, self.lights = rt.make_materials(mats), rt.make_lights(lights)
        d = rt.rt_scene_desc()
        d.num_triangles, d.triangles, d.tri_material = len(self.tris), self.tris.data_ptr(), self.mat.data_ptr()
        d.num_materials, d.materials = len(mats), ctypes.cast(self.mats, ctypes.POINTER(rt.rt_material))
        d.num_lights, d.lights = len(lights), ctypes.cast(self.lights, ctypes.POINTER(rt.rt_light))
        d.ambient, d.background = (ctypes.c_float * 3)(0.05, 0.05, 0.05), (ctypes.c_float * 3)(0.2, 0.3, 0.5)
        d.flags = stereo.GpuScene.ACCEL[case["accel"]]
        self.desc = d
        self.storage_bytes, self.scratch_bytes = rt.rt_scene_storage_size(d)
        self.storage, self.storage_ptr = stereo.aligned_buffer(self.storage_bytes, DEV)
        self.scratch, self.scratch_ptr = stereo.aligned_buffer(self.scratch_bytes, DEV)
        self.handle = None

    def build(self):
        self.release()
        self.handle = rt.rt_scene_build(self.desc, self.storage_ptr, self.storage_bytes, self.scratch_ptr,
                                        self.scratch_bytes, stereo.stream_handle())
        return self.handle

    def release(self):
        if self.handle:
            torch.cuda.current_stream().synchronize()  # no render of the last build may be in flight
            rt.rt_scene_release(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.release()
        except Exception:
            pass


def prepare(case, seed):
    if case["path"] == "frame":
        cam = _case_camera(case, seed)
        gs = stereo.GpuScene(_host_scene(case, seed), accel=case["accel"])
        out = stereo.alloc_outputs(cam, gs.num_lights, gs.device, host=case["host"])
        ws = stereo.Workspace.for_camera(cam, gs.num_lights) if case["entry"] == "stereo" else None
        return {"case": case, "gs": gs, "cam": cam, "out": out, "ws": ws}
    if case["path"] == "batch":
        scenes, pairs = _batch(case, seed)
        built = []
        for k, size in enumerate(scenes):
            tris, mat, mats, lights = _terrain(*size, case["lights"], seed * 10 + k)
            built.append(stereo.GpuScene(_scene(tris.cpu().numpy(), mat.cpu().numpy().view(np.uint32), materials=mats, lights=lights)))
        pairs = [(built[k], cam) for k, cam in pairs]
        outs = stereo.batch_outputs(pairs)
        ws = stereo.Workspace(rt.rt_render_batch_workspace_size(stereo.batch_items(pairs, outs)))
        graph = stereo.BatchGraph(pairs, outs, ws) if case["graph"] else None
        torch.cuda.synchronize()
        return {"case": case, "pairs": pairs, "outs": outs, "ws": ws, "graph": graph}
    if case["path"] == "rebuild":
        cam = _case_camera(case, seed)
        return {"case": case, "scene": _Rebuilt(case, seed), "cam": rt.make_camera_struct(cam),
                "out": stereo.alloc_outputs(cam, case["lights"], DEV), "ws": stereo.Workspace.for_camera(cam, case["lights"])}
    gen = torch.Generator(device=DEV).manual_seed(seed)
    # linear radiance as frames have it: mostly below 1, some highlights above
    rad = torch.rand((2, case["height"], case["width"], 3), generator=gen, device=DEV) ** 2 * 1.2
    return {"case": case, "out": {"radiance": rad}}


def run(state):
    case = state["case"]
    if case["path"] == "frame":
        if case["entry"] == "stereo":
            return stereo.render_stereo(state["gs"], state["cam"], workspace=state["ws"], outputs=state["out"])
        rt.rt_render_stereo_noalloc(state["gs"].handle, rt.make_camera_struct(state["cam"]),
                                    stereo.output_struct(state["out"]), 0, stereo.stream_handle())
        return state["out"]
    if case["path"] == "batch":
        if state["graph"] is not None:
            return state["graph"].launch(state["pairs"], state["outs"])
        return stereo.render_batch(state["pairs"], workspace=state["ws"], outputs=state["outs"])
    if case["path"] == "rebuild":
        handle = state["scene"].build()
        rt.rt_render_stereo(handle, state["cam"], stereo.output_struct(state["out"]), state["ws"].ptr, state["ws"].nbytes, 0,
                            stereo.stream_handle())
        return state["out"]
    return stereo.compose(state["out"], case["mode"])


# ---------------------------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------------------------


def _render_work(tris, prims, brute, pixels, lights, depth, host):
    """Bytes: every triangle once (its three corners and material, 40 bytes) and the outputs (radiance, distance and id
    of both eyes, 20 bytes a pixel and eye; 12 more where they are read back).  Operations: a primary ray and a shadow
    ray for half the lights at each pixel, and a quarter more of both for mirrors, through a balanced 4-wide tree (four
    slab tests of 13 operations a level) and one triangle test (38), or through every primitive."""
    rays = 2 * pixels * (1 + 0.5 * lights) * (1.25 if depth else 1.0)
    per_ray = 38 * prims if brute else 52 * max(1.0, math.log(max(prims, 2), 4)) + 38
    return {"bytes": 40 * tris + 2 * pixels * (20 + (12 if host else 0)), "flops": rays * per_ray}


def work(case):
    if case["path"] == "display":
        px = case["width"] * case["height"]
        out = 4 * px * (2 if case["mode"] == "side_by_side" else 1)
        read = 12 * px * (2 if case["mode"] == "side_by_side" else 1)  # the channels that the image shows
        return {"bytes": read + out, "flops": 5 * read / 4}
    if case["path"] == "batch":
        scenes, pairs = _batch(case, 0)
        t = [2 * (g - 1) ** 2 + n * 20 * 4 ** lv for g, n, lv in scenes]
        total = {"bytes": 40 * sum(t), "flops": 0.0}
        for k, cam in pairs:
            w = _render_work(0, t[k], False, cam.width * cam.height, case["lights"], cam.max_depth, False)
            total = {x: total[x] + w[x] for x in total}
        return total
    if case["path"] == "frame" and case["scene"] != "terrain":
        tris, prims, brute = (0, 9, True) if case["scene"] == "spheres" else (100, 100, False)
    else:
        tris = prims = 2 * (case["grid"] - 1) ** 2 + case["spheres"] * 20 * 4 ** case["level"]
        brute = case["accel"] == "none"
    w = _render_work(tris, prims, brute, case["width"] * case["height"], case["lights"], case["depth"], case.get("host", False))
    if case["path"] == "rebuild":  # the tree and the triangle records are written once: 48 bytes a triangle and a 64-byte node for 2.6
        w["bytes"] += tris * (48 + 25)
    return w


# ---------------------------------------------------------------------------------------------
# The definition in 64 bits: every ray against every primitive
# ---------------------------------------------------------------------------------------------

TMIN = 1e-4
MOST_TESTS = 6e10


def _cross(a, b):
    return (a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0])


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


class _Exact:
    def __init__(self, s):
        def up(a):
            return torch.as_tensor(np.asarray(a, np.float64), device=DEV)
        v = up(s.triangles) if len(s.triangles) else torch.zeros((0, 3, 3), dtype=torch.float64, device=DEV)
        self.v0, self.e1, self.e2 = v[:, 0], v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
        self.spheres, self.planes, self.mats, self.lights = up(s.spheres), up(s.planes), up(s.materials), up(s.lights)
        self.mat = torch.as_tensor(np.concatenate([np.asarray(m).astype(np.int64) for m in
                                                   (s.tri_material, s.sphere_material, s.plane_material)]), device=DEV)
        self.ambient, self.background = up(s.ambient), up(s.background)
        self.T, self.S, self.P = len(v), len(s.spheres), len(s.planes)

    def _hits(self, o, d, tmin, tmax, skip, lo, hi):
        """t of each ray against primitives lo .. hi of one kind (inf where there is none in (tmin, tmax))."""
        O, D = [x[:, None] for x in o.unbind(1)], [x[:, None] for x in d.unbind(1)]
        inf = float("inf")
        if lo < self.T:
            a, e1, e2 = ([x[None] for x in y[lo:hi].unbind(1)] for y in (self.v0, self.e1, self.e2))
            T, P = [x - y for x, y in zip(O, a)], _cross(D, e2)
            det = _dot(e1, P)
            inv = 1 / det
            u = _dot(T, P) * inv
            Q = _cross(T, e1)
            v, t = _dot(D, Q) * inv, _dot(e2, Q) * inv
            ok = (det != 0) & (u >= 0) & (u <= 1) & (v >= 0) & (u + v <= 1) & (t > tmin) & (t < tmax[:, None])
        elif lo < self.T + self.S:
            s = self.spheres[lo - self.T:hi - self.T]
            oc = [x - c[None] for x, c in zip(O, s[:, :3].unbind(1))]
            b = -_dot(oc, D)
            disc = s[None, :, 3] ** 2 - _dot(*[[x + b * y for x, y in zip(oc, D)]] * 2)
            q = disc.clamp(min=0).sqrt()
            near = (b - q > tmin) & (b - q < tmax[:, None])
            t = torch.where(near, b - q, b + q)
            ok = (disc >= 0) & (t > tmin) & (t < tmax[:, None])
        else:
            p = self.planes[lo - self.T - self.S:hi - self.T - self.S]
            n = [x[None] for x in p[:, :3].unbind(1)]
            nd = _dot(n, D)
            t = (p[None, :, 3] - _dot(n, O)) / nd
            ok = (nd != 0) & (t > tmin) & (t < tmax[:, None])
        ok &= torch.arange(lo, hi, device=DEV)[None] != skip[:, None]
        return torch.where(ok, t, inf)

    def nearest(self, o, d, tmin, tmax, skip):
        """(t, id) of each ray's nearest primitive; (inf, -1) where there is none."""
        t = torch.full((len(o),), float("inf"), dtype=torch.float64, device=DEV)
        k = torch.full((len(o),), -1, dtype=torch.int64, device=DEV)
        rays = 8192
        for r in range(0, len(o), rays):
            at = slice(r, min(len(o), r + rays))
            for lo, hi in ((0, self.T), (self.T, self.T + self.S), (self.T + self.S, self.T + self.S + self.P)):
                for c in range(lo, hi, 2048):
                    h, i = self._hits(o[at], d[at], tmin, tmax[at], skip[at], c, min(hi, c + 2048)).min(1)
                    near = h < t[at]
                    k[at] = torch.where(near, i + c, k[at])
                    t[at] = torch.where(near, h, t[at])
        return t, k

    def radiance(self, o, d, depth, skip, tmin):
        inf = torch.full((len(o),), float("inf"), dtype=torch.float64, device=DEV)
        t, k = self.nearest(o, d, tmin, inf, skip)
        rad = self.background[None].repeat(len(o), 1)
        at = (k >= 0).nonzero()[:, 0]
        if not len(at):
            return rad, t
        key, d1 = k[at], d[at]
        p = o[at] + t[at, None] * d1
        n = torch.zeros_like(p)
        m = key < self.T
        n[m] = torch.linalg.cross(self.e1[key[m]], self.e2[key[m]])
        m = (key >= self.T) & (key < self.T + self.S)
        n[m] = p[m] - self.spheres[key[m] - self.T, :3]
        m = key >= self.T + self.S
        n[m] = self.planes[key[m] - self.T - self.S, :3]
        n = n / n.norm(dim=1, keepdim=True)
        n = torch.where(((n * d1).sum(1) > 0)[:, None], -n, n)
        mat = self.mats[self.mat[key]]
        kd, ks, kr, shine = mat[:, :3], mat[:, 3:6], mat[:, 6:9], mat[:, 9]
        c = self.ambient * kd
        for light in self.lights:
            to = light[:3] - p
            dist = to.norm(dim=1)
            to = to / dist[:, None]
            nl = (n * to).sum(1)
            f = ((nl > 0) & (dist > TMIN)).nonzero()[:, 0]
            hit, _ = self.nearest(p[f], to[f], TMIN, dist[f], key[f])
            f = f[torch.isinf(hit)]
            r = 2 * nl[f, None] * n[f] - to[f]
            spec = (-(r * d1[f]).sum(1)).clamp(min=0) ** shine[f]
            c[f] += light[3:] * (kd[f] * nl[f, None] + ks[f] * spec[:, None])
        f = (kr != 0).any(1).nonzero()[:, 0]
        if depth > 0 and len(f):
            r = d1[f] - 2 * (d1[f] * n[f]).sum(1, keepdim=True) * n[f]
            c[f] += kr[f] * self.radiance(p[f], r / r.norm(dim=1, keepdim=True), depth - 1, key[f], TMIN)[0]
        rad[at] = c
        return rad, t

    def frame(self, cam):
        """radiance [2,H,W,3] and hit distance [2,H,W] of both eyes."""
        W, H = cam.width, cam.height
        f, up = cam.forward.astype(np.float64), cam.up.astype(np.float64)
        f /= np.linalg.norm(f)
        right = np.cross(up, f)
        right /= np.linalg.norm(right)
        down = -np.cross(f, right)
        focal = 0.5 * W / math.tan(math.radians(cam.hfov_deg) / 2)
        x = (torch.arange(W, dtype=torch.float64, device=DEV) + 0.5 - W / 2) / focal
        y = (torch.arange(H, dtype=torch.float64, device=DEV) + 0.5 - H / 2) / focal
        f, right, down = (torch.tensor(v, device=DEV) for v in (f, right, down))
        rad, dist = [], []
        for s in (-cam.baseline / 2, cam.baseline / 2):
            shear = s / cam.convergence if cam.convergence > 0 else 0.0
            d = (f + (x[None, :, None] - shear) * right + y[:, None, None] * down).reshape(-1, 3)
            d = d / d.norm(dim=1, keepdim=True)
            o = (torch.tensor(cam.center.astype(np.float64), device=DEV) + s * right).expand_as(d)
            skip = torch.full((len(d),), -1, dtype=torch.int64, device=DEV)
            a, t = self.radiance(o, d, cam.max_depth, skip, 0.0)
            rad.append(a.reshape(H, W, 3))
            dist.append(t.reshape(H, W))
        return {"radiance": torch.stack(rad), "hit_t": torch.stack(dist)}


def _tests(prims, cam_or_case, lights):
    w, h = (cam_or_case[k] if isinstance(cam_or_case, dict) else getattr(cam_or_case, k) for k in ("width", "height"))
    return 2.0 * w * h * prims * (1 + lights) * 1.4


def exact(case, seed):
    if case["path"] == "display":
        return None  # bytes
    if case["path"] == "batch":
        scenes, pairs = _batch(case, seed)
        t = [2 * (g - 1) ** 2 + n * 20 * 4 ** lv for g, n, lv in scenes]
        if sum(_tests(t[k], cam, case["lights"]) for k, cam in pairs) > MOST_TESTS:
            return None
        ex = []
        for k, size in enumerate(scenes):
            tris, mat, mats, lights = _terrain(*size, case["lights"], seed * 10 + k)
            ex.append(_Exact(_scene(tris.cpu().numpy(), mat.cpu().numpy(), materials=mats, lights=lights)))
        return [ex[k].frame(cam) for k, cam in pairs]
    if case["path"] == "rebuild":
        scene = dict(case, scene="terrain")
    else:
        scene = case
    prims = 100 if scene["scene"] != "terrain" else 2 * (case["grid"] - 1) ** 2 + case["spheres"] * 20 * 4 ** case["level"]
    if _tests(prims, case, case["lights"]) > MOST_TESTS:
        return None
    out = _Exact(_host_scene(scene, seed)).frame(_case_camera(case, seed))
    if case.get("host"):
        out["host_radiance"] = out["radiance"]
    return out
