"""Timed work of the pose-scoring library: the calls its users make, over the sizes they make them at.

A case is a dict of plain values.  ``path`` says which calls it stands for:

  score     rm.align_cost / rm.align_cost_grad of a batch of candidate poses, with the pose update of an
            optimizer step where one follows (the inner loop of every alignment)
  align     align.BatchedAligner.run replayed from one captured graph: a whole scan-to-map alignment
  icp       rm.icp_cost_grad + rm.gn_step: one iteration of the render-accelerated ICP of many frame pairs
  odometry  align.sequential_depth_alignment: a depth sequence in, relative poses out
  map       rm.mesh_from_range of every view, Mesh.concat and Mesh.prepare: building the map
  render    rm.render_depth: depth, triangle and class images of a batch of poses

Scenes are those of this repository's workloads (boxes in a room with a doorway, a cluttered 60 m corridor,
Kinect-like cameras, 1 % range noise, 2 % dropouts), drawn anew from every seed and ray-traced on the GPU.
"""
from __future__ import annotations

import math
from dataclasses import dataclass

import numpy as np
import torch

import paper_1702_06813_amd as rm
from paper_1702_06813_amd import align as A

EPS = 0.1                  # Table I threshold of the paper, metres
Z_MIN, Z_MAX = 0.5, 8.0    # sensor range


@dataclass(frozen=True)
class Camera:
    """Pinhole intrinsics, pixel centres at integer coordinates."""
    fx: float
    fy: float
    cx: float
    cy: float
    width: int
    height: int
    z_near: float = 0.1
    z_far: float = 16.0


def _camera(width, height, wide=False):
    """A camera with the Kinect-like (525 px at 640) or the wide (640 px at 1280) field of view."""
    f = width * (0.5 if wide else 525.0 / 640.0)
    return Camera(f, f, 0.5 * (width - 1), 0.5 * (height - 1), int(width), int(height))


# ---------------------------------------------------------------------------- the cases

def _score(name=None, **kw):
    c = dict(path="score", scene="room", map="views", views=27, view_width=640, stride=4, smooth=4, cell=0.0,
             width=640, height=480, scans=1, poses=64, uneven=False, grad=True, step=False, color=False, mask=False,
             spread="fixed")
    c.update(kw)
    return dict({"name": name} if name else {}, **c)


def listed():
    return [
        # the smallest call: one pose of a 64x48 sensor against a 2,400-triangle model, cost only
        _score("smoke_cost", map="grid", cell=0.25, views=0, width=64, height=48, poses=1, grad=False),
        # the paper's plain form: one candidate pose per call, cost only, hundreds of calls per alignment
        _score("plain_cost_1", poses=1, grad=False),
        # a few poses of an odd-sized camera with a validity mask and the color term, cost + gradient
        _score("ragged_color_7", views=20, stride=8, width=333, height=251, poses=7, color=True, mask=True,
               spread="normal"),
        # 64 candidates around an estimate, cost only, a coarse room map
        _score("kinect_cost_64", views=20, stride=8, poses=64, grad=False, spread="normal"),
        # one optimizer iteration of 64 alignments: cost, gradient, Gauss-Newton blocks and pose update
        _score("differentiation_64", poses=64, step=True),
        # 256 candidates of a 1280x960 camera against a 4 M-triangle corridor model with 10 % dead pixels
        _score("wide_256", scene="corridor", map="grid", cell=0.018, views=0, width=1280, height=960, poses=256,
               spread="normal"),
        # 32 scans of three resolutions with 16-128 candidates each, one call
        _score("uneven_32x16_128", scene="corridor", views=56, view_width=320, stride=2, smooth=2, scans=32,
               poses=128, uneven=True, spread="normal"),
        # scan-to-map alignment of a stream: 32 scans of three resolutions, one pose each, 20 iterations
        dict(_score("trajectory_32x20", views=130, stride=6, scans=32, poses=1), path="align", iters=20),
        # one ICP iteration of 32 frame pairs of 320x240
        dict(name="icp_32", path="icp", width=640, height=480, factor=2, stride=1, frames=33),
        # the whole sequential alignment of the same 33 frames, preparation included
        dict(name="odometry_33", path="odometry", width=640, height=480, factor=2, stride=1, frames=33),
        # building the 27-view map of a room, and the prepared buffers of the result
        dict(name="map_27_views", path="map", width=640, height=480, views=27, stride=4, smooth=4),
        # z-buffer images of 16 poses for a viewer or a renderer-in-the-loop
        dict(_score("render_16", poses=16), path="render"),
    ]


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    path = rng.choice(["score"] * 7 + ["align", "icp", "odometry", "map", "render", "render"])
    width = int(log(64, 1280))
    height = max(48, int(width * rng.uniform(0.6, 0.85)))
    if path in ("icp", "odometry"):
        return dict(path=path, width=max(width, 160), height=max(height, 120), factor=rng.choice([1, 2, 2, 3]),
                    stride=rng.choice([1, 1, 2]), frames=int(log(2, 33)))
    if path == "map":
        return dict(path=path, width=max(width, 96), height=max(height, 72), views=int(log(1, 60)),
                    stride=rng.randint(1, 8), smooth=rng.randint(0, 4))
    c = _score(scene=rng.choice(["room", "room", "corridor"]), views=int(log(2, 60)), stride=rng.randint(3, 9),
               view_width=rng.choice([320, 640, 640]), smooth=rng.choice([0, 2, 4, 4]), width=width, height=height,
               poses=int(log(1, 257)), grad=rng.random() < 0.6, spread=rng.choice(["fixed", "normal"]))
    if rng.random() < 0.25:
        c.update(map="grid", views=0, cell=round(log(0.03, 0.3), 4))
    if path == "score":
        c.update(color=rng.random() < 0.25, mask=rng.random() < 0.25, step=c["grad"] and rng.random() < 0.5)
        if rng.random() < 0.3:
            c.update(scans=int(log(2, 33)), uneven=rng.random() < 0.5)
    elif path == "align":
        c.update(path="align", iters=rng.choice([5, 10, 20]), scans=rng.choice([1, 1, int(log(2, 33))]),
                 poses=int(log(1, 65)), grad=True)
    else:
        c.update(path="render", poses=int(log(1, 65)), grad=False)
    # within the largest listed case
    its = c.get("iters", 1)
    while c["poses"] > 1 and (c["poses"] * c["scans"] * c["width"] * c["height"] * its > 2e8
                              or c["poses"] * c["scans"] * _map_tris(c) * its > 4e8):
        c["poses"] = (c["poses"] + 1) // 2
    return c


# ---------------------------------------------------------------------------- what a pass cannot do without

def _map_tris(c):
    if c["map"] == "grid":
        x, y, z = (60.0, 2.5, 2.7) if c["scene"] == "corridor" else (4.0, 4.0, 2.5)
        return int(4 * (x * y + x * z + y * z) / c["cell"] ** 2)
    w, h = c["view_width"], c["view_width"] * 3 // 4
    return 2 * c["views"] * (w // c["stride"]) * (h // c["stride"])


def _scan_sizes(c):
    """(camera width, height) of every scan: one size, or cycling half, whole and double of it."""
    if c["scans"] == 1:
        return [(c["width"], c["height"])]
    f = (1, 2, 4)
    return [(c["width"] * f[k % 3] // 2, c["height"] * f[k % 3] // 2) for k in range(c["scans"])]


def work(case):
    c = case
    p = c["path"]
    if p in ("icp", "odometry"):
        px = -(-c["width"] // c["factor"]) * -(-c["height"] // c["factor"])
        pairs = c["frames"] - 1
        nv = px // c["stride"] ** 2
        tris = 2 * nv
        one = {"bytes": pairs * (24 * nv + 13 * tris + 5 * px + 480), "flops": pairs * (18 * nv + 120 * px)}
        if p == "icp":
            return one
        return {"bytes": 4 * c["frames"] * c["width"] * c["height"] + pairs * 480,
                "flops": 10 * one["flops"] + c["frames"] * px * 100}
    if p == "map":
        px, nv = c["width"] * c["height"], (c["width"] // c["stride"]) * (c["height"] // c["stride"])
        return {"bytes": c["views"] * (4 * px + 12 * nv + 2 * nv * 26),
                "flops": c["views"] * (nv * (20 + 3 * (2 * c["smooth"] + 1) ** 2) + 60 * nv)}
    sizes = _scan_sizes(c)
    tris = _map_tris(c)
    n = (c["poses"] + 16) / 2 if c["uneven"] else c["poses"]
    px = sum(w * h for w, h in sizes)
    poses = n * len(sizes)
    its = c.get("iters", 1)
    mesh = 6 * tris + 13 * tris          # half a vertex and one index triple and class per triangle
    if p == "render":
        return {"bytes": mesh + poses * 96 + n * px * 9, "flops": poses * tris * 9 + n * px * 10}
    return {"bytes": mesh + px * 5 + poses * 480,
            "flops": its * (poses * tris * 9 + n * px * (120 if c["grad"] else 30))}


# ---------------------------------------------------------------------------- scenes and sensors

def _look(pos, yaw, pitch):
    f = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
    x = np.cross(f, [0.0, 0.0, 1.0])
    x /= np.linalg.norm(x)
    return np.concatenate([np.stack([x, np.cross(f, x), f], 1), np.asarray(pos, np.float64)[:, None]], 1)


def _rotation(w):
    th = np.linalg.norm(w)
    k = np.array([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]]) / max(th, 1e-12)
    return np.eye(3) + math.sin(th) * k + (1 - math.cos(th)) * k @ k


def _perturbed(T, rng, spread):
    """A start 10 cm / 5 degrees off ("fixed"), or N(0, 3 cm) / N(0, 1.5 degrees) per axis off the truth."""
    d, a = rng.normal(size=3), rng.normal(size=3)
    if spread == "fixed":
        d, a = d * 0.10 / np.linalg.norm(d), a * math.radians(5.0) / np.linalg.norm(a)
    else:
        d, a = 0.03 * d, math.radians(1.5) * a
    return np.concatenate([T[:, :3] @ _rotation(a), (T[:, 3] + d)[:, None]], 1)


class Scene:
    """An axis-aligned room seen from inside, solid boxes in it, and optionally a doorway in the x = max wall."""

    def __init__(self, rng, kind, size=None, n_boxes=None):
        self.kind = kind
        if kind == "corridor":
            size, n_boxes = size or (60.0, 2.5, 2.7), n_boxes or 60
        else:
            size, n_boxes = size or (6.0, 5.0, 2.8), n_boxes or 16
        self.hi = np.array(size)
        boxes = []
        for _ in range(n_boxes):
            w, d, h = rng.uniform(0.2, 0.8, 3)
            x0 = rng.uniform(0.5, size[0] - 0.5 - w)
            if kind == "corridor":
                y0 = 0.05 if rng.random() < 0.5 else size[1] - 0.05 - d
            else:
                y0 = rng.uniform(0.3, size[1] - 0.3 - d)
            boxes.append([[x0, y0, 0.0], [x0 + w, y0 + d, h]])
        self.boxes = np.round(np.array(boxes) * 64) / 64
        self.door = None if kind == "corridor" else (0.3 * size[1], 0.5 * size[1], 2.1)

    def pose(self, rng, s):
        """A sensor pose on a walk through the scene, s in [0, 1)."""
        if self.kind == "corridor":
            x = 1.0 + 0.93 * s * (self.hi[0] - 4.0)
            return _look([x, 1.25 + 0.3 * math.sin(x / 3.0 + 6.3 * rng.random()), rng.uniform(1.3, 1.5)],
                         rng.uniform(-0.25, 0.25), -0.1)
        c, a = 0.5 * self.hi, 2 * math.pi * s + rng.uniform(-0.1, 0.1)
        pos = [c[0] + 0.75 * c[0] * math.cos(a), c[1] + 0.75 * c[1] * math.sin(a), rng.uniform(1.2, 1.7)]
        tgt = c[:2] + rng.uniform(-0.6, 0.6, 2)
        return _look(pos, math.atan2(tgt[1] - pos[1], tgt[0] - pos[0]), math.radians(rng.uniform(-35.0, -10.0)))

    def range_image(self, cam, T, gen, noise=0.01, dropout=0.02, dead=0.0):
        """Ray-traced depth with multiplicative noise, dropouts to "no return" (0) and dead pixels (NaN)."""
        dev = "cuda"
        f64 = dict(dtype=torch.float64, device=dev)
        v, u = torch.meshgrid(torch.arange(cam.height, **f64), torch.arange(cam.width, **f64), indexing="ij")
        rc = torch.stack([(u - cam.cx) / cam.fx, (v - cam.cy) / cam.fy, torch.ones_like(u)], -1).reshape(-1, 3)
        Tt = torch.tensor(T, **f64)
        rw = (rc @ Tt[:, :3].T).float()
        inv = 1.0 / torch.where(rw.abs() < 1e-9, torch.full_like(rw, 1e-9), rw)
        o, hi = Tt[:, 3].float(), torch.tensor(self.hi, dtype=torch.float32, device=dev)
        t_ax = torch.maximum((hi - o) * inv, -o * inv)
        z, ax = t_ax.min(-1)
        if self.door is not None:
            p = o + rw * z[:, None]
            lo, up, top = self.door
            out = (ax == 0) & (rw[:, 0] > 0) & (p[:, 1] > lo) & (p[:, 1] < up) & (p[:, 2] < top)
            z = torch.where(out, torch.full_like(z, math.inf), z)
        for b in torch.tensor(self.boxes, dtype=torch.float32, device=dev).split(16):
            t1, t2 = (b[:, 0, None] - o) * inv, (b[:, 1, None] - o) * inv
            tn, tf = torch.minimum(t1, t2).amax(-1), torch.maximum(t1, t2).amin(-1)
            tn = torch.where((tn <= tf) & (tn > 0), tn, torch.full_like(tn, math.inf))
            z = torch.minimum(z, tn.amin(0))
        self.z_true = z.reshape(cam.height, cam.width)
        z = z * (1.0 + noise * torch.randn(z.shape, generator=gen, device=dev))
        z = torch.where(torch.isfinite(z) & (z <= Z_MAX), z, torch.zeros_like(z))
        z = torch.where(torch.rand(z.shape, generator=gen, device=dev) < dropout, torch.zeros_like(z), z)
        if dead:
            z = torch.where(torch.rand(z.shape, generator=gen, device=dev) < dead, torch.full_like(z, math.nan), z)
        return z.reshape(cam.height, cam.width).contiguous()

    def grid_mesh(self, cell):
        """The surfaces on a grid of about `cell` metres (boxes 8 x 8 quads a face), free-occupied."""
        xyz, tri, off = [], [], 0

        def face(o, e1, e2, n1, n2):
            nonlocal off
            k = dict(dtype=torch.float64, device="cuda")
            a, b = torch.meshgrid(torch.linspace(0, 1, n1 + 1, **k), torch.linspace(0, 1, n2 + 1, **k), indexing="ij")
            xyz.append((torch.tensor(o, **k) + a.reshape(-1, 1) * torch.tensor(e1, **k)
                        + b.reshape(-1, 1) * torch.tensor(e2, **k)).float())
            i = torch.arange((n1 + 1) * (n2 + 1), device="cuda").reshape(n1 + 1, n2 + 1)
            q = [i[:-1, :-1], i[:-1, 1:], i[1:, 1:], i[1:, :-1]]
            t = torch.stack([q[0], q[1], q[2], q[0], q[2], q[3]], -1).reshape(-1, 3)
            tri.append((t + off).int())
            off += (n1 + 1) * (n2 + 1)

        eye = np.eye(3)
        for k, (lo, hi) in enumerate([(np.zeros(3), self.hi), *self.boxes]):
            ext = hi - lo
            n = np.maximum(1, np.round(ext / cell).astype(int)) if k == 0 else np.full(3, 8 if cell < 0.1 else 1)
            for axis in range(3):
                a1, a2 = [j for j in range(3) if j != axis]
                for side in (0, 1):
                    o = lo.copy()
                    o[axis] = (lo, hi)[side][axis]
                    face(o, eye[a1] * ext[a1], eye[a2] * ext[a2], int(n[a1]), int(n[a2]))
        tri = torch.cat(tri).contiguous()
        return rm.Mesh(torch.cat(xyz).contiguous(), tri, torch.zeros(len(tri), dtype=torch.uint8, device="cuda"))


def _albedo(p):
    """A smooth pattern over world points, in [0.05, 0.95]."""
    return 0.5 + 0.15 * torch.sin(2 * math.pi * p / torch.tensor([0.7, 0.9, 0.8], device=p.device)).sum(-1)


def _generators(seed):
    return np.random.default_rng(seed), torch.Generator("cuda").manual_seed(int(seed))


def _poses(T):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(T).reshape(-1, 12))).cuda()


# ---------------------------------------------------------------------------- prepare and run

def _prepare_scored(c, seed):
    rng, gen = _generators(seed)
    small = c["map"] == "grid" and c["scene"] == "room"
    scene = Scene(rng, c["scene"], (4.0, 4.0, 2.5) if small else None, 8 if small else None)
    if c["map"] == "grid":
        mesh = scene.grid_mesh(c["cell"])
    else:
        cam = _camera(c["view_width"], c["view_width"] * 3 // 4)
        parts = []
        for k in range(c["views"]):
            T = scene.pose(rng, k / c["views"])
            parts.append(rm.mesh_from_range(scene.range_image(cam, T, gen), cam, T, c["stride"], Z_MIN, Z_MAX,
                                            0.05 * c["stride"], c["smooth"]))
        mesh = rm.Mesh.concat(parts)
    if c["color"]:
        mesh.color = _albedo(mesh.xyz[mesh.tri.long()].mean(1)).contiguous()
    mesh.prepare()
    scans, counts, poses = [], [], []
    sizes = np.random.default_rng(c["scans"])             # uneven pose counts belong to the case, not to the inputs
    for k, (w, h) in enumerate(_scan_sizes(c)):
        cam = _camera(w, h, wide=w > 1000)
        T = scene.pose(rng, (k + 0.37) / c["scans"])
        scan = rm.scan_image(scene.range_image(cam, T, gen, dead=0.10 if small or c["map"] == "grid" else 0.0),
                             Z_MIN, Z_MAX, cam=cam)
        if c["mask"]:
            scan.mask = (torch.rand((h, w), generator=gen, device="cuda") < 0.9).to(torch.uint8)
        if c["color"]:
            x, y = torch.meshgrid(torch.arange(w, device="cuda"), torch.arange(h, device="cuda"), indexing="xy")
            ray = torch.stack([(x - cam.cx) / cam.fx, (y - cam.cy) / cam.fy, torch.ones_like(x)], -1)
            Tt = torch.tensor(T, dtype=torch.float32, device="cuda")
            p = (ray * scene.z_true[..., None]) @ Tt[:, :3].T + Tt[:, 3]
            scan.color = (_albedo(p) + 0.01 * torch.randn((h, w), generator=gen, device="cuda")).contiguous()
        n = int(sizes.integers(16, c["poses"] + 1)) if c["uneven"] and c["poses"] > 16 else c["poses"]
        scans.append(scan)
        counts.append(n)
        poses += [_perturbed(T, rng, c["spread"]) for _ in range(n)]
    T0 = _poses(poses)
    return {"case": c, "mesh": mesh, "scans": scans, "counts": counts, "T0": T0, "T": T0.clone(),
            "out": torch.empty((len(T0), rm.OUT_STRIDE), dtype=torch.float64, device="cuda")}


def _sequence(c, seed):
    """Depth frames 3 cm apart on an arc through the room."""
    rng, gen = _generators(seed)
    scene, cam = Scene(rng, "room"), _camera(c["width"], c["height"])
    mid, a0 = 0.5 * scene.hi, rng.uniform(0, 2 * math.pi)
    depths = []
    for k in range(c["frames"]):
        a = a0 + 0.03 * k / (0.75 * mid[0])
        pos = [mid[0] * (1 + 0.75 * math.cos(a)), mid[1] * (1 + 0.75 * math.sin(a)), 1.4 + 0.1 * math.sin(0.2 * k)]
        T = _look(pos, math.atan2(mid[1] - pos[1], mid[0] - pos[0]) + 0.2 * math.sin(0.05 * k),
                  math.radians(-20.0 + 5.0 * math.sin(0.13 * k)))
        depths.append(scene.range_image(cam, T, gen, noise=0.005))
    return depths, cam


def prepare(case, seed):
    c = case
    if c["path"] in ("score", "render"):
        return _prepare_scored(c, seed)
    if c["path"] == "align":
        s = _prepare_scored(c, seed)
        s["aligner"] = A.BatchedAligner(s["mesh"], s["scans"], len(s["T0"]), c["iters"], poses_per_scan=s["counts"])
        s["aligner"].run(s["T0"], use_graph=True)         # captures the graph that the program replays
        return s
    if c["path"] == "map":
        rng, gen = _generators(seed)
        scene, cam = Scene(rng, "room"), _camera(c["width"], c["height"])
        views = [scene.pose(rng, k / c["views"]) for k in range(c["views"])]
        return {"case": c, "cam": cam, "views": views, "depths": [scene.range_image(cam, T, gen) for T in views]}
    depths, cam = _sequence(c, seed)
    if c["path"] == "odometry":
        return {"case": c, "depths": depths, "cam": cam}
    mesh, vn, scans, offs, _ = A.prepare_pairs(depths, cam, list(range(c["frames"] - 1)), c["factor"],
                                               stride=c["stride"], max_edge=0.1 * c["stride"])
    # estimates in the middle of the iterations: 5 mm and a quarter of a degree off, in random directions
    rng = np.random.default_rng(seed)
    T0 = []
    for T in offs:
        d, a = rng.normal(size=3), rng.normal(size=3)
        a *= math.radians(0.25) / np.linalg.norm(a)
        T0.append(np.concatenate([T[:, :3] @ _rotation(a), (T[:, 3] + 0.005 * d / np.linalg.norm(d))[:, None]], 1))
    T0 = _poses(T0)
    return {"case": c, "mesh": mesh, "vn": vn, "scans": scans, "counts": [1] * len(scans), "T0": T0, "T": T0.clone(),
            "out": torch.empty((len(T0), rm.OUT_STRIDE), dtype=torch.float64, device="cuda")}


def run(state):
    s, c = state, state["case"]
    if c["path"] == "score":
        fn = rm.align_cost_grad if c["grad"] else rm.align_cost
        if not c["step"]:
            return fn(s["mesh"], s["scans"], s["T0"], EPS, poses_per_scan=s["counts"], out=s["out"], color_tol=0.02)
        s["T"].copy_(s["T0"])
        fn(s["mesh"], s["scans"], s["T"], EPS, poses_per_scan=s["counts"], out=s["out"], color_tol=0.02)
        rm.gn_step(s["out"], s["T"], 1e-3)
        return s["out"], s["T"]
    if c["path"] == "align":
        al = s["aligner"]
        return al.run(s["T0"], use_graph=True), al.out
    if c["path"] == "render":
        return rm.render_depth(s["mesh"], s["scans"][0].cam, s["T0"])
    if c["path"] == "icp":
        s["T"].copy_(s["T0"])
        rm.icp_cost_grad(s["mesh"], s["scans"], s["T"], s["vn"], 0.1, s["counts"], s["out"])
        rm.gn_step(s["out"], s["T"], 1e-6)
        return s["out"], s["T"]
    if c["path"] == "odometry":
        return A.sequential_depth_alignment(s["depths"], s["cam"], c["factor"], stride=c["stride"],
                                            max_edge=0.1 * c["stride"])
    parts = [rm.mesh_from_range(d, s["cam"], T, c["stride"], Z_MIN, Z_MAX, 0.05 * c["stride"], c["smooth"])
             for d, T in zip(s["depths"], s["views"])]
    mesh = rm.Mesh.concat(parts).prepare()
    nc = -(-mesh.n_tris // rm.rendermap.CLUSTER_TRIS)
    bounds = mesh.clusters[:32 * nc].view(nc, 32)                # between bounds and normals lies unwritten padding
    normals = mesh.clusters[-12 * mesh.n_tris:].view(torch.float32)
    return {"xyz": mesh.xyz, "tri": mesh.tri, "cls": mesh.cls, "bounds": bounds[:, :24].contiguous().view(torch.float32),
            "normals": normals}


# ---------------------------------------------------------------------------- the same in 64 bits

def _nearest(xyz, tri, cam, T):
    """Depth [H,W] (inf where none) and triangle id of the nearest surface at every pixel centre."""
    W, H = cam.width, cam.height
    V = (xyz.double() - T[:, 3]) @ T[:, :3]
    a = V[tri.long()]
    z = a[..., 2]
    front = z >= cam.z_near
    ids = (front.any(1) & (z <= cam.z_far).any(1) & torch.isfinite(a).all(-1).all(-1)).nonzero()[:, 0]
    a, z, front = a[ids], z[ids], front[ids]
    b, zb, fb = a.roll(-1, 1), z.roll(-1, 1), front.roll(-1, 1)
    t = (cam.z_near - z) / torch.where(front != fb, zb - z, torch.ones_like(z))
    pts = torch.cat([a, a + t[..., None] * (b - a)], 1)             # corners, and where edges cross the near plane
    ok = torch.cat([front, front != fb], 1)
    zz = torch.where(ok, pts[..., 2], torch.ones_like(pts[..., 2]))
    u, v = cam.fx * pts[..., 0] / zz + cam.cx, cam.fy * pts[..., 1] / zz + cam.cy

    def ends(x, n):
        lo = torch.where(ok, x, torch.full_like(x, math.inf)).amin(1).clamp(-1, n + 1).ceil().clamp(min=0)
        hi = torch.where(ok, x, torch.full_like(x, -math.inf)).amax(1).clamp(-1, n + 1).floor().clamp(max=n - 1)
        return lo.long(), hi.long()

    (x0, x1), (y0, y1) = ends(u, W), ends(v, H)
    n = ((x1 - x0 + 1).clamp(min=0)) * ((y1 - y0 + 1).clamp(min=0))
    ids, a, x0, x1, y0, n = (q[n > 0] for q in (ids, a, x0, x1, y0, n))
    nrm = torch.linalg.cross(a[:, 1] - a[:, 0], a[:, 2] - a[:, 0])
    off = (nrm * a[:, 0]).sum(-1)
    edge = torch.stack([torch.linalg.cross(a[:, k], a[:, (k + 1) % 3]) for k in range(3)], 1)
    edge = edge * torch.sign(off)[:, None, None]
    pix, dep, who = [], [], []
    end = n.cumsum(0)
    start = 0
    while start < len(n):
        base = int(end[start - 1]) if start else 0
        stop = max(start + 1, int(torch.searchsorted(end, base + 20_000_000, right=True)))
        k = torch.repeat_interleave(torch.arange(start, stop, device=n.device), n[start:stop])
        j = torch.arange(len(k), device=n.device) - (end[k] - n[k] - base)
        w = x1[k] - x0[k] + 1
        px, py = x0[k] + j % w, y0[k] + j // w
        r = torch.stack([(px - cam.cx) / cam.fx, (py - cam.cy) / cam.fy, torch.ones_like(px, dtype=torch.float64)], -1)
        zk = off[k] / (nrm[k] * r).sum(-1)
        m = ((edge[k] * r[:, None]).sum(-1) >= 0).all(-1) & (zk >= cam.z_near) & (zk <= cam.z_far)
        pix.append((py * W + px)[m]); dep.append(zk[m]); who.append(ids[k[m]])
        start = stop
    zbuf = torch.full((H * W,), math.inf, dtype=torch.float64, device=xyz.device)
    idb = torch.full((H * W,), 2 ** 40, dtype=torch.long, device=xyz.device)
    if pix:
        pix, dep, who = torch.cat(pix), torch.cat(dep), torch.cat(who)
        zbuf.scatter_reduce_(0, pix, dep, "amin")
        m = dep == zbuf[pix]
        idb.scatter_reduce_(0, pix[m], who[m], "amin")
    return zbuf.reshape(H, W), torch.where(idb < 2 ** 40, idb, -1).reshape(H, W)


def _n_visible(mesh, cam, T):
    """Triangles of the clusters whose bounds meet the view frustum widened by two pixels."""
    nt = mesh.n_tris
    nc = -(-nt // rm.rendermap.CLUSTER_TRIS)
    b = mesh.clusters[:32 * nc].view(nc, 32)[:, :24].contiguous().view(torch.float32).double().reshape(nc, 2, 3)
    i = torch.arange(8, device=b.device)
    corner = torch.stack([b[:, (i >> k) & 1, k] for k in range(3)], -1)                     # [nc, 8, 3]
    P = (corner - T[:, 3]) @ T[:, :3]
    zn = cam.z_near * (1 - 1e-5)
    front = P[..., 2] >= zn
    pts, ok = [P], [front]
    for bit in (1, 2, 4):
        lo = i[(i & bit) == 0]
        p, q, fp, fq = P[:, lo], P[:, lo + bit], front[:, lo], front[:, lo + bit]
        t = (zn - p[..., 2]) / torch.where(fp != fq, q[..., 2] - p[..., 2], torch.ones_like(p[..., 2]))
        pts.append(p + t[..., None] * (q - p)); ok.append(fp != fq)
    pts, ok = torch.cat(pts, 1), torch.cat(ok, 1)
    z = torch.where(ok, pts[..., 2], torch.ones_like(pts[..., 2]))
    u, v = cam.fx * pts[..., 0] / z + cam.cx, cam.fy * pts[..., 1] / z + cam.cy
    big = torch.full_like(u, math.inf)
    u0, u1 = torch.where(ok, u, big).amin(1) - 2, torch.where(ok, u, -big).amax(1) + 2
    v0, v1 = torch.where(ok, v, big).amin(1) - 2, torch.where(ok, v, -big).amax(1) + 2
    vis = (front.any(1) & (P[..., 2] <= cam.z_far * (1 + 1e-5)).any(1) & (u1 >= 0) & (v1 >= 0)
           & (u0 <= cam.width - 1) & (v0 <= cam.height - 1))
    size = torch.full((nc,), 256, device=b.device)
    if nc:
        size[-1] = nt - 256 * (nc - 1)
    return float(size[vis].sum())


def _sums(r, J, act):
    r, J = r[act], J[act]
    H = J.T @ J
    iu = torch.triu_indices(6, 6, device=H.device)
    return (r[:, None] * J).sum(0), H[iu[0], iu[1]], float(act.sum())


def _record(mesh, scan, T, grad, icp_normals=None, tol=EPS):
    """One result record."""
    cam = scan.cam
    o = torch.zeros(rm.OUT_STRIDE, dtype=torch.float64, device="cuda")
    z, ids = _nearest(mesh.xyz, mesh.tri, cam, T)
    z, ids = z.reshape(-1), ids.reshape(-1)
    v, u = torch.meshgrid(torch.arange(cam.height, device="cuda"), torch.arange(cam.width, device="cuda"), indexing="ij")
    use = torch.ones_like(ids, dtype=torch.bool) if scan.mask is None else scan.mask.reshape(-1) != 0
    z, ids, u, v = z[use], ids[use], u.reshape(-1)[use], v.reshape(-1)[use]
    ray = torch.stack([(u - cam.cx) / cam.fx, (v - cam.cy) / cam.fy, torch.ones_like(u, dtype=torch.float64)], -1)
    cs, ds = scan.cls.reshape(-1)[use].long(), scan.depth.reshape(-1)[use].double()
    hit = ids >= 0
    cr = torch.where(hit, mesh.cls[ids.clamp(min=0)].long(), 3)
    dz = z - ds
    tri = mesh.tri[ids.clamp(min=0)].long()
    if icp_normals is None:
        p = mesh.xyz.double()[tri]
        n = torch.linalg.cross(p[:, 1] - p[:, 0], p[:, 2] - p[:, 0])
    else:
        n = icp_normals.double()[tri].sum(1)
    n = (n / n.norm(dim=-1, keepdim=True)) @ T[:, :3]
    ndr = (n * ray).sum(-1)
    n = torch.where((ndr < 0)[:, None], n, -n)
    Ps = ds[:, None] * ray
    J = torch.cat([n, torch.linalg.cross(Ps, n)], -1)
    o[rm.OUT_N_VISIBLE] = _n_visible(mesh, cam, T)
    if icp_normals is not None:
        o[rm.OUT_ICP_N_SCAN] = (cs == 0).sum()
        model = (cs == 0) & (cr == 0) & torch.isfinite(ndr)
        o[rm.OUT_ICP_N_MODEL] = model.sum()
        act = model & (dz.abs() < tol)
        e = dz * ndr.abs()
        o[rm.OUT_ICP_COST], o[rm.OUT_ICP_SSE] = dz[act].abs().sum(), (e[act] ** 2).sum()
        b, H, o[rm.OUT_N_ACTIVE] = _sums(e, J, act)
        o[rm.OUT_GRAD:rm.OUT_GRAD + 6], o[rm.OUT_JTR:rm.OUT_JTR + 6], o[rm.OUT_JTJ:rm.OUT_JTJ + 21] = 2 * b, b, H
        return o
    scanned, mapped = (cs == 0) | (cs == 1), (cr == 0) | (cr == 1)
    both = scanned & mapped
    oo, ou, uo = both & (cr == 0) & (cs == 0), both & (cr == 0) & (cs == 1), both & (cr == 1) & (cs == 0)
    pen = torch.where(oo, dz.abs() > EPS, torch.where(ou, dz <= 0, dz > 0))
    cells = [oo & ~pen, oo & pen, ou & ~pen, ou & pen, uo & ~pen, uo & pen, ~scanned, scanned & ~mapped,
             both & (cr == 1) & (cs == 1)]
    counts = torch.stack([m.sum() for m in cells]).double()
    o[rm.OUT_COUNTS:rm.OUT_COUNTS + 9] = counts
    o[rm.OUT_E_TABLE] = (counts[1:6:2] - counts[0:6:2]).sum()
    scored = oo | ou | uo
    e = dz * ndr.abs()
    r = torch.where(oo, e, torch.where(ou, e.clamp(max=0), e.clamp(min=0)))
    o[rm.OUT_E_SOFT] = (2 * (r / EPS).square().clamp(max=1)[scored] - 1).sum()
    if mesh.color is not None and scan.color is not None:
        d = (mesh.color[ids.clamp(min=0)] - scan.color.reshape(-1)[use]).abs()
        ok = cells[0] & torch.isfinite(d)
        o[rm.OUT_COLOR_REWARD], o[rm.OUT_COLOR_PENALTY] = (ok & (d <= 0.02)).sum(), (ok & (d > 0.02)).sum()
    if grad:
        act = scored & (r.abs() < EPS) & (oo | (ou & (dz < 0)) | (uo & (dz > 0)))
        b, H, o[rm.OUT_N_ACTIVE] = _sums(r, J, act)
        o[rm.OUT_GRAD:rm.OUT_GRAD + 6], o[rm.OUT_JTR:rm.OUT_JTR + 6], o[rm.OUT_JTJ:rm.OUT_JTJ + 21] = \
            4 / EPS ** 2 * b, b, H
    return o


def _stepped(out, T, lam):
    """Poses after the Levenberg-Marquardt update of their records."""
    iu = torch.triu_indices(6, 6)
    new = []
    for o, t in zip(out.cpu(), T.cpu().reshape(-1, 3, 4)):
        H = torch.zeros((6, 6), dtype=torch.float64)
        H[iu[0], iu[1]] = o[rm.OUT_JTJ:rm.OUT_JTJ + 21]
        H = H + H.T - torch.diag(H.diag())
        L, bad = torch.linalg.cholesky_ex(H + lam * torch.diag(H.diag()))
        d = torch.zeros(6, dtype=torch.float64) if bad else \
            -torch.cholesky_solve(o[rm.OUT_JTR:rm.OUT_JTR + 6, None], L)[:, 0]
        X = torch.zeros((4, 4), dtype=torch.float64)
        X[0, 1], X[0, 2], X[1, 2] = -d[5], d[4], -d[3]
        X[:3, :3] = X[:3, :3] - X[:3, :3].T
        X[:3, 3] = d[:3]
        M = torch.cat([t, torch.tensor([[0.0, 0.0, 0.0, 1.0]], dtype=torch.float64)])
        new.append((M @ torch.linalg.matrix_exp(X))[:3].reshape(12))
    return torch.stack(new).cuda()


def _exact_map(s):
    """Vertices of every view's grid and triangle normals, in 64 bits (classes and indices have no such value)."""
    c, cam = s["case"], s["cam"]
    parts, normals, bounds = [], [], []
    for d, T in zip(s["depths"], s["views"]):
        R, st = c["smooth"], c["stride"]
        z = d.double()
        valid = torch.isfinite(z) & (z >= Z_MIN) & (z <= Z_MAX)
        none = (z == 0) | torch.isinf(z) | (z > Z_MAX)
        node = z[::st, ::st]
        if R:
            pad = torch.nn.functional.pad(torch.where(valid, z, torch.full_like(z, math.inf)), (R, R, R, R),
                                          value=math.inf)
            tot, cnt = torch.zeros_like(node), torch.zeros_like(node)
            for i in range(2 * R + 1):
                for j in range(2 * R + 1):
                    w = pad[i:i + z.shape[0], j:j + z.shape[1]][::st, ::st]
                    near = (w - node).abs() <= 0.03 * node
                    tot += torch.where(near, w, torch.zeros_like(w))
                    cnt += near
            node = torch.where(valid[::st, ::st], tot / cnt, node)
        k = torch.where(valid[::st, ::st], 2, torch.where(none[::st, ::st], 1, 0))
        node = torch.where(k == 1, torch.full_like(node, Z_MAX), torch.where(k == 0, torch.full_like(node, math.nan), node))
        gh, gw = node.shape
        v, u = torch.meshgrid(torch.arange(gh, device="cuda") * st, torch.arange(gw, device="cuda") * st, indexing="ij")
        p = torch.stack([(u - cam.cx) / cam.fx, (v - cam.cy) / cam.fy, torch.ones_like(node)], -1) * node[..., None]
        Tt = torch.tensor(T, dtype=torch.float64, device="cuda")
        p = p @ Tt[:, :3].T + Tt[:, 3]
        parts.append(p.reshape(-1, 3))
        q = torch.stack([p[:-1, :-1], p[:-1, 1:], p[1:, 1:], p[1:, :-1]], 2)                 # [gh-1, gw-1, 4, 3]
        pad = (0, 0, 0, 0, 0, -(gw - 1) % 8, 0, -(gh - 1) % 8)
        q = torch.nn.functional.pad(q, pad, value=math.nan)                                    # 8x8 blocks of quads
        q = q.reshape(q.shape[0] // 8, 8, q.shape[1] // 8, 8, 4, 3).transpose(1, 2).reshape(-1, 4, 3)
        q = q[torch.isfinite(q).all(-1).all(-1)]
        t = torch.stack([q[:, [0, 1, 2]], q[:, [0, 2, 3]]], 1).reshape(-1, 3, 3)
        n = torch.linalg.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0])
        normals.append(n / n.norm(dim=-1, keepdim=True))
        bounds.append(t)
    t = torch.cat(bounds)
    t = torch.cat([t, t[-1:].expand(-len(t) % 256, 3, 3)]).reshape(-1, 768, 3)
    return {"xyz": torch.cat(parts), "tri": None, "cls": None,
            "bounds": torch.cat([t.amin(1), t.amax(1)], -1), "normals": torch.cat(normals).reshape(-1)}


def exact(case, seed):
    c = case
    if c["path"] in ("align", "odometry"):
        return None                    # every iteration rasterizes again: minutes in this form
    if c["path"] == "map":
        return _exact_map(prepare(c, seed))
    if c["path"] != "icp":
        n = c["poses"] * c["scans"] * (_map_tris(c) + 8 * c["width"] * c["height"])
        if n > 2.5e8:
            return None
    s = prepare(c, seed)
    T = s["T0"].reshape(-1, 3, 4)
    if c["path"] == "render":
        z = torch.stack([_nearest(s["mesh"].xyz, s["mesh"].tri, s["scans"][0].cam, t)[0] for t in T])
        return {"depth": torch.where(torch.isfinite(z), z, torch.full_like(z, math.nan)), "tri": None, "cls": None}
    scan_of = [scan for scan, n in zip(s["scans"], s["counts"]) for _ in range(n)]
    out = torch.stack([_record(s["mesh"], scan, t, c.get("grad", True), s.get("vn")) for scan, t in zip(scan_of, T)])
    if c["path"] == "icp":
        return out, _stepped(out, s["T0"], 1e-6)
    return (out, _stepped(out, s["T0"], 1e-3)) if c["step"] else out
