"""The work a program has this library do, as cases that can be timed and whose outputs can be compared.

A case is a dict of plain values; `family` names the entry points it goes through:

  fuse     tf_reset, then allocation, integration and raycast of a short clip (offline fusion of a sequence)
  swap     the same with host swapping: the camera turns, what leaves the view is swapped out and comes back
  render   raycasts of a finished map from views that are not the last frame's (free views, training targets)
  submaps  one frame fused into the nearest of n rigid submaps and several views of the combined field
  infer    the learned depth prefilter on a batch of frames
  grads    the prefilter's forward pass and every parameter gradient of a training batch
  track    the depth tracker against a rendered map
  mesh     marching cubes over every block of a finished map
  filter   the bilateral depth filter
  surfel   a clip fused into an empty surfel map, and the map

Sizes and parameters are those of the repository's benchmark and tests: 160x120 at 1 cm voxels, 640x480 at 5 mm,
4 mm for the large map, views of 320x240 to 1280x720, ragged 333x251 images, training crops of 8 x 256 x 256.
Every input is a seeded room of 4 x 4 x 3 m with 20 spheres and boxes seen from a loop around its centre, with
Kinect-like noise, rendered on the GPU.
"""
import ctypes
import math
import types

import numpy as np
import torch

import paper_1708_00783_amd as T

# ---- the cases ------------------------------------------------------------------------------------


def listed():
    return [
        # the smallest volume and image: launches and latency are the cost
        dict(name="fuse_160x120_f32_1cm", family="fuse", w=160, h=120, fmt="f32", voxel=0.010, frames=10),
        # the ordinary depth camera at the benchmark's voxel size
        dict(name="fuse_640x480_u16_5mm", family="fuse", w=640, h=480, fmt="u16", voxel=0.005, frames=12),
        # a large depth image on the finest voxels
        dict(name="fuse_1280x720_f32_4mm", family="fuse", w=1280, h=720, fmt="f32", voxel=0.004, frames=6),
        # a camera turning on the spot in a map that does not stay on the device
        dict(name="swap_640x480_u16_5mm", family="swap", w=640, h=480, fmt="u16", voxel=0.005, frames=8),
        # free views of a finished map
        dict(name="render_960x540_5mm", family="render", w=960, h=540, voxel=0.005, frames=24, views=2),
        # submaps: a frame into 6 of 12, four views from 320x240 to 1280x720
        dict(name="submaps_12_views_4", family="submaps", n=12, sel=6, views=4, w=640, h=480, fmt="u16"),
        # the prefilter in front of the fusion, one frame at a time
        dict(name="infer_640x480_u16", family="infer", batch=1, w=640, h=480, fmt="u16"),
        # a training batch
        dict(name="grads_8x256x256_u16", family="grads", batch=8, w=256, h=256, fmt="u16"),
        # frame-to-model tracking of a camera frame
        dict(name="track_640x480_u16_3", family="track", w=640, h=480, fmt="u16", levels=3),
        # the mesh of a room at the end of a scan
        dict(name="mesh_room_5mm", family="mesh", voxel=0.005, frames=24),
        # the classical prefilter, ragged image
        dict(name="filter_333x251_f32_r2", family="filter", w=333, h=251, fmt="f32", radius=2),
        # surfel fusion of a clip
        dict(name="surfel_640x480_u16", family="surfel", w=640, h=480, fmt="u16", frames=6),
    ]


def _between(rng, lo, hi):
    """a whole number, spread over the logarithm of the range"""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["fuse", "fuse", "swap", "render", "submaps", "infer", "infer", "grads", "track", "mesh",
                         "filter", "surfel"])
    fmt = rng.choice(["u16", "f32"])
    w = _between(rng, 96, 1280)
    h = max(64, min(720, int(w * rng.uniform(0.55, 0.8))))
    voxel = rng.choice([0.004, 0.005, 0.01])
    if family == "fuse":
        return dict(family=family, w=w, h=h, fmt=fmt, voxel=voxel, frames=rng.randint(4, 6))
    if family == "swap":
        return dict(family=family, w=min(w, 640), h=min(h, 480), fmt=fmt, voxel=rng.choice([0.005, 0.01]),
                    frames=rng.randint(6, 8))
    if family == "render":
        return dict(family=family, w=w, h=h, voxel=voxel, frames=rng.randint(6, 24), views=rng.randint(1, 2))
    if family == "submaps":
        n = rng.randint(4, 12)
        return dict(family=family, n=n, sel=rng.randint(1, min(6, n)), views=rng.randint(1, 4), w=min(w, 640),
                    h=min(h, 480), fmt=fmt)
    if family == "infer":
        w, h = 8 * _between(rng, 5, 80), 8 * _between(rng, 4, 60)
        return dict(family=family, batch=rng.randint(1, max(1, min(8, 614400 // (w * h)))), w=w, h=h, fmt=fmt)
    if family == "grads":
        return dict(family=family, batch=rng.randint(1, 8), w=8 * _between(rng, 5, 32), h=8 * _between(rng, 4, 32),
                    fmt=fmt)
    if family == "track":
        return dict(family=family, w=w, h=h, fmt=fmt, levels=rng.randint(1, 4))
    if family == "mesh":
        return dict(family=family, voxel=rng.choice([0.005, 0.01]), frames=rng.randint(2, 24))
    if family == "filter":
        return dict(family=family, w=w, h=h, fmt=fmt, radius=rng.randint(1, 7))
    return dict(family=family, w=min(w, 640), h=min(h, 480), fmt=fmt, frames=rng.randint(2, 6))


# ---- rooms, cameras, depth ------------------------------------------------------------------------


def _look_at(eye, target):
    z = target - eye
    z = z / np.linalg.norm(z)
    x = np.cross(z, [0.0, 0.0, 1.0])
    x = x / np.linalg.norm(x)
    R = np.stack([x, np.cross(z, x), z])
    M = np.eye(4)
    M[:3, :3], M[:3, 3] = R, -R @ eye
    return M


class _Room:
    """a seeded room, a loop of 300 camera poses in it, and depth images"""

    def __init__(self, seed):
        self.rng = np.random.default_rng(seed)
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        self.th0, ph = self.rng.uniform(0, 2 * math.pi), self.rng.uniform(0, 2 * math.pi, 3)

        def ring(th):
            return np.array([2.0 + 1.2 * math.cos(th) + 0.2 * math.sin(3 * th + ph[0]),
                             2.0 + 1.2 * math.sin(th) + 0.2 * math.cos(2 * th + ph[1]),
                             1.3 + 0.2 * math.sin(2 * th + ph[2])])
        self.ring = ring
        eyes = np.stack([ring(2 * math.pi * k / 100) for k in range(100)])
        self.solids = []                           # (centre, half size, yaw; yaw None: a sphere)
        while len(self.solids) < 20:
            size = self.rng.uniform(0.1, 0.6)
            c = np.array([*self.rng.uniform(0.4, 3.6, 2), self.rng.uniform(size / 2, 2.0)])
            if np.linalg.norm(eyes - c, axis=1).min() > 0.35 + 0.87 * size:
                self.solids.append((c, size / 2, self.rng.uniform(0, math.pi / 2) if self.rng.uniform() < 0.5 else None))

    def pose(self, k):
        """the k-th of 300 poses of the loop, ~2 cm and ~1 degree apart"""
        th = self.th0 + 2 * math.pi * 0.8 * k / 300
        eye = self.ring(th)
        ahead = self.ring(th + 0.5) - eye + np.array([0.0, 0.0, -0.3])
        return _look_at(eye, eye + ahead).astype(np.float32)

    def turned(self, angle):
        """a pose at the room's centre, looking at a heading"""
        eye = np.array([2.0, 2.0, 1.4])
        return _look_at(eye, eye + [math.cos(angle), math.sin(angle), -0.2]).astype(np.float32)

    def depth(self, pose, intr, fmt, noise=True):
        fx, fy, cx, cy, W, H = intr
        f64 = dict(dtype=torch.float64, device="cuda")
        M = torch.tensor(pose.astype(np.float64), **f64)
        eye = -(M[:3, :3].T @ M[:3, 3])
        ray = torch.stack(torch.broadcast_tensors(((torch.arange(W, **f64) - cx) / fx)[None, :],
                                                  ((torch.arange(H, **f64) - cy) / fy)[:, None],
                                                  torch.ones((), **f64)), -1) @ M[:3, :3]
        hi = torch.tensor([4.0, 4.0, 3.0], **f64)
        z = torch.where(ray > 0, (hi - eye) / ray, torch.where(ray < 0, -eye / ray, math.inf)).amin(-1)
        for c, half, yaw in self.solids:
            if yaw is None:
                oc = eye - torch.tensor(c, **f64)
                a, b, q = (ray * ray).sum(-1), 2 * (ray @ oc), oc @ oc - half * half
                disc = b * b - 4 * a * q
                t = (-b - disc.clamp(min=0).sqrt()) / (2 * a)
                z = torch.where((disc >= 0) & (t > 0) & (t < z), t, z)
            else:
                B = torch.tensor([[math.cos(yaw), -math.sin(yaw), 0], [math.sin(yaw), math.cos(yaw), 0], [0, 0, 1]], **f64)
                o, d = (eye - torch.tensor(c, **f64)) @ B, ray @ B
                t1, t2 = (-half - o) / d, (half - o) / d
                near, far = torch.minimum(t1, t2).amax(-1), torch.maximum(t1, t2).amin(-1)
                z = torch.where((near <= far) & (near > 0) & (near < z), near, z)
        if noise:                                  # axial noise, and holes along depth edges
            g = torch.randn(z.shape, generator=self.gen, **f64)
            holes = torch.rand(z.shape, generator=self.gen, **f64) < 0.5
            edge = torch.zeros_like(holes)
            dx, dy = (z[:, 1:] - z[:, :-1]).abs() > 0.05, (z[1:] - z[:-1]).abs() > 0.05
            edge[:, 1:] |= dx
            edge[:, :-1] |= dx
            edge[1:] |= dy
            edge[:-1] |= dy
            z = z + g * (0.0012 + 0.0019 * (z - 0.4) ** 2)
            z = torch.where(edge & holes, 0.0, z)
        z = torch.where((z >= 0.3) & (z <= 4.0), z, 0.0)
        return (z * 1000).round().to(torch.int16) if fmt == "u16" else z.float()


def _intr(w, h):
    f = 525.0 * w / 640.0
    return (f, f, (w - 1) / 2.0, (h - 1) / 2.0, w, h)


def _volume(voxel, buckets=1 << 20, excess=1 << 17, blocks=1 << 18):
    return types.SimpleNamespace(voxel_size=voxel, mu=4 * voxel, max_w=100, n_buckets=buckets, n_excess=excess,
                                 n_blocks=blocks)


def _maps(w, h):
    return (torch.empty((h, w, 4), dtype=torch.float32, device="cuda"),
            torch.empty((h, w, 4), dtype=torch.float32, device="cuda"))


def _scanned(room, vp, frames, most=(640, 480)):
    """a volume for images up to `most`, with `frames` 640x480 frames spread over the whole loop"""
    intr = _intr(640, 480)
    poses = [room.pose(375.0 * k / frames) for k in range(frames)]
    depths = [room.depth(p, intr, "u16") for p in poses]
    vol = T.Volume(vp, max(640, most[0]), max(480, most[1]))
    for d, p in zip(depths, poses):
        vol.alloc_and_visible(d, intr, p)
        vol.integrate(d, p)
    return vol, depths, poses


# ---- what a program has in hand before the call ----------------------------------------------------


def prepare(case, seed):
    s = types.SimpleNamespace(case=case)
    _PREPARE[case["family"]](s, case, seed)
    torch.cuda.synchronize()
    return s


def _prepare_fuse(s, c, seed):
    room = _Room(seed)
    s.intr = T.make_intrinsics(_intr(c["w"], c["h"]))
    first = room.rng.integers(0, 250)
    s.poses = [room.pose(first + k) for k in range(c["frames"])]
    s.depth = [room.depth(p, _intr(c["w"], c["h"]), c["fmt"]) for p in s.poses]
    small = c["voxel"] >= 0.01
    s.vol = T.Volume(_volume(c["voxel"], *((1 << 16, 1 << 14, 1 << 15) if small else ())), c["w"], c["h"])
    s.out = _maps(c["w"], c["h"])


def _prepare_swap(s, c, seed):
    room = _Room(seed)
    s.intr = T.make_intrinsics(_intr(c["w"], c["h"]))
    a0 = room.rng.uniform(0, 2 * math.pi)
    n = c["frames"]                                # out by half of the frames, and back
    s.poses = [room.turned(a0 + 0.45 * min(k, n - 1 - k)) for k in range(n)]
    s.depth = [room.depth(p, _intr(c["w"], c["h"]), c["fmt"]) for p in s.poses]
    s.vol = T.Volume(_volume(c["voxel"], 1 << 17, 1 << 15, 1 << 17), c["w"], c["h"], swap_transfer_blocks=1 << 14)
    s.out = _maps(c["w"], c["h"])


def _prepare_render(s, c, seed):
    room = _Room(seed)
    s.vol, _, _ = _scanned(room, _volume(c["voxel"]), c["frames"], (c["w"], c["h"]))
    s.intr = T.make_intrinsics(_intr(c["w"], c["h"]))
    s.poses = [room.pose(room.rng.uniform(0, 300)) for _ in range(c["views"])]
    s.out = [_maps(c["w"], c["h"]) for _ in range(c["views"])]


def _prepare_submaps(s, c, seed):
    room, n = _Room(seed), c["n"]
    subs = []
    for _ in range(n):                             # uniform rotations, origins inside the room
        q = room.rng.normal(size=4)
        w, x, y, z = q / np.linalg.norm(q)
        P = np.eye(4)
        P[:3, :3] = [[1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w)],
                     [2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w)],
                     [2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)]]
        P[:3, 3] = -P[:3, :3] @ room.rng.uniform([0, 0, 0], [4, 4, 3])
        subs.append(P.astype(np.float32))
    sizes = [(320, 240), (640, 480), (960, 540), (1280, 720)][-c["views"]:]
    s.map = T.MultiMap(_volume(0.005, 1 << 19, 1 << 17, 1 << 18), np.stack(subs), 640, 480, 1280, 720, 1 << 24)
    small = _intr(320, 240)
    for i in range(n):                             # each submap has seen its own stretch of the loop
        for j in range(5):
            p = room.pose(375.0 * (i + 0.4 * j) / n)
            s.map.integrate(room.depth(p, small, "f32", noise=False), small, p, [i])
    k = room.rng.integers(0, n)
    s.sel = [int((k + j) % n) for j in range(c["sel"])]
    s.pose = room.pose(375.0 * (k + 0.5) / n)
    s.intr = T.make_intrinsics(_intr(c["w"], c["h"]))
    s.depth = room.depth(s.pose, _intr(c["w"], c["h"]), c["fmt"])
    s.out = [_maps(w, h) for w, h in sizes]
    s.views = [(T.make_intrinsics(_intr(w, h)), room.pose(375.0 * (k + 0.7 * j) / n), *o)
               for j, ((w, h), o) in enumerate(zip(sizes, s.out))]


def _prefilter(c, seed):
    """(frames, targets, parameters): noisy frames, noiseless depth as the target, He-normal convolutions with small
    biases and a head that corrects by millimetres, as after training"""
    room = _Room(seed)
    intr = _intr(max(c["w"], 320), max(c["h"], 240))
    poses = [room.pose(room.rng.uniform(0, 300)) for _ in range(c["batch"])]
    crop = (slice(0, c["h"]), slice(0, c["w"]))
    frames = torch.stack([room.depth(p, intr, c["fmt"])[crop] for p in poses]).contiguous()
    target = torch.stack([room.depth(p, intr, "f32", noise=False)[crop] for p in poses]).contiguous()
    parts = []
    for name, cin, cout in T.NN_LAYERS:
        std = 0.01 if name == "head" else math.sqrt(2.0 / (9 * cin))
        parts += [room.rng.standard_normal(cout * 9 * cin) * std, room.rng.standard_normal(cout) * 0.01]
    return frames, target, np.concatenate(parts).astype(np.float32)


def _prepare_infer(s, c, seed, training=False):
    s.frames, s.target, params = _prefilter(c, seed)
    s.net = T.Denoiser(c["batch"], c["h"], c["w"], training=training)
    s.net.set_params(params)
    s.out = torch.empty((c["batch"], c["h"], c["w"]), dtype=torch.float32, device="cuda")
    if training:
        s.grads = s.net.tensor("grads")


def _prepare_grads(s, c, seed):
    _prepare_infer(s, c, seed, training=True)


def _prepare_track(s, c, seed):
    room = _Room(seed)
    intr = _intr(c["w"], c["h"])
    first = int(room.rng.integers(0, 250))
    vol = T.Volume(_volume(0.005), c["w"], c["h"])
    for k in range(3):
        s.ref_pose = room.pose(first + k)
        s.ref = vol.frame(room.depth(s.ref_pose, intr, c["fmt"]), intr, s.ref_pose)
    s.depth = room.depth(room.pose(first + 3), intr, c["fmt"])
    s.intr = T.make_intrinsics(intr)
    L = c["levels"]
    s.params = T.make_track_params((4, 5, 10, 10)[:L], (0.1, 0.2, 0.3, 0.3)[:L])
    s.tracker = T.Tracker(c["w"], c["h"], L)


def _prepare_mesh(s, c, seed):
    """Two blocks of one hash bucket land on its entries in the order of a race, and the triangles follow the entries.
    Surface in such blocks is cut out of the depth, so that the arrays of two runs can be compared."""
    room, intr = _Room(seed), _intr(640, 480)
    vp = _volume(c["voxel"], 1 << 22, 1 << 19, 1 << 18)
    vol, depths, poses = _scanned(room, vp, c["frames"])
    pos, off, ptr = vol.entries()
    head = off[:vp.n_buckets] > 0
    shared = np.concatenate([pos[:vp.n_buckets][head], pos[vp.n_buckets:][ptr[vp.n_buckets:] >= 0]]).astype(np.int64)
    side = 8 * c["voxel"]
    lo, n = -8, int(4.6 / side) + 24
    grid = torch.zeros((1, 1, n, n, n), device="cuda")
    at = torch.from_numpy(np.clip(shared - lo, 0, n - 1)).cuda()
    grid[0, 0, at[:, 0], at[:, 1], at[:, 2]] = 1.0
    near = torch.nn.functional.max_pool3d(grid, 3, 1, 1)[0, 0] > 0     # a ray segment ends at most one block away
    vol.reset()
    for d, p in zip(depths, poses):
        M = torch.tensor(p.astype(np.float64), device="cuda")
        z = d.double() / 1000
        x = (torch.arange(640, device="cuda", dtype=torch.float64) - intr[2]) / intr[0]
        y = (torch.arange(480, device="cuda", dtype=torch.float64) - intr[3]) / intr[1]
        cam = torch.stack([z * x[None], z * y[:, None], z], -1)
        b = (((cam - M[:3, 3]) @ M[:3, :3]) / side).floor().long().sub(lo).clamp(0, n - 1)
        d = torch.where(near[b[..., 0], b[..., 1], b[..., 2]], torch.zeros_like(d), d)
        vol.alloc_and_visible(d, intr, p)
        vol.integrate(d, p)
    s.vol, s.count = vol, torch.zeros(1, dtype=torch.int64, device="cuda")
    s.ws = torch.empty(int(T.lib().tf_mesh_workspace_bytes(ctypes.byref(vol.params))), dtype=torch.uint8, device="cuda")
    s.n = 1 << 23                                  # room for a whole scan; the arrays stay 0 beyond the count
    s.verts = torch.zeros((s.n, 3, 3), dtype=torch.float32, device="cuda")
    s.keys = torch.zeros((s.n, 3), dtype=torch.int64, device="cuda")


def _prepare_filter(s, c, seed):
    room = _Room(seed)
    s.depth = room.depth(room.pose(room.rng.uniform(0, 300)), _intr(c["w"], c["h"]), c["fmt"])
    s.out = torch.empty((c["h"], c["w"]), dtype=torch.float32, device="cuda")


def _prepare_surfel(s, c, seed):
    room = _Room(seed)
    first = room.rng.integers(0, 250)
    s.intr = T.make_intrinsics(_intr(c["w"], c["h"]))
    s.poses = [room.pose(first + k) for k in range(c["frames"])]
    s.depth = [room.depth(p, _intr(c["w"], c["h"]), c["fmt"]) for p in s.poses]
    s.map = T.SurfelMap(c["w"] * c["h"] * c["frames"], c["w"], c["h"])
    s.corr = torch.empty((2, c["h"], c["w"]), dtype=torch.int32, device="cuda")
    for d, p in zip(s.depth, s.poses):
        s.map.fuse(d, s.intr, p)
    s.n = s.map.stats()["count"]                   # the map of this clip; the arrays stay 0 beyond it
    s.pos, s.nrm = (torch.zeros((s.map.params.capacity, 4), dtype=torch.float32, device="cuda") for _ in range(2))
    s.time = torch.zeros(s.map.params.capacity, dtype=torch.int32, device="cuda")


_PREPARE = dict(fuse=_prepare_fuse, swap=_prepare_swap, render=_prepare_render, submaps=_prepare_submaps,
                infer=_prepare_infer, grads=_prepare_grads, track=_prepare_track, mesh=_prepare_mesh,
                filter=_prepare_filter, surfel=_prepare_surfel)

# ---- one pass --------------------------------------------------------------------------------------


def run(s):
    return _RUN[s.case["family"]](s)


def _run_fuse(s):
    s.vol.reset()
    for d, p in zip(s.depth, s.poses):
        s.vol.frame(d, s.intr, p, *s.out)
    return s.out


def _run_swap(s):
    s.vol.reset()
    for d, p in zip(s.depth, s.poses):
        s.vol.frame(d, s.intr, p, *s.out)
        s.vol.swap_out()
    return s.out


def _run_render(s):
    for p, o in zip(s.poses, s.out):
        s.vol.raycast(p, s.intr, *o)
    return s.out


def _run_submaps(s):
    s.map.frame(s.depth, s.intr, s.pose, s.sel, s.views)
    return s.out


def _run_infer(s):
    return s.net.forward(s.frames, s.out)


def _run_grads(s):
    s.net.forward(s.frames, s.out)
    return dict(loss=s.net.backward(s.target), grads=s.grads, out=s.out)


def _run_track(s):
    s.tracker.track_async(s.depth, s.intr, *s.ref, s.intr, s.ref_pose, s.ref_pose, s.params)
    r = s.tracker.result                           # pose, then iterations, pairs and status, then the last systems' sums
    return dict(pose=r[:64].view(torch.float32), counts=r[64:100].view(torch.int32), sums=r[104:].view(torch.float64))


def _run_mesh(s):
    v, k, n, w = (ctypes.c_void_p(t.data_ptr()) for t in (s.verts, s.keys, s.count, s.ws))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    T.check(T.lib().tf_mesh(s.vol.ctx, v, k, s.n, n, w, s.ws.numel(), stream), "tf_mesh")
    return dict(count=s.count, keys=s.keys, verts=s.verts)


def _run_filter(s):
    return T.tf_bilateral(s.depth, s.out, s.case["radius"], 2.5, 0.025)


def _run_surfel(s):
    s.map.reset()
    for d, p in zip(s.depth, s.poses):
        s.map.fuse(d, s.intr, p)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (s.pos, s.nrm, s.time, s.corr[0], s.corr[1])]
    T.check(T.lib().tf_surfel_export(s.map.h, s.n, *ptr[:3], stream), "tf_surfel_export")
    T.check(T.lib().tf_surfel_export_frame(s.map.h, *ptr[3:], stream), "tf_surfel_export_frame")
    return dict(pos=s.pos, nrm=s.nrm, time=s.time, corr=s.corr)


_RUN = dict(fuse=_run_fuse, swap=_run_swap, render=_run_render, submaps=_run_submaps, infer=_run_infer,
            grads=_run_grads, track=_run_track, mesh=_run_mesh, filter=_run_filter, surfel=_run_surfel)

# ---- what a pass cannot do without -----------------------------------------------------------------


def _blocks(w, h, voxel, depth=2.0):
    """blocks of 8^3 voxels along the surface that a w x h camera sees: its area over a block's face, times the blocks
    that the truncation band reaches across"""
    return 1.4 * (w / (525.0 * w / 640.0)) * (h / (525.0 * w / 640.0)) * depth * depth / (8 * voxel) ** 2


def work(case):
    c, fam = case, case["family"]
    px = c.get("w", 0) * c.get("h", 0)
    es = 2 if c.get("fmt") == "u16" else 4
    if fam in ("fuse", "swap"):                    # depth in, maps out, the visible blocks' voxels read and written
        b = _blocks(c["w"], c["h"], c["voxel"])
        return dict(bytes=c["frames"] * (px * (es + 32) + 2 * 1536 * b), flops=c["frames"] * (40 * 512 * b + 300 * px))
    if fam == "render":                            # the distances of the blocks in view, maps out
        return dict(bytes=c["views"] * (32 * px + 1024 * _blocks(c["w"], c["h"], c["voxel"])), flops=c["views"] * 300 * px)
    if fam == "submaps":
        sizes = [(320, 240), (640, 480), (960, 540), (1280, 720)][-c["views"]:]
        b = _blocks(c["w"], c["h"], 0.005)
        return dict(bytes=px * es + c["sel"] * 2 * 1536 * b + sum(32 * w * h + 1536 * _blocks(w, h, 0.005) for w, h in sizes),
                    flops=c["sel"] * 40 * 512 * b + sum(600 * w * h for w, h in sizes))
    if fam in ("infer", "grads"):                  # frames in and out, the parameters; the 3x3 convolutions
        n, flops, scale = c["batch"] * px, 0, dict(e1=1, e2=4, e3=16, e4=64, d3=16, d2=4, d1=1, head=1)
        for name, cin, cout in T.NN_LAYERS:
            flops += 2 * 9 * cin * cout * n / scale[name]
        if fam == "infer":
            return dict(bytes=n * (es + 4) + 4 * 259649, flops=flops)
        return dict(bytes=n * (es + 8) + 8 * 259649, flops=3 * flops)
    if fam == "track":                             # the depth and the reference maps, once; ~100 operations a pair
        its = (4, 5, 10, 10)[:c["levels"]]
        return dict(bytes=px * (es + 32), flops=sum(100 * n * px / 4 ** l for l, n in enumerate(its)))
    if fam == "mesh":                              # voxels in; 60 bytes for each of about 80 triangles a block
        b = min(1.0, 0.25 + c["frames"] / 16) * 90.0 / (8 * c["voxel"]) ** 2
        return dict(bytes=b * (1536 + 60 * 80), flops=b * 512 * 30)
    if fam == "filter":
        return dict(bytes=px * (es + 4), flops=px * 8 * (2 * c["radius"] + 1) ** 2)
    n = 0.45 * px * c["frames"]                    # surfel: depth in, the map read and written by each frame, copied out
    return dict(bytes=c["frames"] * (px * (es + 8) + 36 * n) + 72 * n, flops=c["frames"] * (60 * px + 60 * n))


# ---- the same in 64 bits ---------------------------------------------------------------------------


def exact(case, seed):
    """The prefilter, its gradients and the bilateral filter. The other paths round to stored 16-bit distances and
    decide by 32-bit comparisons at every step (voxel under a pixel, state of a ray, pairs, gates): there is no value
    in more bits that their outputs approach."""
    if case["family"] == "filter":
        s = types.SimpleNamespace()
        _prepare_filter(s, case, seed)
        return _exact_filter(s.depth, case["radius"])
    if case["family"] not in ("infer", "grads"):
        return None
    frames, target, params = _prefilter(case, seed)
    p = torch.from_numpy(params).cuda().double()
    if case["family"] == "infer":
        with torch.no_grad():
            return _exact_prefilter(frames, p)[0]
    p.requires_grad_(True)
    out, depth = _exact_prefilter(frames, p)
    m = (depth > 0) & (target > 0)
    n = m.sum()
    loss = ((out - target.double()).abs() * m).sum() / n
    loss.backward()
    return dict(loss=torch.stack([loss.detach(), n.double()]), grads=p.grad.reshape(-1, 1, 1, 1), out=out.detach())


def _metres(d):
    return (d.float() / 1000.0 if d.dtype.itemsize == 2 else d).double()


def _exact_filter(depth, r):
    d = _metres(depth)
    H, W = d.shape
    pad = torch.nn.functional.pad(d, (r, r, r, r))
    sw, swd = torch.zeros_like(d), torch.zeros_like(d)
    sr, ss = float(np.float32(0.025)), 2.5
    for dy in range(2 * r + 1):
        for dx in range(2 * r + 1):
            q = pad[dy:dy + H, dx:dx + W]
            g = math.exp(-((dy - r) ** 2 + (dx - r) ** 2) / (2 * ss * ss))
            w = torch.where(q > 0, g * torch.exp(-(q - d) ** 2 / (2 * sr * sr)), 0.0)
            sw += w
            swd += w * (q - d)
    return torch.where(d > 0, d + swd / sw.clamp(min=1e-300), 0.0)


def _exact_prefilter(frames, p):
    F = torch.nn.functional
    d = _metres(frames)[:, None]
    B, _, H, W = d.shape
    v = (d > 0).double()
    ones = torch.ones((1, 1, 3, 3), dtype=torch.float64, device="cuda")

    def box(t):
        return (F.unfold(t, 3, padding=1) * ones.reshape(1, 9, 1)).sum(1).reshape(B, 1, H, W)
    hp = torch.where(d > 0, (d - box(d * v) / box(v).clamp(min=1)) / 0.05, 0.0)
    P, o = {}, 0
    for name, cin, cout in T.NN_LAYERS:
        n = cout * 9 * cin
        P[name] = (p[o:o + n].reshape(cout, 3, 3, cin).permute(0, 3, 1, 2).reshape(cout, -1), p[o + n:o + n + cout])
        o += n + cout

    def conv(t, name, stride=1):
        w, b = P[name]
        cols = F.unfold(t, 3, padding=1, stride=stride)
        y = torch.stack([w @ cols[i] for i in range(B)])
        return (y + b[:, None]).reshape(B, -1, (t.shape[2] - 1) // stride + 1, (t.shape[3] - 1) // stride + 1)

    def up(t):
        return t.repeat_interleave(2, 2).repeat_interleave(2, 3)
    e1 = conv(torch.cat([d / 4.0, v, hp], 1), "e1").relu()
    e2 = conv(e1, "e2", 2).relu()
    e3 = conv(e2, "e3", 2).relu()
    e4 = conv(e3, "e4", 2).relu()
    d3 = (conv(up(e4), "d3") + e3).relu()
    d2 = (conv(up(d3), "d2") + e2).relu()
    d1 = (conv(up(d2), "d1") + e1).relu()
    out = torch.where(d > 0, d + 0.05 * conv(d1, "head"), 0.0)
    return out[:, 0], d[:, 0]
