"""Workloads of the framework whose speed is watched, each one pass through the
public entry points as a program that fuses depth video calls them.

    listed()             the named cases
    draw(rng)            one more case of the same ranges, sizes drawn at random
    prepare(case, seed)  what the program holds before the call: images on the GPU,
                         a scene with part of its stream already fused, weights
    run(state)           one pass; returns its outputs
    work(case)           bytes and operations the pass cannot do without
    exact(case, seed)    the outputs in 64 bits from plain torch, where the outputs
                         are numbers computed in one closed sequence (None where a
                         ray's march decides them sample by sample)

Inputs are rendered here: a room with boxes on its floor and balls in the air,
seen by a hand-held depth sensor (noise 0.0012 z^2 m, 5% dropouts, nothing past
4 m), so the sizes of the visible set, the surface angles and the holes are those
of indoor RGB-D video.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1410_0925_amd as itm

RING = 24          # frames of a stream: one closed path of the camera
FUSED = 12         # of them fused before the first pass
MAX_W = 100


def listed():
    return [
        # the smallest calls: a quarter-VGA-sized preview at 1 cm voxels, where
        # launches and host time count
        _frame("frame_160x120_1cm", 160, 120, 0.01, buckets=14),
        # the ordinary frame: VGA at 5 mm, the benchmark's sizes, float32 voxels
        _frame("frame_vga_5mm", 640, 480, 0.005),
        # registered colour beside the depth, in the 3-byte default voxel type
        _frame("frame_vga_colour_s16u8", 640, 480, 0.005, fmt="s16u8", colour=True),
        # the largest frame: 1280x720 in a 7 m hall at 4 mm, the large table, half voxels
        _frame("frame_720p_4mm_f16", 1280, 720, 0.004, fmt="f16", room=7.0, buckets=22),
        # a map larger than its device pool: blocks move to the host and back each frame
        # (a whole turn of the camera; the pool holds every frame's visible set)
        _frame("frame_vga_swap", 640, 480, 0.005, kind="swap", pool=16384, transfer=2048),
        # free-viewpoint rendering of a finished map over [z_near, z_far] (the
        # library's default range), at an odd image size
        {"name": "view_639x479_fixed", "kind": "view", "width": 639, "height": 479, "voxel": 0.005, "fmt": "f32",
         "search_range": False, "room": 4.0, "buckets": 20},
        # the learned refiner over a few-frame map's visible blocks, then the raycast that reads it
        {"name": "refine_vga", "kind": "refine", "width": 640, "height": 480, "voxel": 0.005, "fmt": "f32",
         "room": 4.0, "buckets": 20},
        # the camera pose of a new depth image (default hierarchy, 20 steps)
        {"name": "track_vga", "kind": "track", "width": 640, "height": 480},
        # refiner inference on the blocks of a VGA frame
        {"name": "forward_4001", "kind": "forward", "blocks": 4001},
        # refiner training: minibatches of 256 blocks, Adam, the weights read back at the end
        {"name": "train_256", "kind": "train", "blocks": 256, "steps": 8},
        # saving a map of a room's size, float32
        {"name": "export_32k", "kind": "export", "blocks": 32768, "voxel": 0.005, "fmt": "f32", "buckets": 20},
        # loading a saved map and looking at it
        {"name": "load_32k", "kind": "load", "blocks": 32768, "voxel": 0.005, "fmt": "f32", "buckets": 20,
         "width": 640, "height": 480},
    ]


def _frame(name, width, height, voxel, kind="frame", fmt="f32", colour=False, search_range=True, room=4.0,
           buckets=20, **more):
    return {"name": name, "kind": kind, "width": width, "height": height, "voxel": voxel, "fmt": fmt,
            "colour": colour, "search_range": search_range, "room": room, "buckets": buckets, **more}


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["frame"] * 5 + ["swap", "view", "refine", "track", "forward", "train", "export", "load"])
    if kind == "forward":
        return {"kind": kind, "blocks": int(_log_uniform(rng, 1, 4001))}
    if kind == "train":
        return {"kind": kind, "blocks": int(_log_uniform(rng, 1, 600)), "steps": rng.choice([1, 4, 8])}
    if kind in ("export", "load"):
        c = {"kind": kind, "blocks": 2 * int(_log_uniform(rng, 200, 16384)), "voxel": rng.choice([0.004, 0.005, 0.01]),
             "fmt": rng.choice(["f32", "f32", "f16", "s16u8"]), "buckets": rng.choice([16, 18, 20])}
        if kind == "load":
            c.update(width=rng.randint(160, 640), height=rng.randint(120, 480))
        return c
    width = int(_log_uniform(rng, 96, 1280 if kind == "frame" else 640))
    height = max(60, int(width * rng.choice([0.5625, 0.75])) + rng.randint(-3, 3))
    if kind == "track":
        return {"kind": kind, "width": width, "height": height}
    voxel = round(_log_uniform(rng, 0.005, 0.016), 4)
    c = {"kind": kind, "width": width, "height": height, "voxel": voxel,
         "fmt": rng.choice(["f32", "f32", "f16", "s16u8"]), "room": round(rng.uniform(3.0, 6.0 if kind == "frame" else 4.0), 2),
         "buckets": 20 if voxel < 0.008 else 18}
    if kind == "frame":
        c["colour"] = rng.random() < 0.3
        c["search_range"] = rng.random() < 0.75
    if kind == "view":
        c["search_range"] = rng.random() < 0.5
    if kind == "swap":
        c.update(colour=False, search_range=True, pool=16384, transfer=2048)
    return c


# ---------------------------------------------------------------------------
# inputs: the room, the camera's path, the sensor
# ---------------------------------------------------------------------------
def _room(seed, size):
    """(room lo/hi [2, 3], boxes [n, 2, 3], balls [m, 4]), nothing within 0.8 m of the centre."""
    rng = np.random.default_rng(seed)
    hi = np.array([size, 3.0, size])
    mid = hi / 2
    boxes, balls = [], []
    while len(boxes) < 20:
        s = rng.uniform(0.1, 0.8, 3) * size / 4
        s[1] = min(s[1], 1.2)
        p = np.array([rng.uniform(0, hi[0] - s[0]), 0.0, rng.uniform(0, hi[2] - s[2])])
        if np.linalg.norm(np.maximum(np.maximum(p - mid, mid - p - s), 0)) > 0.8:
            boxes.append(np.stack([p, p + s]))
    while len(balls) < 10:
        r = rng.uniform(0.05, 0.4)
        c = rng.uniform(r, hi - r)
        if np.linalg.norm(c - mid) - r > 0.8:
            balls.append(np.append(c, r))
    return np.stack([np.zeros(3), hi]), np.stack(boxes), np.stack(balls)


def _pose(pos, yaw, pitch):
    """Camera to world; the camera looks along -z at yaw 0 with image "up" = +y."""
    cy, sy, cp, sp = math.cos(yaw), math.sin(yaw), math.cos(pitch), math.sin(pitch)
    Ry = np.array([[cy, 0, sy], [0, 1, 0], [-sy, 0, cy]])
    R0 = np.diag([1.0, -1.0, -1.0])
    Rx = np.array([[1, 0, 0], [0, cp, -sp], [0, sp, cp]])
    T = np.eye(4)
    T[:3, :3] = Ry @ R0 @ Rx
    T[:3, 3] = pos
    return T


def _path(seed, size, turn):
    """RING poses on a closed path, about 1 cm and 1.5 degrees apart; with turn, one whole turn."""
    rng = np.random.default_rng(seed + 77)
    mid = np.array([size / 2, 1.5, size / 2])
    yaw0, a0 = rng.uniform(0, 2 * math.pi, 2)
    poses = []
    for k in range(RING):
        a = 2 * math.pi * k / RING
        pos = mid + 0.045 * np.array([math.cos(a + a0), 0.5 * math.sin(2 * a), math.sin(a + a0)])
        yaw = yaw0 + (a if turn else 0.1 * math.sin(a))
        poses.append(_pose(pos, yaw, 0.1 * math.cos(a) - 0.1))
    return np.stack(poses)


def _camera(c):
    """(fx, fy, cx, cy, width, height); 62 degrees across, square pixels."""
    f = 525.0 / 640.0 * c["width"]
    return (f, f, (c["width"] - 1) / 2, (c["height"] - 1) / 2, c["width"], c["height"])


def _cast(room, K, T):
    """First hits of the camera's rays: camera z, world points and unit normals, float64 [H, W(, 3)]."""
    fx, fy, cx, cy, W, H = K
    dev = "cuda"
    lohi, boxes, balls = (torch.from_numpy(x).to(dev) for x in room)
    R = torch.from_numpy(T[:3, :3].copy()).to(dev)
    o = torch.from_numpy(T[:3, 3].copy()).to(dev)
    xs = (torch.arange(W, dtype=torch.float64, device=dev) - cx) / fx
    ys = (torch.arange(H, dtype=torch.float64, device=dev) - cy) / fy
    ray = torch.stack([xs[None, :].expand(H, W), ys[:, None].expand(H, W),
                       torch.ones((H, W), dtype=torch.float64, device=dev)], -1).reshape(-1, 3)
    d = (R[None, :, 0] * ray[:, :1] + R[None, :, 1] * ray[:, 1:2] + R[None, :, 2] * ray[:, 2:]).T.contiguous()
    d = torch.where(d == 0, torch.full_like(d, 1e-12), d)      # [3, P]
    axis = torch.eye(3, dtype=torch.float64, device=dev)
    far = torch.maximum((lohi[0][:, None] - o[:, None]) / d, (lohi[1][:, None] - o[:, None]) / d)
    t, ax = far.min(0)
    N = -axis[ax] * torch.sign(d.gather(0, ax[None])[0])[:, None]
    for b in boxes:
        t1, t2 = (b[0][:, None] - o[:, None]) / d, (b[1][:, None] - o[:, None]) / d
        tn, bx = torch.minimum(t1, t2).max(0)
        hit = (tn <= torch.maximum(t1, t2).min(0).values) & (tn > 0) & (tn < t)
        t = torch.where(hit, tn, t)
        N = torch.where(hit[:, None], -axis[bx] * torch.sign(d.gather(0, bx[None])[0])[:, None], N)
    a2 = (d * d).sum(0)
    for s in balls:
        oc = o - s[:3]
        b = (d * oc[:, None]).sum(0)
        disc = b * b - a2 * ((oc * oc).sum() - s[3] * s[3])
        th = (-b - torch.sqrt(torch.clamp(disc, min=0))) / a2
        hit = (disc >= 0) & (th > 0) & (th < t)
        t = torch.where(hit, th, t)
        N = torch.where(hit[:, None], (oc[None] + th[:, None] * d.T) / s[3], N)
    X = o[None] + t[:, None] * d.T
    return t.view(H, W), X.view(H, W, 3), N.view(H, W, 3)


def _sensor(z, gen):
    z = z + torch.randn(z.shape, dtype=torch.float64, device="cuda", generator=gen) * (0.0012 * z * z)
    bad = (z <= 0) | (z > 4.0) | (torch.rand(z.shape, device="cuda", generator=gen) < 0.05)
    return torch.where(bad, torch.zeros_like(z), z).float()


def _colour(X, depth, gen):
    """The registered colour image of world points X: three smooth waves, sensor noise, black where invalid."""
    k = torch.tensor([[2.3, 0.7, -1.1], [-0.9, 2.8, 0.6], [1.2, -1.4, 2.5]], dtype=torch.float64, device="cuda")
    ph = torch.tensor([0.3, 1.9, 4.1], dtype=torch.float64, device="cuda")
    wave = (X[..., None, :] * k).sum(-1) * (2 * math.pi / 1.6) + ph
    c = 128 + 110 * torch.sin(wave) + 1.5 * torch.randn(wave.shape, dtype=torch.float64, device="cuda", generator=gen)
    c = torch.where((depth > 0)[..., None], torch.clamp(torch.round(c), 0, 255), torch.zeros_like(c))
    out = torch.zeros((*depth.shape, 4), dtype=torch.uint8, device="cuda")
    out[..., :3] = c.to(torch.uint8)
    return out


def _stream(c, seed, turn=False, frames=RING):
    room, K, poses = _room(seed, c["room"]), _camera(c), _path(seed, c["room"], turn)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    depth, rgb = [], []
    for k in range(frames):
        z, X, _ = _cast(room, K, poses[k])
        depth.append(_sensor(z, gen))
        if c.get("colour"):
            rgb.append(_colour(X, depth[-1], gen))
    return K, poses, depth, rgb


def _new_scene(c):
    v = c["voxel"]
    sc = itm.Scene(v, 4 * v, MAX_W, 2 ** c["buckets"], 2 ** (c["buckets"] - 2), fmt=c["fmt"])
    if c["kind"] == "swap":
        sc.enable_swapping(c["pool"], c["transfer"], c["transfer"])
    if c.get("colour"):
        sc.enable_colour()
    sc.set_search_range(c.get("search_range", c["kind"] == "refine"))
    return sc


def _refiner_params(seed):
    """He-normal layers 1-3, a small last layer: corrections of a few hundredths, as after training."""
    rng = np.random.default_rng(seed)
    W = np.zeros((4, 27, 16, 16))
    W[0, :, :, :2] = rng.standard_normal((27, 16, 2)) * np.sqrt(2.0 / 54)
    W[1:3] = rng.standard_normal((2, 27, 16, 16)) * np.sqrt(2.0 / 432)
    W[3, :, 0] = rng.standard_normal((27, 16)) * 0.003
    b = np.zeros((4, 16))
    b[:3] = rng.standard_normal((3, 16)) * 0.05
    return np.concatenate([W.ravel(), b.ravel()]).astype(np.float32)


def _blocks(n, seed):
    """Haloed blocks [n, 2000]: a noisy plane's TSDF after a few frames, part of it not yet seen."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    nrm = r(n, 3)
    nrm = nrm / nrm.norm(dim=1, keepdim=True)
    g = torch.arange(10, device="cuda", dtype=torch.float32) - 4.5
    dist = (nrm[:, 0, None, None, None] * g + nrm[:, 1, None, None, None] * g[:, None]
            + nrm[:, 2, None, None, None] * g[:, None, None]) + 2 * r(n, 1, 1, 1)
    F = torch.clamp(dist / 4 + 0.15 * r(n, 10, 10, 10), -1, 1)
    Wt = torch.randint(1, 6, (n, 10, 10, 10), device="cuda", generator=gen).float()
    unseen = dist < -4
    F, Wt = torch.where(unseen, torch.ones_like(F), F), torch.where(unseen, torch.zeros_like(Wt), Wt)
    clean = torch.clamp(dist / 4, -1, 1)[:, 1:9, 1:9, 1:9].reshape(n, 512).contiguous()
    mask = (~unseen[:, 1:9, 1:9, 1:9]).to(torch.uint8).reshape(n, 512).contiguous()
    return torch.stack([F, Wt / MAX_W], 1).reshape(n, 2000).contiguous(), clean, mask


def _terrain(c, seed):
    """A saved map: two layers of blocks along a rolling surface y = h(x, z), in random
    order: keys [n, 3], F and W [n, 512] on the host, the surface height at the origin."""
    n = c["blocks"] // 2
    nx = max(1, math.isqrt(n))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    i = torch.arange(n, device="cuda")
    bx, bz = i % nx - nx // 2, i // nx - nx // 2
    ph = torch.rand(4, device="cuda", generator=gen, dtype=torch.float64) * 6
    s, mu = c["voxel"], 4 * c["voxel"]

    def height(x, z):
        return 0.15 * torch.sin(2.1 * x + ph[0]) + 0.1 * torch.sin(3.3 * z + ph[1]) + 0.05 * torch.sin(4 * (x + z) + ph[2])

    by = torch.floor((height((bx + 0.5) * 8.0 * s, (bz + 0.5) * 8.0 * s) - mu) / (8 * s)).long()
    key = torch.cat([torch.stack([bx, by + k, bz], 1) for k in (0, 1)])
    key = key[torch.randperm(2 * n, device="cuda", generator=gen)]
    v = torch.arange(512, device="cuda")
    at = (8 * key[:, None, :] + torch.stack([v % 8, v // 8 % 8, v // 64], 1)[None]).double() * s
    dist = at[..., 1] - height(at[..., 0], at[..., 2])
    noise = 0.05 * torch.randn(dist.shape, dtype=torch.float64, device="cuda", generator=gen)
    F = torch.clamp(dist / mu + noise, -1, 1).float()
    W = torch.randint(1, MAX_W + 1, dist.shape, device="cuda", generator=gen).float()
    unseen = dist < -mu
    F, W = torch.where(unseen, torch.ones_like(F), F), torch.where(unseen, torch.zeros_like(W), W)
    o = torch.zeros(1, dtype=torch.float64, device="cuda")
    return key.int().cpu().numpy(), F.cpu().numpy(), W.cpu().numpy(), float(height(o, o))


def _track_inputs(c, seed):
    """A depth image, reference maps at the pose of the frame before (5% holes), that pose: the
    camera looks down into a corner of the room and has moved by about 1 cm and 1 degree."""
    room, K = _room(seed, 4.0), _camera(c)
    rng = np.random.default_rng(seed + 5)
    pos, yaw = np.array([2.0, 1.5, 2.0]) + rng.uniform(-0.05, 0.05, 3), math.pi * (0.25 + 0.5 * rng.integers(4))
    yaw += rng.uniform(-0.2, 0.2)
    poses = [_pose(pos, yaw, -0.45), _pose(pos + rng.uniform(-0.008, 0.008, 3), yaw + rng.uniform(-0.02, 0.02), -0.44)]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    depth = _sensor(_cast(room, K, poses[1])[0], gen)
    _, X, N = _cast(room, K, poses[0])
    hit = (torch.rand(X.shape[:2], device="cuda", generator=gen) >= 0.05)[..., None]
    maps = [torch.where(hit, torch.cat([m, torch.ones_like(m[..., :1])], -1), 0.0).float().contiguous() for m in (X, N)]
    return K, depth, maps[0], maps[1], poses[0]


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind, "k": 0}
    if kind == "forward":
        x = _blocks(c["blocks"], seed)[0]
        s.update(refiner=itm.Refiner(_refiner_params(seed)), x=x, out=torch.empty((c["blocks"], 512), device="cuda"))
        return s
    if kind == "train":
        s["batches"] = [_blocks(c["blocks"], seed + 1000 * i) for i in range(c["steps"])]
        s.update(refiner=itm.Refiner(_refiner_params(seed)), losses=torch.empty(c["steps"], device="cuda"))
        return s
    if kind == "track":
        s["K"], s["depth"], s["V"], s["N"], s["T"] = _track_inputs(c, seed)
        s["scene"] = itm.Scene(0.005, 0.02, MAX_W, 2 ** 14, 2 ** 12)
        return s
    if kind in ("export", "load"):
        coords, F, Wt, h = _terrain(c, seed)
        s["scene"] = _new_scene(c)
        s["blocks"] = (coords, F, Wt)
        if kind == "export":
            s["scene"].import_blocks(*s.pop("blocks"))
        else:
            s.update(K=_camera(c), T=_pose(np.array([0.0, h + 0.6, 0.3]), 0.4, -1.0))
        return s
    K, poses, depth, rgb = _stream(c, seed, turn=kind in ("view", "swap"), frames=5 if kind == "refine" else RING)
    sc = _new_scene(c)
    fused = 5 if kind == "refine" else FUSED if kind in ("frame", "swap") else RING
    for k in range(fused):
        if rgb:
            sc.integrate_colour(depth[k], rgb[k], K, poses[k])
        else:
            sc.integrate(depth[k], K, poses[k])
    s.update(scene=sc, K=K, poses=poses, depth=depth, rgb=rgb, k=fused)
    if kind in ("frame", "swap"):
        H, W = c["height"], c["width"]
        s["pts"] = torch.empty((H, W, 4), device="cuda")
        s["nrm"] = torch.empty((H, W, 4), device="cuda")
        if rgb:
            s["crgb"] = torch.empty((H, W, 4), dtype=torch.uint8, device="cuda")
    if kind == "view":      # looked at from poses the sensor never took
        s["poses"] = np.stack([_pose(p[:3, 3] + np.array([0.2, -0.1, 0.1]), 0.7 + 0.26 * k, -0.15)
                               for k, p in enumerate(poses)])
    if kind == "refine":
        s["refiner"] = itm.Refiner(_refiner_params(seed))
        sc.set_refiner(s["refiner"], w_threshold=10.0)
    torch.cuda.synchronize()
    return s


def run(state):
    s, kind = state, state["kind"]
    if kind == "forward":
        return s["refiner"].forward(s["x"], s["out"])
    if kind == "train":
        for i, (x, t, m) in enumerate(s["batches"]):
            s["refiner"].train_step(x, t, m, 1e-3, loss=s["losses"][i:i + 1])
        return {"losses": s["losses"], "params": s["refiner"].params()}
    if kind == "track":
        T, info = s["scene"].track(s["depth"], s["K"], s["V"], s["N"], s["T"])
        return {"pose": T, **info}
    sc = s["scene"]
    if kind == "export":
        return sc.export()
    K = s["K"]
    if kind == "load":
        sc.import_blocks(*s["blocks"])
        return sc.raycast(K, s["T"])
    k = s["k"] % len(s["depth"])
    if kind == "refine":
        sc.refine_visible()
        return sc.raycast(K, s["poses"][4])
    s["k"] += 1
    T = s["poses"][k]
    if kind == "view":
        return sc.raycast(K, T)
    if s["rgb"]:
        sc.integrate_colour(s["depth"][k], s["rgb"][k], K, T)
        return sc.raycast_colour(K, T, s["pts"], s["nrm"], s["crgb"])
    sc.integrate(s["depth"][k], K, T)
    return sc.raycast(K, T, s["pts"], s["nrm"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
FORWARD_FLOP = 2 * 512 * 27 * (2 * 16 + 16 * 16 + 16 * 16 + 16)   # per block, real channels
BACKWARD_FLOP = FORWARD_FLOP + 2 * 512 * 27 * (16 * 16 + 16 * 16 + 16)


def _visible_blocks(c):
    """Blocks a frame's band crosses: the surface in view (mean distance 0.42 of the room, at
    most 2.6 m) in block faces, 1.5 blocks deep, no more than 3 a pixel."""
    z = min(0.42 * c["room"], 2.6)
    area = c["height"] / c["width"] * (640.0 / 525.0) ** 2 * z * z * 1.2
    return min(1.5 * area / (8 * c["voxel"]) ** 2, 3.0 * c["width"] * c["height"])


def work(case):
    c, kind = case, case["kind"]
    if kind == "forward":
        return {"bytes": c["blocks"] * 4 * (2000 + 512), "flops": c["blocks"] * FORWARD_FLOP}
    if kind == "train":
        n = c["blocks"] * c["steps"]
        return {"bytes": n * (4 * (2000 + 512) + 512) + 4 * 27712 * (6 * c["steps"] + 1),
                "flops": n * (FORWARD_FLOP + BACKWARD_FLOP)}
    px = c.get("width", 0) * c.get("height", 0)
    vox = {"f32": 8, "f16": 4, "s16u8": 3}[c.get("fmt", "f32")]
    if kind in ("export", "load"):     # the voxels in the storage form on one side, in float32 on the other
        return {"bytes": c["blocks"] * (512 * (vox + 8) + 28) + 32 * px, "flops": 0}
    if kind == "track":   # 10, 6 and 4 steps on 1/16, 1/4 and all of the pixels: the image and both maps once a step
        steps = 10 / 16 + 6 / 4 + 4
        return {"bytes": steps * px * 36, "flops": steps * px * 140}
    sdf = 4 if c["fmt"] == "f32" else 2
    vis = _visible_blocks(c)
    if kind == "view":
        return {"bytes": 32 * px + vis * (512 * sdf + 16), "flops": 600 * px}
    if kind == "refine":
        return {"bytes": 32 * px + vis * (512 * (vox + 2) + 16), "flops": vis * FORWARD_FLOP + 600 * px}
    upd = 300 * vis       # voxels a frame updates: those in front of or inside the band
    b = 4 * px + 32 * px + 36 * vis + 2 * vox * upd
    if c.get("colour"):
        b += 8 * px + 8 * upd
    if kind == "swap":    # blocks to the host and back, read and written on either side
        b += 4 * c["transfer"] * 512 * vox
    return {"bytes": b, "flops": 30 * 512 * vis + 600 * px}


# ---------------------------------------------------------------------------
# the same numbers in 64 bits
# ---------------------------------------------------------------------------
def _unpack(params):
    p = torch.from_numpy(params.astype(np.float64)).cuda()
    return p[:27 * 16 * 16 * 4].view(4, 27, 16, 16), p[27 * 16 * 16 * 4:].view(4, 16)


def _net(x, W, b):
    """Refined F [n, 512] of haloed blocks x [n, 2000], float64."""
    n = x.shape[0]
    x = x.double().view(n, 2, 10, 10, 10)
    centre = x[:, 0, 1:9, 1:9, 1:9].reshape(n, 512)
    a = x.permute(0, 2, 3, 4, 1)
    for layer in range(4):
        ch = a.shape[-1]
        y = b[layer].expand(n * 512, 16)
        for tap in range(27):
            dz, dy, dx = tap // 9, tap // 3 % 3, tap % 3
            p = a[:, dz:dz + 8, dy:dy + 8, dx:dx + 8].reshape(n * 512, ch)
            y = y + p @ W[layer, tap, :, :ch].T
        if layer < 3:
            a = torch.nn.functional.pad(torch.relu(y).view(n, 8, 8, 8, 16), (0, 0, 1, 1, 1, 1, 1, 1))
    return torch.clamp(centre + y[:, 0].reshape(n, 512), -1, 1)


def _exact_train(c, seed):
    flat = torch.from_numpy(_refiner_params(seed).astype(np.float64)).cuda().requires_grad_(True)
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    losses = []
    for i in range(c["steps"]):
        x, target, mask = _blocks(c["blocks"], seed + 1000 * i)
        F = _net(x, flat[:27 * 1024].view(4, 27, 16, 16), flat[27 * 1024:].view(4, 16))
        loss = (((F - target.double()) ** 2) * mask.double()).sum() / max(1, int(mask.sum()))
        losses.append(loss.detach())
        g, = torch.autograd.grad(loss, flat)
        with torch.no_grad():
            m = 0.9 * m + 0.1 * g
            v = 0.999 * v + 0.001 * g * g
            flat -= 1e-3 * (m / (1 - 0.9 ** (i + 1))) / (torch.sqrt(v / (1 - 0.999 ** (i + 1))) + 1e-8)
    return {"losses": torch.stack(losses), "params": flat.detach()}


def _exact_track(c, seed):
    (fx, fy, cx, cy, W, H), depth, V, N, T_ref = _track_inputs(c, seed)
    depth, V, N = depth.double(), V.double().view(-1, 4), N.double().view(-1, 4)
    Tr = torch.from_numpy(T_ref).cuda()
    T = Tr.clone()
    steps = 0
    system = None
    for level, iters, dist in ((2, 10, 0.1), (1, 6, 0.05), (0, 4, 0.02)):
        q = 1 << level
        d = depth[::q, ::q]
        h, w = d.shape
        v, u = torch.meshgrid(torch.arange(h, device="cuda"), torch.arange(w, device="cuda"), indexing="ij")
        p = torch.stack([d * (u - cx / q) / (fx / q), d * (v - cy / q) / (fy / q), d], -1).reshape(-1, 3)
        p = p[p[:, 2] > 0]
        for _ in range(iters):
            P = p @ T[:3, :3].T + T[:3, 3]
            X = (P - Tr[:3, 3]) @ Tr[:3, :3]
            x = torch.floor(fx * X[:, 0] / X[:, 2] + cx + 0.5)
            y = torch.floor(fy * X[:, 1] / X[:, 2] + cy + 0.5)
            ok = (X[:, 2] > 0) & (x >= 0) & (x <= W - 1) & (y >= 0) & (y <= H - 1)
            at = torch.where(ok, y * W + x, torch.zeros_like(x)).long()
            vv, nn = V[at], N[at]
            e = P - vv[:, :3]
            ok = ok & (vv[:, 3] > 0) & (nn[:, 3] > 0) & ((e * e).sum(1).sqrt() <= dist)
            P, n_, e = P[ok], nn[ok, :3], e[ok]
            r = (e * n_).sum(1)
            J = torch.cat([torch.linalg.cross(P, n_), n_], 1)
            system = (int(ok.sum()), float((r * r).sum()))
            if system[0] < 100:
                break
            xi = torch.linalg.solve(J.T @ J, -(J.T @ r))
            wx = xi[:3]
            K = torch.zeros((4, 4), dtype=torch.float64, device="cuda")
            K[0, 1], K[0, 2], K[1, 2] = -wx[2], wx[1], -wx[0]
            K = K - K.T
            M = torch.matrix_exp(K)
            M[:3, 3] = xi[3:]
            T = M @ T
            steps += 1
    return {"pose": T, "pairs": system[0], "rms": math.sqrt(system[1] / max(1, system[0])), "steps": steps}


def exact(case, seed):
    kind = case["kind"]
    if kind == "forward":
        x = _blocks(case["blocks"], seed)[0]
        W, b = _unpack(_refiner_params(seed))
        return torch.cat([_net(y, W, b) for y in x.split(512)])
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "track":
        return _exact_track(case, seed)
    if kind == "export":
        coords, F, Wt, _ = _terrain(case, seed)
        at = np.lexsort((coords[:, 2], coords[:, 1], coords[:, 0]))
        return coords[at], F[at].astype(np.float64), Wt[at].astype(np.float64)
    return None   # maps and voxels decided by a walk or a march through the grid, sample by sample
