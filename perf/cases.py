"""Timed work of the renderer: what a user of the framework has it do, through
its public entry points (paper_2603_15186_amd.hgs.Renderer and .lod).

Kinds of cases (the dict's "kind"):
  flat    render of a flat Gaussian box (no hierarchy), SH degree 0
  render  render of a hierarchical floor plan, SH degree 3: threshold cut,
          learned cut, or threshold cut with level-of-detail blending
  fit     one step of scene reconstruction: render and backward pass
  slice   collision map of a floor (GS-slices) and collision checks on it
  nav     shortest-path planning: navigable map, distance fields, trajectories
  train   one training step of the learned cut's network
  eval    PSNR of a learned cut over poses (calibration and evaluation)

Scenes play the part of weights: one floor plan per leaf count, loaded once
into a renderer that all passes of a case share, as a simulator keeps it.
Poses, image gradients, queries, batches and references come from the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2603_15186_amd import hgs, lod
from paper_2603_15186_amd.synth import FreeSpace, make_random_box, mlp_init, random_poses, yaw_camera
from paper_2603_15186_amd.synth import workloads

PLAN_CELL = dict(x0=-0.1, y0=-0.1, cell=0.05, nx=404, ny=304)
ROBOT_RADIUS = 0.25


def listed():
    return [
        # the smallest call: the 20,000-Gaussian box at 256 x 256, one blocking render
        dict(name="box-256", kind="flat", gaussians=20000, views=1, width=256, height=256, graph=False),
        # one robot camera in a closed loop: the policy waits for every frame
        dict(name="robot-480p", kind="render", leaves=2000000, sizes="1@640x480", mode="threshold", tau=1.0,
             blend=False, graph=False),
        # a stream of single 720p frames, the render replayed from a graph
        dict(name="frame-720p", kind="render", leaves=2000000, sizes="1@1280x720", mode="learned", tau=1.0,
             blend=False, graph=True),
        # the headline batch: 50 robots' 720p views with the learned cut
        dict(name="batch50-720p", kind="render", leaves=2000000, sizes="50@1280x720", mode="learned", tau=1.0,
             blend=False, graph=True),
        # a large batch of mixed resolutions (more views than one group)
        dict(name="mixed-96", kind="render", leaves=2000000, sizes="48@320x240,36@640x480,12@1280x720",
             mode="threshold", tau=2.0, blend=False, graph=False),
        # video of a few cameras with smooth level transitions, ragged sizes
        dict(name="blend-ragged", kind="render", leaves=700003, sizes="5@1001x563", mode="threshold", tau=2.0,
             blend=True, graph=False),
        # reconstruction on a few posed photographs per step
        dict(name="fit-plan", kind="fit", leaves=700003, views=4, width=640, height=480, keep=True),
        # reconstruction of a small object, one odd-sized photograph per step
        dict(name="fit-box", kind="fit", leaves=0, views=1, width=253, height=191, keep=False),
        # the collision map of a floor, rebuilt when the scene changes, and checks of many robots on it
        dict(name="slice-floor", kind="slice", leaves=2000000, planes=15, queries=100000),
        # expert trajectories: 9 goals with 200 starts each
        dict(name="plan-9x200", kind="nav", leaves=200001, goals=9, per_goal=200),
        # training of the learned cut: the trainer's batch of 4,096 candidates
        dict(name="train-4096", kind="train", batch=4096),
        # calibration of the learned cut: one chunk of 16 poses against their references
        dict(name="eval-16", kind="eval", leaves=700003, views=16, width=1280, height=720),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["flat", "render", "render", "render", "fit", "slice", "nav", "train", "eval"])
    leaves = rng.choice([50000, 200001, 700003])
    if kind == "flat":
        return dict(kind=kind, gaussians=_log_int(rng, 1000, 200000), views=_log_int(rng, 1, 8),
                    width=_log_int(rng, 64, 640), height=_log_int(rng, 64, 480), graph=rng.random() < 0.5)
    if kind == "render":
        views = _log_int(rng, 1, 100)
        width = _log_int(rng, 160, 1920)
        width = min(width, int(math.sqrt(30e6 / views * 16 / 9)))
        mode = rng.choice(["threshold", "threshold", "learned"])
        return dict(kind=kind, leaves=leaves, sizes=f"{views}@{width}x{max(90, width * 9 // 16 + rng.randrange(-3, 4))}",
                    mode=mode, tau=round(math.exp(rng.uniform(0.0, math.log(8.0))), 3) if mode == "threshold" else 1.0,
                    blend=mode == "threshold" and rng.random() < 0.25, graph=rng.random() < 0.5)
    if kind == "fit":
        return dict(kind=kind, leaves=rng.choice([0, leaves]), views=_log_int(rng, 1, 8), width=_log_int(rng, 100, 800),
                    height=_log_int(rng, 75, 600), keep=rng.random() < 0.7)
    if kind == "slice":
        return dict(kind=kind, leaves=leaves, planes=rng.randrange(1, 31), queries=_log_int(rng, 100, 1000000))
    if kind == "nav":
        return dict(kind=kind, leaves=rng.choice([50000, 200001]), goals=rng.randrange(1, 17), per_goal=_log_int(rng, 10, 500))
    if kind == "train":
        return dict(kind=kind, batch=_log_int(rng, 256, 65536))
    return dict(kind=kind, leaves=leaves, views=_log_int(rng, 1, 16), width=_log_int(rng, 160, 1280),
                height=_log_int(rng, 120, 720))


# ------------------------------------------------------------------ inputs

@functools.lru_cache(maxsize=3)
def _plan(leaves):
    """Floor plan of 20 x 15 m with `leaves` leaf Gaussians, and its free space."""
    scene, plan = workloads.floorplan_scene(leaves, (20.0, 15.0), 1, seed=1, use_cache=False)
    return scene, plan, FreeSpace(plan, 0)


@functools.lru_cache(maxsize=2)
def _box(n):
    return make_random_box(n, seed=0)


def _scene(case):
    if case["kind"] == "flat":
        return _box(case["gaussians"])
    return _plan(case["leaves"])[0] if case.get("leaves") else _box(20000)


_kept = {}


def _renderer(case, **options):
    """The program's renderer for a case: scene loaded, options set.  Every
    state of the case shares it; the renderer of the case before is let go."""
    key = (case["kind"], case.get("leaves"), case.get("gaussians"), case.get("mode"), case.get("tau"),
           case.get("views"), case.get("sizes"), case.get("width"), case.get("height"), tuple(sorted(options.items())))
    r = _kept.get(key)
    if r is None:
        _kept.clear()
        r = hgs.Renderer(0)
        r.load_scene(_scene(case))
        for name, value in options.items():
            r.set_option(getattr(hgs, name), value)
        _kept[key] = r
    return r


def _sizes(case):
    out = []
    for part in case["sizes"].split(","):
        n, wh = part.split("@")
        w, h = wh.split("x")
        out += [(int(w), int(h))] * int(n)
    return out


def _plan_cams(leaves, sizes, seed):
    """Random robot poses (0.3 to 1.5 m high, any heading); f = 900 px at a width of 1280."""
    pos, yaw = random_poses(_plan(leaves)[2], len(sizes), 1000 + seed, height=(0.3, 1.5))
    return [yaw_camera(w, h, 900.0 * w / 1280.0, p, y, bg=(0.1, 0.2, 0.3)) for (w, h), p, y in zip(sizes, pos, yaw)]


def _box_cams(n, w, h, seed):
    """Cameras about 3 m from the middle of the 4 x 4 x 3 m box, looking at it."""
    rng = np.random.default_rng(2000 + seed)
    cams = []
    for a in rng.uniform(0.0, 2.0 * math.pi, n):
        p = (2.0 - 3.0 * math.cos(a), 2.0 - 3.0 * math.sin(a), rng.uniform(1.2, 1.8))
        cams.append(yaw_camera(w, h, float(max(w, h)), p, a, bg=(0.1, 0.2, 0.3)))
    return cams


def _cams(case, seed):
    if case["kind"] == "flat":
        return _box_cams(case["views"], case["width"], case["height"], seed)
    if case["kind"] == "render":
        return _plan_cams(case["leaves"], _sizes(case), seed)
    size = [(case["width"], case["height"])] * case["views"]
    return _plan_cams(case["leaves"], size, seed) if case.get("leaves") else \
        _box_cams(case["views"], case["width"], case["height"], seed)


def _flat_outputs(cams):
    """One rgb, one depth and one alpha buffer for all views, and each view's part of them."""
    px = [c.width * c.height for c in cams]
    total = sum(px)
    rgb = torch.empty(3 * total, dtype=torch.float32, device="cuda")
    depth = torch.empty(total, dtype=torch.float32, device="cuda")
    alpha = torch.empty(total, dtype=torch.float32, device="cuda")
    outs, o = [], 0
    for c, n in zip(cams, px):
        outs.append((rgb[3 * o:3 * (o + n)].view(3, c.height, c.width), depth[o:o + n].view(c.height, c.width),
                     alpha[o:o + n].view(c.height, c.width)))
        o += n
    return dict(rgb=rgb, depth=depth, alpha=alpha), outs


def _image_grads(case, seed):
    """Image gradients as a photometric loss gives them: of both signs, about 1 / pixels."""
    g = torch.Generator(device="cuda").manual_seed(3000 + seed)
    h, w = case["height"], case["width"]
    f = 1.0 / (w * h)
    return [(torch.randn((3, h, w), generator=g, device="cuda") * f, torch.randn((h, w), generator=g, device="cuda") * 0.1 * f,
             torch.randn((h, w), generator=g, device="cuda") * f) for _ in range(case["views"])]


def _train_batch(case, seed):
    """Candidate features in their usual ranges, rare labels balanced by the
    sampler, the network in the middle of its training."""
    rng = np.random.default_rng(4000 + seed)
    n = case["batch"]
    f = np.stack([rng.normal(2.5, 0.8, n), rng.normal(1.0, 0.6, n), rng.uniform(0.3, 0.99, n), rng.integers(1, 9, n),
                  rng.exponential(0.01, n), rng.uniform(0.0, 1.0, n), rng.integers(3, 8, n), rng.normal(3.2, 0.8, n)], axis=1)
    score = 0.8 * (f[:, 0] - 2.5) + 20.0 * (f[:, 4] - 0.01) + rng.normal(0.0, 0.5, n)
    y = (score > np.median(score)).astype(np.float32)
    mean, std = f.mean(0).astype(np.float32), np.maximum(f.std(0), 1e-6).astype(np.float32)
    master = (mlp_init(seed) + rng.normal(0.0, 0.02, hgs.N_MLP_PARAMS)).astype(np.float32)
    m = rng.normal(0.0, 1e-3, hgs.N_MLP_PARAMS).astype(np.float32)
    v = rng.uniform(1e-6, 1e-5, hgs.N_MLP_PARAMS).astype(np.float32)
    w = torch.from_numpy(master).to(torch.bfloat16)
    return f.astype(np.float32), y, mean, std, master, w, m, v


def _floor_queries(n, seed):
    rng = np.random.default_rng(5000 + seed)
    return rng.uniform([-0.1, -0.1], [20.1, 15.1], size=(n, 2))


@functools.lru_cache(maxsize=1)
def _model():
    return lod.LodModel.load(lod.default_model_path())


# ------------------------------------------------------------------ states

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("flat", "render"):
        cams = _cams(case, seed)
        options = {}
        if case["graph"]:
            options.update(HGS_OPT_USE_GRAPH=1, HGS_OPT_SYNC_CHECK=0)
        if case.get("blend"):
            options.update(HGS_OPT_LOD_BLEND=1)
        if kind == "render" and len(cams) > 1:      # the tuned launch plan of batches
            options.update(HGS_OPT_PIXELS_PER_THREAD=2, HGS_OPT_BATCH_DEPTH=128)
        r = _renderer(case, **options)
        flat, outs = _flat_outputs(cams)
        if kind == "render":
            mode = {"threshold": hgs.HGS_LOD_THRESHOLD, "learned": hgs.HGS_LOD_LEARNED}[case["mode"]]
            if mode == hgs.HGS_LOD_LEARNED:
                _model().install(r)
            r.set_lod(mode, case["tau"])
        if case["graph"]:                           # buffers settled before asynchronous renders
            r.set_option(hgs.HGS_OPT_SYNC_CHECK, 1)
            r.set_cameras(cams)
            r.render(outs)
            r.set_option(hgs.HGS_OPT_SYNC_CHECK, 0)
        return dict(kind=kind, r=r, cams=cams, outs=outs, flat=flat)
    if kind == "fit":
        options = dict(HGS_OPT_KEEP_STATE=1) if case["keep"] else {}
        r = _renderer(case, **options)
        cams = _cams(case, seed)
        flat, outs = _flat_outputs(cams)
        n, K = r.scene_n, (r.scene_sh_degree + 1) ** 2
        shapes = dict(means=(n, 3), scales=(n, 3), quats=(n, 4), opacity=(n,), sh=(n, K, 3))
        grads = {k: torch.zeros(s, dtype=torch.float32, device="cuda") for k, s in shapes.items()}
        return dict(kind=kind, r=r, cams=cams, outs=outs, flat=flat, dimg=_image_grads(case, seed), grads=grads)
    if kind == "slice":
        r = _renderer(case)
        rng = np.random.default_rng(6000 + seed)
        heights = np.linspace(0.1, 1.5, case["planes"]) + rng.uniform(-0.05, 0.05)
        return dict(kind=kind, r=r, heights=heights.astype(np.float32),
                    xy=torch.from_numpy(_floor_queries(case["queries"], seed)).cuda())
    if kind == "nav":
        r = _renderer(case)
        rng = np.random.default_rng(7000 + seed)
        heights = np.arange(0.1, 1.55, 0.1) + rng.uniform(-0.05, 0.05)
        _, occ = r.slice_occupancy(heights=heights, occ=False, **PLAN_CELL)
        nav = r.navigable_map(occ, PLAN_CELL["x0"], PLAN_CELL["y0"], PLAN_CELL["cell"], ROBOT_RADIUS).cpu().numpy()
        goals, starts, slots = workloads.nav_queries(nav, case["goals"], case["per_goal"], seed=seed)
        return dict(kind=kind, r=r, occ=occ, goals=goals, starts=torch.from_numpy(starts).cuda(),
                    slots=torch.from_numpy(slots).cuda())
    if kind == "train":
        f, y, mean, std, master, w, m, v = _train_batch(case, seed)
        if "train" not in _kept:
            _kept.clear()
            _kept["train"] = hgs.Renderer(0)
        d = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
        return dict(kind=kind, r=_kept["train"], f=d(f), y=d(y), mean=mean, std=std, master=d(master),
                    w=w.view(torch.int16).cuda(), m=d(m), v=d(v), step=100,
                    grad=torch.empty(hgs.N_MLP_PARAMS, dtype=torch.float32, device="cuda"),
                    loss=torch.empty(1, dtype=torch.float32, device="cuda"))
    if kind == "eval":
        r = _renderer(case)
        cams = _cams(case, seed)
        g = torch.Generator(device="cuda").manual_seed(8000 + seed)
        refs = []
        for img in lod.render_rgb(r, cams, hgs.HGS_LOD_THRESHOLD, 1.0):
            refs.append((img + 0.03 * torch.randn(img.shape, generator=g, device="cuda")).clamp(0.0, 1.0))
        return dict(kind=kind, r=r, cams=cams, refs=refs)
    raise ValueError(kind)


def run(s):
    kind, r = s["kind"], s["r"]
    if kind in ("flat", "render"):
        r.set_cameras(s["cams"])
        r.render(s["outs"])
        return s["flat"]
    if kind == "fit":
        for g in s["grads"].values():
            g.zero_()
        r.set_cameras(s["cams"])
        r.render(s["outs"])
        r.backward(s["dimg"], out=s["grads"])
        return dict(s["grads"], **s["flat"])
    if kind == "slice":
        occ, m = r.slice_occupancy(heights=s["heights"], **PLAN_CELL)
        hits = r.disc_collision(m, PLAN_CELL["x0"], PLAN_CELL["y0"], PLAN_CELL["cell"], s["xy"], ROBOT_RADIUS)
        return occ, m, hits
    if kind == "nav":
        cap = 2048
        nav = r.navigable_map(s["occ"], PLAN_CELL["x0"], PLAN_CELL["y0"], PLAN_CELL["cell"], ROBOT_RADIUS)
        dist, _ = r.distance_fields(nav, s["goals"])
        paths, lens = r.trace_paths(nav, dist, s["starts"], s["slots"], cap)
        # cells past a trajectory's end are not written: padded with -1
        paths = paths.masked_fill(torch.arange(cap, device="cuda") >= lens[:, None], -1)
        return nav, dist, paths, lens
    if kind == "train":
        s["step"] += 1
        r.mlp_train_step(s["f"], s["y"], s["mean"], s["std"], s["master"], s["w"], s["m"], s["v"], s["step"], 3e-3,
                         grad_out=s["grad"], loss_out=s["loss"])
        return dict(grad=s["grad"], loss=s["loss"], master=s["master"], m=s["m"], v=s["v"], w=s["w"].view(torch.bfloat16))
    mean, cut, ps = lod.evaluate(r, s["cams"], s["refs"], _model())
    return dict(mean=mean, cut=cut, psnr=ps)


def work(case):
    """Bytes and FP32 operations one pass cannot do without.  Rendering: the
    cut's Gaussians once per batch (236 B each at SH degree 3; a view's cut
    is about a fifth of the leaves at tau = 1), 20 B written per pixel, 21
    operations for each of about 27 blended Gaussians per pixel."""
    kind = case["kind"]
    if kind in ("flat", "render", "fit", "eval"):
        if kind == "render":
            px, views = sum(w * h for w, h in _sizes(case)), len(_sizes(case))
        else:
            px, views = case["views"] * case["width"] * case["height"], case["views"]
        if case.get("leaves"):
            read = case["leaves"] * 240.0 * min(1.0, 0.2 * views / case.get("tau", 1.0))
        else:
            read = case.get("gaussians", 20000) * 56.0
        w = dict(bytes=read + 20.0 * px, flops=21.0 * 27.0 * px)
        if kind == "fit":            # gradients in and out, the reverse walk
            nodes = case["leaves"] * 8 / 7 * 236.0 if case["leaves"] else 20000 * 56.0
            w = dict(bytes=w["bytes"] + 20.0 * px + nodes, flops=w["flops"] + 64.0 * 27.0 * px)
        if kind == "eval":
            w = dict(bytes=w["bytes"] + 24.0 * px, flops=w["flops"] + 9.0 * px)
        return w
    cells = PLAN_CELL["nx"] * PLAN_CELL["ny"]
    if kind == "slice":
        return dict(bytes=case["leaves"] * 52.0 + (case["planes"] + 1.0) * cells + 17.0 * case["queries"],
                    flops=case["leaves"] * 60.0 + case["queries"] * 600.0)
    if kind == "nav":
        return dict(bytes=2.0 * cells + case["goals"] * cells * 17.0 + case["goals"] * case["per_goal"] * 800.0,
                    flops=case["goals"] * cells * 24.0)
    n = case["batch"]
    return dict(bytes=36.0 * n + 1377 * 30.0, flops=6.0 * 1377 * n)


# ------------------------------------------------- the same values in 64 bits

_C99, _C255, _C1E4 = (float(np.float32(x)) for x in (0.99, 1.0 / 255.0, 1e-4))


def _t(a):
    return torch.as_tensor(np.asarray(a, np.float64), device="cuda")


def _exact_cut(scene, cam, tau):
    """Threshold cut: drop a node whose sphere lies outside the frustum, keep
    leaves and nodes whose projected size is at most tau, refine the others."""
    R, o = np.asarray(cam.R, np.float64), np.asarray(np.float32(cam.position), np.float64)
    fx, fy, cx, cy, W, H = cam.fx, cam.fy, cam.cx, cam.cy, cam.width, cam.height
    front = np.arange(int(scene.level_offset[1]))
    kept = []
    while front.size:
        b = scene.bound[front].astype(np.float64)
        d, r = b[:, :3] - o, b[:, 3]
        p = d @ R.T
        inside = p[:, 2] + r >= cam.znear
        for e, n2 in ((fx * p[:, 0] + cx * p[:, 2], fx * fx + cx * cx),
                      (-(fx * p[:, 0] + (cx - W) * p[:, 2]), fx * fx + (cx - W) ** 2),
                      (fy * p[:, 1] + cy * p[:, 2], fy * fy + cy * cy),
                      (-(fy * p[:, 1] + (cy - H) * p[:, 2]), fy * fy + (cy - H) ** 2)):
            inside &= ~((e < 0) & (e * e > r * r * n2))
        front, d, r = front[inside], d[inside], r[inside]
        nc = scene.child_count[front]
        refine = (nc > 0) & ((2.0 * max(fx, fy) * r) ** 2 > tau * tau * (d * d).sum(1))
        kept.append(front[~refine])
        up = front[refine]
        front = (scene.first_child[up][:, None] + np.arange(nc.max() if nc.size else 0))
        front = front[np.arange(front.shape[1]) < scene.child_count[up][:, None]] if up.size else up
    return np.concatenate(kept)


def _sh_basis(d, deg):
    x, y, z = d.unbind(1)
    Y = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if deg >= 1:
        c = math.sqrt(3.0 / (4.0 * math.pi))
        Y += [-c * y, c * z, -c * x]
    if deg >= 2:
        a, b = 0.5 * math.sqrt(15.0 / math.pi), 0.25 * math.sqrt(5.0 / math.pi)
        Y += [a * x * y, -a * y * z, b * (3 * z * z - 1), -a * x * z, 0.5 * a * (x * x - y * y)]
    if deg >= 3:
        a, b = 0.25 * math.sqrt(35.0 / (2.0 * math.pi)), 0.5 * math.sqrt(105.0 / math.pi)
        c, e = 0.25 * math.sqrt(21.0 / (2.0 * math.pi)), 0.25 * math.sqrt(7.0 / math.pi)
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (5 * z * z - 1), e * z * (5 * z * z - 3),
              -c * x * (5 * z * z - 1), 0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


def _exact_view(p, deg, cam, grads=None):
    """Image of the Gaussians p (float64 tensors means, scales, quats,
    opacity, sh) for one camera: (rgb, depth, alpha).  With grads (the
    image's gradients), p's .grad are added to."""
    R, o = _t(cam.R), _t(np.float32(cam.position))
    W, H, fx, fy, cx, cy = cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy
    d = p["means"] - o
    front = torch.nonzero((d @ R.T)[:, 2].detach() > cam.znear)[:, 0]
    d = d[front]
    t = d @ R.T
    tx, ty, tz = t.unbind(1)
    u, v = fx * tx / tz + cx, fy * ty / tz + cy
    xr = (tx / tz).clamp((-cx - 0.15 * W) / fx, (W - cx + 0.15 * W) / fx)
    yr = (ty / tz).clamp((-cy - 0.15 * H) / fy, (H - cy + 0.15 * H) / fy)
    M = torch.stack([fx / tz[:, None] * (R[0] - xr[:, None] * R[2]), fy / tz[:, None] * (R[1] - yr[:, None] * R[2])], 1)
    q = p["quats"][front]
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                      1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                      1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
    T = (M @ Rq.contiguous()) * p["scales"][front][:, None, :]
    s00, s11 = (T[:, 0] ** 2).sum(1) + 0.3, (T[:, 1] ** 2).sum(1) + 0.3
    s01 = (T[:, 0] * T[:, 1]).sum(1)
    det = s00 * s11 - s01 * s01
    A, B, C = s11 / det, -s01 / det, s00 / det
    Y = _sh_basis(d / d.norm(dim=1, keepdim=True), deg)
    col = ((p["sh"][front] * Y[:, :, None]).sum(1) + 0.5).clamp(0.0, 1.0)
    vals = [u, v, A, B, C, p["opacity"][front], tz, col]
    order = torch.sort(tz.detach().float(), stable=True)[1]
    ex, ey = torch.sqrt(9.01 * s00.detach())[order], torch.sqrt(9.01 * s11.detach())[order]
    leaf = [a.detach()[order].requires_grad_(grads is not None) for a in vals]
    uo, vo = leaf[0].detach(), leaf[1].detach()
    x_lo, x_hi, y_lo, y_hi = uo - ex, uo + ex, vo - ey, vo + ey
    img = torch.zeros((5, H, W), dtype=torch.float64, device="cuda")
    bg = _t(np.float32(cam.bg))
    for y0 in range(0, H, 16):
        y1 = min(y0 + 16, H)
        row = torch.nonzero((y_hi >= y0) & (y_lo <= y1))[:, 0]
        rx_lo, rx_hi = x_lo[row], x_hi[row]
        for x0 in range(0, W, 16):
            x1 = min(x0 + 16, W)
            ids = row[(rx_hi >= x0) & (rx_lo <= x1)]
            iu, iv, ia, ib, ic, io, iz, icol = (a[ids] for a in leaf)
            gy, gx = torch.meshgrid(torch.arange(y0, y1, device="cuda") + 0.5, torch.arange(x0, x1, device="cuda") + 0.5,
                                    indexing="ij")
            dx, dy = gx.reshape(-1, 1).double() - iu, gy.reshape(-1, 1).double() - iv
            qq = ia * dx * dx + 2 * ib * dx * dy + ic * dy * dy
            al = (io * torch.exp(-0.5 * qq)).clamp(max=_C99)
            al = torch.where((qq <= 9.0) & (al >= _C255), al, torch.zeros_like(al))
            P = torch.cumprod(1.0 - al, 1)
            keep = P >= _C1E4
            before = torch.cat([torch.ones_like(P[:, :1]), P[:, :-1]], 1)
            wgt = torch.where(keep, al * before, torch.zeros_like(al))
            tot = wgt.sum(1)
            rgb = wgt @ icol + (1.0 - tot)[:, None] * bg
            out = torch.cat([rgb, (wgt @ iz)[:, None], tot[:, None]], 1)
            img[:, y0:y1, x0:x1] = out.detach().T.reshape(5, y1 - y0, x1 - x0)
            if grads is not None:
                out.backward(grads[:, y0:y1, x0:x1].reshape(5, -1).T)
    if grads is not None:
        back = [torch.empty_like(a.grad).index_copy_(0, order, a.grad) for a in leaf]
        torch.autograd.backward(vals, back)
    return img[:3], img[3], img[4]


def _exact_images(case, seed, grads=None):
    scene, cams = _scene(case), _cams(case, seed)
    flat, outs = _flat_outputs(cams)
    flat = {k: v.double() for k, v in flat.items()}
    acc = None
    if grads is not None:
        acc = {k: torch.zeros(np.shape(getattr(scene, k)), dtype=torch.float64, device="cuda")
               for k in ("means", "scales", "quats", "opacity", "sh")}
    o = 0
    for i, c in enumerate(cams):
        ids = np.arange(scene.n) if scene.parent is None else _exact_cut(scene, c, case.get("tau", 1.0))
        p = {k: _t(getattr(scene, k)[ids]).requires_grad_(grads is not None)
             for k in ("means", "scales", "quats", "opacity", "sh")}
        up = None if grads is None else torch.cat([grads[i][0], grads[i][1][None], grads[i][2][None]]).double()
        rgb, dep, alp = _exact_view(p, scene.sh_degree, c, up)
        n = c.width * c.height
        flat["rgb"][3 * o:3 * (o + n)] = rgb.reshape(-1)
        flat["depth"][o:o + n] = dep.reshape(-1)
        flat["alpha"][o:o + n] = alp.reshape(-1)
        o += n
        if grads is not None:
            at = torch.as_tensor(ids, device="cuda")
            for k, a in acc.items():
                a.index_add_(0, at, p[k].grad)
    return flat if acc is None else dict(acc, **flat)


def _exact_train(case, seed):
    f, y, mean, std, master, w, m, v = _train_batch(case, seed)
    x = (_t(f) - _t(mean)) / _t(std)
    yy = _t(y)
    p = w.double().cuda().requires_grad_(True)
    h = torch.relu(x @ p[:256].view(32, 8).T + p[256:288])
    h = torch.relu(h @ p[288:1312].view(32, 32).T + p[1312:1344])
    z = h @ p[1344:1376] + p[1376]
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, yy)
    loss.backward()
    g, step = p.grad, 101
    m1, v1 = 0.9 * _t(m) + 0.1 * g, 0.999 * _t(v) + 0.001 * g * g
    new = _t(master) - 3e-3 * (m1 / (1 - 0.9 ** step)) / (torch.sqrt(v1 / (1 - 0.999 ** step)) + 1e-8)
    return dict(grad=g, loss=loss.detach().reshape(1), master=new, m=m1, v=v1, w=None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "fit":
        work_px = case["views"] * case["width"] * case["height"]
        return _exact_images(case, seed, _image_grads(case, seed)) if work_px <= 320000 else None
    if kind == "flat" or (kind == "render" and case["mode"] == "threshold" and not case["blend"]):
        sizes = _sizes(case) if kind == "render" else [(case["width"], case["height"])] * case["views"]
        return _exact_images(case, seed) if sum(w * h for w, h in sizes) <= 1500000 else None
    return None
