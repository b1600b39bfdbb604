"""Workloads of the Quantile Rendering library, as its users run them.

Every case is one pass through the public entry points on inputs that are drawn from a seed on the GPU:
``prepare`` makes what a program has in hand before the call, ``run`` makes the call, ``exact`` gives the same
outputs in 64-bit arithmetic by plain torch, and ``work`` the bytes and operations the pass cannot do without.

Kinds of case:

* ``frame``   one view: projection, binning, render (an interactive viewer or a query on one picture)
* ``batch``   many views of one scene: the same three steps in one launch sequence each, then one batched launch
* ``rgb``     the batch with view-dependent colours instead of stored features
* ``train``   forward and backward of one view through the autograd function, records and lists given
* ``views``   forward and backward of many views of several scenes in one launch each, gradients cleared first
* ``devox``   per-Gaussian features from voxel predictions, forward and backward
* ``encode``  storage encoding of a feature table
"""

import dataclasses
import math
import random

import numpy as np
import torch

import paper_2512_20927_amd as qr
from paper_2512_20927_amd import _lib as L
from paper_2512_20927_amd.batched import BatchedDense, BatchedQuantile

TILE = 16
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}
RULE = {"quantile": L.QR_SELECT_QUANTILE, "stratified": L.QR_SELECT_STRATIFIED, "topk": L.QR_SELECT_TOPK,
        "dense": L.QR_SELECT_QUANTILE}


def listed():
    room = dict(scene="room", n=200_000, width=640, height=480)
    return [
        # the smallest call: a few launches on a 64 x 64 picture, where latency is everything (tests, previews)
        dict(name="frame_tiny", kind="frame", scene="tiny", n=1000, width=64, height=64, dim=16, store="f32",
             rule="quantile", K=8),
        # an ordinary single picture of ragged size with a compressed feature table and the Top-K sampler
        dict(name="frame_ragged", kind="frame", scene="room", n=60_000, width=333, height=251, dim=48, store="bf16",
             rule="topk", K=5),
        # the flagship: 16 poses of a room, 512 float32 features, K = 8
        dict(name="batch_room", kind="batch", dim=512, store="f32", rule="quantile", K=8, views=16, order="heavy",
             per_cu=3, **room),
        # the renderer it is compared with, over the same items
        dict(name="batch_dense", kind="batch", dim=512, store="f32", rule="dense", K=0, views=16, order="natural",
             per_cu=2, **room),
        # a large scene at a ScanNet frame size (ragged tiles), bfloat16 table, more quantiles, default launch shape
        dict(name="batch_large", kind="batch", scene="room", n=1_000_000, width=1296, height=968, dim=512,
             store="bf16", rule="quantile", K=16, views=4, order="natural", per_cu=0),
        # colours from spherical harmonics: narrow rows, where everything before the render counts
        dict(name="rgb_room", kind="rgb", dim=16, store="f32", rule="quantile", K=8, views=16, order="heavy",
             per_cu=3, degree=3, **room),
        # a training step through the renderer: 500k Gaussians, bfloat16 storage
        dict(name="train_quantile", kind="train", scene="room", n=500_000, width=640, height=480, dim=512,
             store="bf16", rule="quantile", K=8),
        # the same at the K that the method is trained with, float32 table
        dict(name="train_k40", kind="train", dim=512, store="f32", rule="quantile", K=40, **room),
        # a training step through the dense blend
        dict(name="train_dense", kind="train", scene="room", n=500_000, width=640, height=480, dim=512, store="bf16",
             rule="dense", K=0),
        # batched training: eight views of two uneven scenes, e4m3 tables
        dict(name="train_views", kind="views", scene="room", n=300_000, scenes=2, views=4, width=1280, height=720,
             dim=512, store="fp8", rule="quantile", K=8, order="natural", per_cu=0),
        # the step that makes the feature table: 200k Gaussians covering 8 of 100k voxels each
        dict(name="devox_max", kind="devox", n=200_000, unique=100_000, slots=1_600_000, dim=512, reduce="max"),
        # encoding a table of a large scene for storage
        dict(name="encode_fp8", kind="encode", n=1_000_000, dim=512, store="fp8"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Gaussians, pixels a view, feature values a pass and K: from the smallest to the largest listed call
def draw(rng):
    kind = rng.choice(["frame", "frame", "batch", "batch", "rgb", "train", "train", "views", "devox", "encode"])
    if kind == "devox":
        n = _log(rng, 1000, 200_000)
        return dict(kind=kind, n=n, unique=_log(rng, 200, 100_000), slots=n * rng.randint(1, 8) + rng.randint(0, 7),
                    dim=4 * rng.choice([3, 4, 9, 16, 25, 64, 96, 128]), reduce=rng.choice(["max", "mean"]))
    if kind == "encode":
        return dict(kind=kind, n=_log(rng, 1000, 1_000_000), dim=rng.choice([16, 48, 100, 256, 333, 512]),
                    store=rng.choice(["bf16", "fp8"]))
    width, height = _log(rng, 48, 1296), _log(rng, 48, 968)
    dim = 16 if kind == "rgb" else 16 * rng.choice([1, 2, 3, 4, 6, 8, 16, 24, 27, 32, 32, 32])
    rule = rng.choice({"frame": ["quantile", "quantile", "dense", "topk", "stratified"],
                       "batch": ["quantile", "quantile", "dense"], "rgb": ["quantile", "dense"],
                       "train": ["quantile", "dense"], "views": ["quantile"]}[kind])
    tiny = kind == "frame" and rng.random() < 0.3
    c = dict(kind=kind, scene="tiny" if tiny else "room", n=_log(rng, 300, 5000) if tiny else _log(rng, 20_000, 500_000),
             width=width, height=height, dim=dim, store="f32" if kind == "rgb" else rng.choice(["f32", "bf16", "fp8"]),
             rule=rule, K=0 if rule == "dense" else rng.choice([1, 4, 5, 8, 8, 16, 24, 40]))
    if kind in ("train", "views") and c["K"] == 1:  # one Gaussian a pixel has no geometric gradient to compare
        c["K"] = 2
    if kind in ("batch", "rgb", "views"):
        per_cu = rng.choice([0, 0, 2, 3])
        most = max(1, (2 if kind == "views" else 16) * 307_200 // (width * height))
        c.update(views=min(rng.randint(1, 16), most), order=rng.choice(["natural", "heavy"]), per_cu=per_cu)
    if kind == "rgb":
        c.update(degree=rng.choice([0, 1, 2, 3, 3]))
    if kind == "views":
        c.update(scenes=rng.randint(1, 3), n=min(c["n"], 300_000))
    return c


# ---- inputs ------------------------------------------------------------------------------------------

@dataclasses.dataclass
class Camera:
    """Pinhole camera with OpenCV axes: a point X is at R_cw X + t."""
    R_cw: np.ndarray
    t: np.ndarray
    fx: float
    fy: float
    cx: float
    cy: float
    width: int
    height: int
    z_near: float = 0.2


def _camera(c, rng):
    W, H = c["width"], c["height"]
    if c["scene"] == "tiny":  # looks at the origin from distance 3, 60 degrees of view over the shorter side
        f = (min(W, H) / 2) / math.tan(math.pi / 6)
        return Camera(np.eye(3, dtype=np.float32), np.array([rng.uniform(-.1, .1), rng.uniform(-.1, .1), 3], np.float32),
                      f, f, W / 2, H / 2, W, H)
    pos = np.array([rng.uniform(1, 5), rng.uniform(1, 5), rng.uniform(1, 2)])
    yaw, pitch = rng.uniform(0, 2 * math.pi), math.radians(rng.uniform(-15, 15))
    fwd = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
    right = np.cross(fwd, [0., 0., 1.])
    right /= np.linalg.norm(right)
    R = np.stack([right, np.cross(fwd, right), fwd])
    f = 577.0 * W / 640
    return Camera(R.astype(np.float32), (-R @ pos).astype(np.float32), f, f, W / 2, H / 2, W, H)


def _cameras(c, seed, count):
    rng = random.Random("cameras %d" % seed)
    return [_camera(c, rng) for _ in range(count)]


def _gen(seed):
    return torch.Generator("cuda").manual_seed(int(seed))


def _scene(c, n, g):
    """Means, scales, quaternions and opacities: 70 % of a room's Gaussians lie on its floor and walls."""
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    z = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    if c["scene"] == "tiny":
        means, lo, hi, o = r(n, 3) * 2 - 1, 0.01, 0.1, z(n)
    else:
        size = torch.tensor([6., 6., 3.], device="cuda")
        means = r(n, 3) * size
        k = int(0.7 * n)
        side = torch.multinomial(torch.tensor([36., 18., 18., 18., 18.], device="cuda"), k, True, generator=g)
        off = r(k) * 0.05
        for s, (axis, far) in enumerate([(2, 0), (0, 0), (0, 1), (1, 0), (1, 1)]):
            means[:k, axis] = torch.where(side == s, size[axis] - off if far else off, means[:k, axis])
        lo, hi, o = 0.005, 0.05, z(n) * 1.5 + 1
    scales = torch.exp(math.log(lo) + r(n, 3) * (math.log(hi) - math.log(lo)))
    q = z(n, 4)
    return means.contiguous(), scales, q / q.norm(dim=1, keepdim=True), torch.sigmoid(o)


def _features(c, n, g):
    """The float32 table (rows of length 1), and its stored form: (tensor, scale or None)."""
    f = torch.randn(n, c["dim"], generator=g, device="cuda")
    f /= f.norm(dim=1, keepdim=True)
    if c["store"] == "bf16":
        return f, (f.to(torch.bfloat16), None)
    if c["store"] == "fp8":
        scale = f.abs().amax(1) / 448
        return f, ((f / scale[:, None]).to(torch.float8_e4m3fn).view(torch.uint8), scale)
    return f, (f, None)


def _f32(x):
    return float(np.float32(x))


ALPHA_MIN, ALPHA_MAX, T_EPS, DILATION, GUARD = map(_f32, (1 / 255, 0.99, 1e-4, 0.3, 1.3))


def _project64(scene, cam):
    """EWA projection in 64 bits: means2d, conic and opacity, depth, tile rectangle and its tile count."""
    mu, s, q, o = (x.double() for x in scene)
    R = torch.tensor(cam.R_cw, device="cuda").double()
    t = torch.tensor(cam.t, device="cuda").double()
    fx, fy, cx, cy = map(_f32, (cam.fx, cam.fy, cam.cx, cam.cy))
    W, H = cam.width, cam.height
    p = mu @ R.T + t
    z = p[:, 2]
    u, v = fx * p[:, 0] / z + cx, fy * p[:, 1] / z + cy
    w_, x, y, zz = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rot = torch.stack([1 - 2 * (y * y + zz * zz), 2 * (x * y - w_ * zz), 2 * (x * zz + w_ * y),
                       2 * (x * y + w_ * zz), 1 - 2 * (x * x + zz * zz), 2 * (y * zz - w_ * x),
                       2 * (x * zz - w_ * y), 2 * (y * zz + w_ * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
    lx, ly = GUARD * 0.5 * W / fx, GUARD * 0.5 * H / fy
    xz, yz = (p[:, 0] / z).clamp(-lx, lx), (p[:, 1] / z).clamp(-ly, ly)
    J = torch.zeros(len(z), 2, 3, dtype=torch.float64, device="cuda")
    J[:, 0, 0], J[:, 0, 2], J[:, 1, 1], J[:, 1, 2] = fx / z, -fx * xz / z, fy / z, -fy * yz / z
    A = (J @ R) @ (rot * s[:, None, :])
    cxx = (A[:, 0] * A[:, 0]).sum(1) + DILATION
    cxy = (A[:, 0] * A[:, 1]).sum(1)
    cyy = (A[:, 1] * A[:, 1]).sum(1) + DILATION
    det = cxx * cyy - cxy * cxy
    conic = torch.stack([cyy / det, -cxy / det, cxx / det, o], 1)
    r2 = 2 * torch.log(o / ALPHA_MIN)
    hx, hy = (r2 * cxx).clamp(min=0).sqrt(), (r2 * cyy).clamp(min=0).sqrt()
    x0, x1 = (u - hx - 0.5).ceil().clamp(min=0), (u + hx - 0.5).floor().clamp(max=W - 1)
    y0, y1 = (v - hy - 0.5).ceil().clamp(min=0), (v + hy - 0.5).floor().clamp(max=H - 1)
    ok = (z > _f32(cam.z_near)) & (o >= ALPHA_MIN) & (x1 >= x0) & (y1 >= y0)
    box = torch.stack([x0, y0, x1, y1], 1)
    box = torch.where(ok[:, None], box, torch.zeros_like(box)).long() // TILE
    tiles = torch.where(ok, (box[:, 2] - box[:, 0] + 1) * (box[:, 3] - box[:, 1] + 1), torch.zeros_like(box[:, 0]))
    return torch.stack([u, v], 1), conic, z, box, tiles


def _lists(depth, box, tiles, W, H):
    """Tile offsets and Gaussian ids in (tile, depth, id) order."""
    order = torch.argsort(depth, stable=True)
    order = order[tiles[order] > 0]
    cnt = tiles[order]
    gid = torch.repeat_interleave(order, cnt)
    k = torch.arange(len(gid), device="cuda") - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
    b = box[gid]
    w = b[:, 2] - b[:, 0] + 1
    tx, ty = -(-W // TILE), -(-H // TILE)
    tile = (b[:, 1] + k // w) * tx + b[:, 0] + k % w
    tile, at = torch.sort(tile, stable=True)
    offsets = torch.searchsorted(tile, torch.arange(tx * ty + 1, device="cuda"))
    return offsets, gid[at]


def _records(c, scene, cam):
    """What projection and binning leave in hand for the renderer: float32 records and the lists."""
    m, co, z, box, tiles = _project64(scene, cam)
    offsets, gid = _lists(z, box, tiles, c["width"], c["height"])
    gid = gid if len(gid) else torch.zeros(1, dtype=torch.int64, device="cuda")
    return dict(m=m.float(), co=co.float(), offsets=offsets.int(), gid=gid.int())


def _params(c):
    return qr.RenderParams(selection=RULE[c["rule"]])


def _bins(r):
    return qr.Bins(r["offsets"], r["gid"], r["offsets"][-1:].clone(), r["gid"].numel())


def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "encode":
        return dict(c=c, f=_features(dict(c, store="f32"), c["n"], g)[0])
    if kind == "devox":
        return _prepare_devox(c, g)
    W, H, dim = c["width"], c["height"], c["dim"]
    if kind == "train":
        scene = _scene(c, c["n"], g)
        f, stored = _features(c, c["n"], g)
        r = _records(c, scene, _cameras(c, seed, 1)[0])
        return dict(c=c, prm=_params(c), f=f.requires_grad_(), bins=_bins(r),
                    storage=None if c["store"] == "f32" else stored,
                    m=r["m"].requires_grad_(), co=r["co"].requires_grad_(),
                    g=torch.randn(H, W, dim, generator=g, device="cuda"))
    if kind == "views":
        return _prepare_views(c, seed, g)
    scene = _scene(c, c["n"], g)
    V = c.get("views", 1)
    cams = _cameras(c, seed, V)
    s = dict(c=c, scene=scene, prm=_params(c), cams=cams)
    if kind == "rgb":
        sh = torch.randn(c["n"], 16, 3, generator=g, device="cuda") * 0.2
        sh[:, 0] = torch.rand(c["n"], 3, generator=g, device="cuda") * 2.8 - 1.4
        s["sh"], s["colours"] = sh, torch.empty(V, c["n"], dim, device="cuda")
        stored = None
    else:
        _, stored = _features(c, c["n"], g)
    s["stored"] = stored
    if kind == "frame":  # a viewer keeps its buffers, sized by the scene's first projection
        s["pr"] = qr.project(*scene, cams[0], s["prm"])
        s["binner"] = qr.Binner(c["n"], W, H, int(1.25 * qr.count_pairs(s["pr"])) + 1024)
        s["out"] = torch.empty(H, W, dim, device="cuda")
        return s
    s["pr"] = qr.project_views(*scene, cams, s["prm"])
    s["binner"] = qr.ViewsBinner(V, c["n"], W, H, int(1.25 * qr.count_pairs(s["pr"])) + 1024)
    s["out"] = torch.empty(V, H, W, dim, device="cuda")
    s["T"] = torch.empty(V, H, W, device="cuda")
    s["n"] = torch.empty(V, H, W, dtype=torch.int32, device="cuda")
    views = []
    for v in range(V):
        pr, b = s["binner"].view(s["pr"], v)
        views.append(dict(tile_offsets=b.tile_offsets, sorted_gid=b.sorted_gid, means2d=pr.means2d,
                          conic_opacity=pr.conic_opacity, features=s["colours"][v] if kind == "rgb" else stored[0],
                          feature_scale=None if kind == "rgb" else stored[1], out=s["out"][v], T_q=s["T"][v],
                          n_sel=s["n"][v], width=W, height=H))
    s["batch"] = _batch(c, views, s["prm"])
    return s


def _batch(c, views, prm):
    code = L.DTYPE_CODE[DTYPE[c["store"]]]
    if c["rule"] == "dense":
        return BatchedDense(views, c["dim"], code, prm.c())
    return BatchedQuantile(views, c["K"], c["dim"], code, prm.c())


def _view_scenes(c, seed, g):
    """Scenes of the batched training case, each larger than the one before, and their views' records."""
    out = []
    for k in range(c["scenes"]):
        n = int(c["n"] * (1 + 1.6 * k))
        scene = _scene(c, n, g)
        stored = _features(c, n, g)[1]
        out.append((n, stored, [_records(c, scene, cam) for cam in _cameras(c, seed * 16 + k, c["views"])]))
    return out


def _prepare_views(c, seed, g):
    W, H, dim = c["width"], c["height"], c["dim"]
    V = c["scenes"] * c["views"]
    s = dict(c=c, prm=_params(c), out=torch.empty(V, H, W, dim, device="cuda"), T=torch.empty(V, H, W, device="cuda"),
             n=torch.empty(V, H, W, dtype=torch.int32, device="cuda"), grads=[])
    views, grads = [], []
    scenes = _view_scenes(c, seed, g)
    s["g"] = torch.randn(V, H, W, dim, generator=g, device="cuda")
    for n, stored, records in scenes:
        acc = [torch.empty(n, k, device="cuda") for k in (dim, 2, 4)]
        s["grads"].append(acc)
        for r in records:
            v = len(views)
            views.append(dict(tile_offsets=r["offsets"], sorted_gid=r["gid"], means2d=r["m"], conic_opacity=r["co"],
                              features=stored[0], feature_scale=stored[1], out=s["out"][v], T_q=s["T"][v],
                              n_sel=s["n"][v], width=W, height=H))
            grads.append(dict(grad_out=s["g"][v], grad_features=acc[0], grad_means2d=acc[1], grad_conic_opacity=acc[2]))
    s["batch"] = _batch(c, views, s["prm"])
    s["batch"].set_grads(grads)
    return s


def _prepare_devox(c, g):
    n, M, U, dim = c["n"], c["slots"], c["unique"], c["dim"]
    cut = torch.sort(torch.randint(0, M + 1, (n - 1,), generator=g, device="cuda"))[0]
    ends = torch.tensor([0, M], device="cuda")
    return dict(c=c, offsets=torch.cat([ends[:1], cut, ends[1:]]),
                voxel=torch.randint(0, U, (M,), generator=g, device="cuda").int(),
                pred=torch.randn(U, dim, generator=g, device="cuda"),
                g=torch.randn(n, dim, generator=g, device="cuda"),
                out=torch.empty(n, dim, device="cuda"), grad=torch.empty(U, dim, device="cuda"),
                arg=torch.empty(n, dim, dtype=torch.int32, device="cuda") if c["reduce"] == "max" else None)


# ---- one pass ------------------------------------------------------------------------------------------

def run(s):
    c = s["c"]
    return {"frame": _run_frame, "batch": _run_batch, "rgb": _run_batch, "train": _run_train, "views": _run_views,
            "devox": _run_devox, "encode": _run_encode}[c["kind"]](s, c)


def _run_frame(s, c):
    pr = qr.project(*s["scene"], s["cams"][0], s["prm"], out=s["pr"])
    bins = s["binner"](pr)
    f, scale = s["stored"]
    if c["rule"] == "dense":
        return qr.render_dense(pr, bins, f, c["width"], c["height"], s["prm"], scale, out=s["out"])
    return qr.render_quantile(pr, bins, f, c["width"], c["height"], c["K"], s["prm"], scale, out=s["out"])


def _run_batch(s, c):
    if c["kind"] == "rgb":
        L.qr_sh_to_rgb_views(s["scene"][0], s["sh"], c["degree"], s["cams"], s["colours"])
    pr = qr.project_views(*s["scene"], s["cams"], s["prm"], out=s["pr"])
    s["binner"](pr)
    s["batch"].render(c["order"], c["per_cu"])
    return dict(out=s["out"], T=s["T"], n=s["n"])


def _run_train(s, c):
    size = (c["width"], c["height"])
    if c["rule"] == "dense":
        out, T, n = qr.DenseRenderFn.apply(s["m"], s["co"], s["f"], s["bins"], *size, s["prm"], s["storage"])
    else:
        out, T, n = qr.QuantileRenderFn.apply(s["m"], s["co"], s["f"], s["bins"], *size, c["K"], s["prm"], s["storage"])
    gm, gc, gf = torch.autograd.grad(out, (s["m"], s["co"], s["f"]), s["g"])
    return dict(out=out.detach(), T=T, n=n, gm=gm, gc=gc, gf=gf)


def _run_views(s, c):
    s["batch"].render(c["order"], c["per_cu"])
    for acc in s["grads"]:
        for t in acc:
            t.zero_()
    s["batch"].backward(c["order"], c["per_cu"])
    return dict(out=s["out"], T=s["T"], n=s["n"], grads=s["grads"])


def _run_devox(s, c):
    reduce = L.QR_REDUCE_MAX if c["reduce"] == "max" else L.QR_REDUCE_MEAN
    L.qr_devoxelize(s["offsets"], s["voxel"], s["pred"], reduce, s["out"], s["arg"])
    s["grad"].zero_()
    L.qr_devoxelize_backward(s["offsets"], s["voxel"], c["unique"], reduce, s["g"], s["arg"], s["grad"])
    return dict(out=s["out"], arg=s["arg"], grad=s["grad"])


def _run_encode(s, c):
    codes, scale = qr.quantize(s["f"], c["store"])
    return dict(codes=codes.view(torch.int16) if c["store"] == "bf16" else codes, scale=scale)


# ---- what a pass cannot do without ---------------------------------------------------------------------

def work(case):
    c = case
    if c["kind"] == "encode":
        return dict(bytes=c["n"] * c["dim"] * (4 + (2 if c["store"] == "bf16" else 1)), flops=0)
    if c["kind"] == "devox":
        # forward: indices, every voxel row and every result; backward: gradients, arguments, voxel gradients
        args = 8 if c["reduce"] == "max" else 4
        return dict(bytes=4 * c["slots"] + 8 * c["n"] + c["dim"] * (8 * c["unique"] + c["n"] * (args + args)), flops=0)
    px = c["width"] * c["height"] * c.get("views", 1) * c.get("scenes", 1)
    size = {"f32": 4, "bf16": 2, "fp8": 1}[c["store"]]
    # rows that show: about one per 128 pixels when K are chosen, one per 15 in the dense blend
    rows = min(px // (15 if c["rule"] == "dense" else 128), c["n"] * c.get("views", 1))
    taken = 40 if c["rule"] == "dense" else min(5, c["K"])  # Gaussians blended per pixel
    back = c["kind"] in ("train", "views")
    b = px * (4 * c["dim"] + 8) + rows * c["dim"] * size
    if back:  # the gradient map, every gradient once, the lists' records
        total = sum(int(c["n"] * (1 + 1.6 * k)) for k in range(c.get("scenes", 1)))
        b += px * 4 * c["dim"] + total * 4 * (c["dim"] + 6)
    else:
        b += c["n"] * (44 + (12 * (c["degree"] + 1) ** 2 if c["kind"] == "rgb" else 0))
    return dict(bytes=b, flops=2 * px * taken * c["dim"] * (3 if back else 1))


# ---- the same outputs in 64 bits -----------------------------------------------------------------------

def exact(case, seed):
    c, g = case, _gen(seed)
    if c["kind"] == "encode":
        if c["store"] == "bf16":
            return None
        a = _features(dict(c, store="f32"), c["n"], g)[0].double().abs().amax(1)
        return dict(codes=None, scale=torch.where(a > 0, a / 448, torch.ones_like(a)))
    if c["kind"] == "devox":
        return _exact_devox(_prepare_devox(c, g), c)
    if c["kind"] == "train":
        s = prepare(c, seed)
        table = s["f"].detach() if s["storage"] is None else s["storage"][0]
        scale = None if s["storage"] is None else s["storage"][1]
        r = _blend64(c, s["m"].detach().double(), s["co"].detach().double(), s["bins"].tile_offsets.long(),
                     s["bins"].sorted_gid.long(), table, scale, s["g"])
        return dict(out=r[0], T=r[1], n=None, gm=r[2][0], gc=r[2][1], gf=r[2][2])
    if c["kind"] == "views":
        out, T, grads = [], [], []
        scenes = _view_scenes(c, seed, g)
        gmap = torch.randn(c["scenes"] * c["views"], c["height"], c["width"], c["dim"], generator=g, device="cuda")
        for n, stored, records in scenes:
            acc = None
            for r in records:
                o, t, acc = _blend64(c, r["m"].double(), r["co"].double(), r["offsets"].long(), r["gid"].long(),
                                     stored[0], stored[1], gmap[len(out)], acc)
                out.append(o)
                T.append(t)
            grads.append([acc[2], acc[0], acc[1]])
        return dict(out=torch.stack(out), T=torch.stack(T), n=None, grads=grads)
    scene = _scene(c, c["n"], g)
    cams = _cameras(c, seed, c.get("views", 1))
    if c["kind"] == "rgb":
        sh = torch.randn(c["n"], 16, 3, generator=g, device="cuda") * 0.2
        sh[:, 0] = torch.rand(c["n"], 3, generator=g, device="cuda") * 2.8 - 1.4
    else:
        table, scale = _features(c, c["n"], g)[1]
    out, T = [], []
    for cam in cams:
        if c["kind"] == "rgb":
            table, scale = _colours64(c, scene[0].double(), sh.double(), cam), None
        m, co, z, box, tiles = _project64(scene, cam)
        offsets, gid = _lists(z, box, tiles, c["width"], c["height"])
        o, t, _ = _blend64(c, m, co, offsets, gid, table, scale)
        out.append(o)
        T.append(t)
    if c["kind"] == "frame":
        return dict(out=out[0], **({"T_final": T[0], "n_contrib": None} if c["rule"] == "dense" else
                                   {"T_q": T[0], "n_sel": None}))
    return dict(out=torch.stack(out), T=torch.stack(T), n=None)


def _decode(rows, scale):
    if rows.dtype == torch.uint8:
        return rows.view(torch.float8_e4m3fn).double() * scale.double()[..., None]
    return rows.double()


def _weights(c, a):
    """Blending weights [B, 256, L] and the remaining transmittance from alpha' (0 off the ray)."""
    T = torch.cumprod(1 - a.detach(), 2)
    K = c["K"]
    if c["rule"] == "quantile":
        seen = torch.ones_like(T, dtype=torch.bool)
        t = [_f32(1 - m / (K + 1)) for m in range(1, K + 1)]
    else:
        seen = T >= T_EPS
        if c["rule"] == "stratified":
            on = seen & (a.detach() > 0)
            n = 1 + on.sum(2)
            s1, s2 = 1 + (T * on).sum(2), 1 + (T * T * on).sum(2)
            mu = s1 / n
            sigma = (s2 / n - mu * mu).clamp(min=0).sqrt()
            p = torch.tensor([1 - m / (K + 1) for m in range(1, K + 1)], dtype=torch.float64, device="cuda")
            z = torch.special.ndtri(p)
            t = [(mu + sigma * z[m]).clamp(0, 1).float().double()[..., None] for m in range(K)]
    if c["rule"] in ("quantile", "stratified"):
        k = torch.zeros(T.shape, dtype=torch.int8, device="cuda")
        for tm in t:
            k += T < tm
        before = torch.cat([torch.zeros_like(k[..., :1]), k[..., :-1]], 2)
        take = (k > before) & seen
    else:
        take = seen & (a.detach() > 0)
    x = a * take
    left = torch.cumprod(1 - x, 2)
    w = x * torch.cat([torch.ones_like(left[..., :1]), left[..., :-1]], 2)
    if c["rule"] == "dense":
        return w, left[..., -1]
    if c["rule"] == "topk":
        if w.shape[2] > K:
            at = torch.sort(w.detach(), dim=2, descending=True, stable=True)[1][..., :K]
            w = w * torch.zeros_like(w).scatter_(2, at, 1.0)
        rest = 1 - w.sum(2)
    else:
        rest = left[..., -1]
    some = (w.detach() > 0).any(2)
    return w / torch.where(some, 1 - rest, torch.ones_like(rest))[..., None], rest


def _blend64(c, m, co, offsets, gid, table, scale, grad=None, acc=None):
    """Map, transmittance and, given the map's gradient, the gradients of means, conics and features (added to acc)."""
    W, H, dim = c["width"], c["height"], c["dim"]
    tx, dev = -(-W // TILE), "cuda"
    out = torch.zeros(H, W, dim, dtype=torch.float64, device=dev)
    rest = torch.ones(H, W, dtype=torch.float64, device=dev)
    if grad is not None and acc is None:
        acc = [torch.zeros(len(m), k, dtype=torch.float64, device=dev) for k in (2, 4, dim)]
    size, tiles = torch.sort(offsets[1:] - offsets[:-1], descending=True)
    lengths = size.tolist()
    ii = torch.arange(TILE * TILE, device=dev)
    at = 0
    while at < len(lengths) and lengths[at] > 0:
        n = lengths[at]
        B = max(1, min(65536 // n, len(lengths) - at))
        t, s = tiles[at:at + B], size[at:at + B]
        at += B
        j = torch.arange(n, device=dev)[None]
        live = j < s[:, None]
        ids = gid[(offsets[t][:, None] + j).clamp(max=len(gid) - 1)]
        px = (t % tx)[:, None] * TILE + ii % TILE
        py = torch.div(t, tx, rounding_mode="floor")[:, None] * TILE + ii // TILE
        inside = (px < W) & (py < H)
        leaf = [x.detach().requires_grad_(grad is not None) for x in
                (m[ids], co[ids], _decode(table[ids], None if scale is None else scale[ids]))]
        with torch.set_grad_enabled(grad is not None):
            mm, cc, F = leaf
            dx = px[..., None] + 0.5 - mm[:, None, :, 0]
            dy = py[..., None] + 0.5 - mm[:, None, :, 1]
            cc = cc[:, None]
            power = -0.5 * (cc[..., 0] * dx * dx + cc[..., 2] * dy * dy) - cc[..., 1] * dx * dy
            a = (cc[..., 3] * torch.exp(power)).clamp(max=ALPHA_MAX)
            a = a * ((a.detach() >= ALPHA_MIN) & live[:, None])
            w, left = _weights(c, a)
            o = w @ F
            if grad is not None:
                go = torch.zeros_like(o)
                go[inside] = grad[py[inside], px[inside]].double()
                for x, d in zip(acc, torch.autograd.grad(o, leaf, go)):
                    x.index_add_(0, ids[live], d[live])
        out[py[inside], px[inside]] = o.detach()[inside]
        rest[py[inside], px[inside]] = left.detach()[inside]
    return out, rest, acc


def _colours64(c, mu, sh, cam):
    R = torch.tensor(cam.R_cw, device="cuda").double()
    d = mu + R.T @ torch.tensor(cam.t, device="cuda").double()
    x, y, z = (d / d.norm(dim=1, keepdim=True)).unbind(1)
    pi, one = math.pi, torch.ones_like(mu[:, 0])
    q = lambda k: math.sqrt(k / pi)  # noqa: E731
    Y = [0.5 * q(1) * one,
         -q(3 / 4) * y, q(3 / 4) * z, -q(3 / 4) * x,
         q(15 / 4) * x * y, -q(15 / 4) * y * z, q(5 / 16) * (3 * z * z - 1), -q(15 / 4) * x * z, q(15 / 16) * (x * x - y * y),
         -q(35 / 32) * y * (3 * x * x - y * y), q(105 / 4) * x * y * z, -q(21 / 32) * y * (5 * z * z - 1),
         q(7 / 16) * (5 * z ** 3 - 3 * z), -q(21 / 32) * x * (5 * z * z - 1), q(105 / 16) * z * (x * x - y * y),
         -q(35 / 32) * x * (x * x - 3 * y * y)]
    n = (c["degree"] + 1) ** 2
    rgb = 0.5 + sum(Y[k][:, None] * sh[:, k] for k in range(n))
    out = torch.zeros(len(mu), c["dim"], dtype=torch.float64, device="cuda")
    out[:, :3] = rgb.clamp(min=0)
    return out


def _exact_devox(s, c):
    n, dim, U = c["n"], c["dim"], c["unique"]
    size = s["offsets"][1:] - s["offsets"][:-1]
    of = torch.repeat_interleave(torch.arange(n, device="cuda"), size)
    vox = s["voxel"].long()
    out = torch.zeros(n, dim, dtype=torch.float64, device="cuda")
    grad = torch.zeros(U, dim, dtype=torch.float64, device="cuda")
    if c["reduce"] == "mean":
        out.index_add_(0, of, s["pred"][vox].double())
        k = size.clamp(min=1)[:, None]
        grad.index_add_(0, vox, (s["g"].double() / k)[of])
        return dict(out=out / k, arg=None, grad=grad)
    for c0 in range(0, dim, 64):  # columns at a time: the gathered rows take memory
        cols = slice(c0, min(dim, c0 + 64))
        rows = s["pred"][:, cols][vox]
        at = of[:, None].expand_as(rows)
        best = torch.full((n, rows.shape[1]), -math.inf, device="cuda").scatter_reduce_(0, at, rows, "amax")
        slot = torch.arange(len(of), device="cuda")[:, None].expand_as(rows)
        first = torch.full(best.shape, len(of), device="cuda").scatter_reduce_(
            0, at, torch.where(rows == best[of], slot, torch.full_like(slot, len(of))), "amin")
        some = first < len(of)
        out[:, cols] = torch.where(some, best, torch.zeros_like(best)).double()
        to = vox[first.clamp(max=len(of) - 1)]
        grad[:, cols] = grad[:, cols].scatter_add(0, to, torch.where(some, s["g"][:, cols], torch.zeros_like(best)).double())
    return dict(out=out, arg=None, grad=grad)
