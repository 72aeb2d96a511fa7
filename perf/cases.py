"""The measured work of the renderer: what a program that uses it calls, over the range of sizes it calls it with.

Kinds of case:
  view   a viewer's frame: the forward render of one camera, the BVH kept between frames or (rebuild) built for
         the frame, as after an edit of the scene; no ray state is written
  train  an optimisation step on one camera through autograd: BVH rebuild, forward, loss, adjoint; the adjoint
         replays stored hit lists (hit_list > 0) or traverses again (hit_list = 0, the default of Params)
  batch  a step on several cameras at once in one persistent launch, on buffers that the program keeps
  mesh   Gaussians with a triangle mesh: mirrors, glass and shadows; forward, or forward and adjoint
  loss   the training loss of one image and its gradient

Scenes (layout): "box", means uniform in a cube, the scene of the small examples; "clusters", eight blobs of
larger splats; "ground", a ground plane with 64 clusters, log-normal scales and a fifth of the Gaussians nearly
opaque, the shape of a captured outdoor scene. Sizes are those of the measured workloads of this repository
(1k at 64x64, 100k at 800x800, 300k on eight views, 1M at 1920x1080, 500k with a mesh at four 1024x768 views)
and ragged ones between them.
"""

import math

import numpy as np
import torch

from paper_2501_19196_amd import renderer as R
from paper_2501_19196_amd._lib import RS_BUILD_LBVH, RS_PAPER_GRADIENT, RS_PERSISTENT

DEV = "cuda"


def listed():
    return [
        # the smallest call: the example scene in a thumbnail, built for this frame
        dict(name="view-1k-64x64", kind="view", layout="box", n=1000, width=64, height=64, rebuild=True, lbvh=False),
        # the quick start's optimisation step: default parameters, a thumbnail
        dict(name="train-1k-64x64", kind="train", layout="box", n=1000, width=64, height=64, hit_list=0, loss="l1",
             paper=False),
        # an object capture early in its training: few Gaussians, a ragged image
        dict(name="train-20k-251x187", kind="train", layout="clusters", n=20011, width=251, height=187, hit_list=64,
             loss="paper", paper=False),
        # an ordinary training step of an object capture
        dict(name="train-100k-800x800", kind="train", layout="clusters", n=100000, width=800, height=800, hit_list=64,
             loss="paper", paper=False),
        # the same step without stored hit lists, for programs short of memory (the default of Params)
        dict(name="train-100k-640x479-lean", kind="train", layout="clusters", n=99991, width=640, height=479,
             hit_list=0, loss="l1", paper=False),
        # the scene-scale training step
        dict(name="train-1M-1920x1080", kind="train", layout="ground", n=1000000, width=1920, height=1080, hit_list=64,
             loss="l1", paper=False),
        # a viewer of a finished scene-scale capture: the BVH is kept
        dict(name="view-1M-1920x1080", kind="view", layout="ground", n=1000000, width=1920, height=1080, rebuild=False,
             lbvh=False),
        # an editor's preview: the scene was changed, so its BVH is built for this small frame
        dict(name="edit-1M-320x180", kind="view", layout="ground", n=1000000, width=320, height=180, rebuild=True,
             lbvh=False),
        # a step on eight cameras of two resolutions
        dict(name="batch-300k-8views", kind="batch", layout="clusters", n=300000, width=800, height=800, views=4,
             small_width=400, small_height=300, small_views=4, hit_list=64),
        # mirror floor, diffuse sphere and shadows among Gaussians: one step on four views
        dict(name="mesh-500k-4x1024x768", kind="mesh", layout="ground", n=500000, width=1024, height=768, views=4,
             glass=False, bounces=1, hit_list=64, backward=True),
        # a viewer's frame with glass, three bounces
        dict(name="glass-150k-640x361", kind="mesh", layout="ground", n=150001, width=640, height=361, views=1,
             glass=True, bounces=3, hit_list=0, backward=False),
        # the training loss and its gradient at full resolution
        dict(name="loss-1920x1080", kind="loss", width=1920, height=1080, grad=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """An image of lo to hi pixels, of a common aspect ratio, its sides rounded to whatever they come to."""
    pixels, aspect = _log_int(rng, lo, hi), rng.choice((1.0, 4 / 3, 16 / 9, 3 / 4, 1.5))
    w = max(8, int(round(math.sqrt(pixels * aspect))))
    return w, max(8, pixels // w)


def _scene_size(rng, most):
    """Each layout over the counts that it stands for (a denser box or denser clusters would be no scene)."""
    layout = rng.choice(("box", "clusters", "ground"))
    lo, hi = {"box": (300, 3000), "clusters": (3000, 300000), "ground": (20000, 1000000)}[layout]
    return layout, _log_int(rng, lo, min(hi, most))


def draw(rng):
    kind = rng.choice(("view", "view", "train", "train", "train", "batch", "mesh", "loss"))
    if kind == "loss":
        w, h = _size(rng, 64 * 64, 1920 * 1080)
        return dict(kind="loss", width=w, height=h, grad=rng.random() < 0.8)
    if kind == "mesh":
        w, h = _size(rng, 160 * 120, 1024 * 768)
        glass = rng.random() < 0.4
        return dict(kind="mesh", layout="ground", n=_log_int(rng, 20000, 500000), width=w, height=h,
                    views=rng.choice((1, 2, 3)), glass=glass, bounces=rng.choice((1, 2, 3)) if glass else 1,
                    hit_list=rng.choice((0, 64, 64)), backward=rng.random() < 0.6)
    if kind == "batch":
        w, h = _size(rng, 100 * 75, 800 * 800)
        return dict(kind="batch", layout="clusters", n=_log_int(rng, 3000, 300000), width=w, height=h,
                    views=rng.choice((2, 3, 4)), small_width=max(8, w // 2), small_height=max(8, h * 3 // 8),
                    small_views=rng.choice((0, 2, 4)), hit_list=64)
    layout, n = _scene_size(rng, 1000000)
    w, h = _size(rng, 48 * 48, 1920 * 1080 if layout == "ground" else 800 * 800)
    if kind == "view":
        rebuild = rng.random() < 0.6
        return dict(kind="view", layout=layout, n=n, width=w, height=h, rebuild=rebuild,
                    lbvh=rebuild and rng.random() < 0.15)
    hit_list = rng.choice((0, 64, 64, 128))
    paper = hit_list > 0 and w * h <= 500000 and rng.random() < 0.15
    return dict(kind="train", layout=layout, n=n, width=w, height=h, hit_list=648 if paper else hit_list,
                loss=rng.choice(("l1", "paper")), paper=paper)


# ------------------------------------------------------------------ inputs

def _scene(layout, n, gen):
    """mean, scale, quat, opacity, rgb of a seeded scene."""
    u = lambda *s: torch.rand(*s, generator=gen, device=DEV, dtype=torch.float64)
    z = lambda *s: torch.randn(*s, generator=gen, device=DEV, dtype=torch.float64)
    if layout == "box":
        mean = u(n, 3) * 2 - 1
    elif layout == "clusters":
        centres = (u(8, 3) * 2 - 1) * 1.4
        k = torch.randint(0, 8, (n,), generator=gen, device=DEV)
        mean = (centres[k] + 0.3 * z(n, 3)).clamp(-2, 2)
    else:
        half = n // 2
        mean = torch.empty(n, 3, device=DEV, dtype=torch.float64)
        mean[:half, :2] = u(half, 2) * 8 - 4
        mean[:half, 2] = 0.02 * z(half)
        centres = torch.cat([u(64, 2) * 6 - 3, u(64, 1) * 1.8 + 0.2], 1)
        k = torch.randint(0, 64, (n - half,), generator=gen, device=DEV)
        mean[half:] = centres[k] + 0.3 * z(n - half, 3)
        mean = mean[torch.randperm(n, generator=gen, device=DEV)]
    if layout == "ground":
        scale = torch.exp(math.log(0.02) + 0.7 * z(n, 3))
        opacity = torch.sigmoid(z(n) - 1)
        opacity = torch.where(u(n) < 0.2, 0.95 + 0.049 * u(n), opacity)
    else:
        scale = torch.exp(math.log(0.01) + u(n, 3) * math.log(10.0))
        opacity = torch.sigmoid(z(n))
    flat = u(n) < 0.3  # a third are flat: one axis of 1e-5
    axis = torch.randint(0, 3, (n,), generator=gen, device=DEV)
    scale[flat, axis[flat]] = 1e-5
    quat = z(n, 4)
    quat = quat / quat.norm(dim=1, keepdim=True)
    rgb = u(n, 3)
    return [a.float().contiguous() for a in (mean, scale, quat, opacity.clamp(max=0.999), rgb)]


def _camera(eye, target, up, w, h):
    """Origins and unit directions of a pinhole camera (60 degrees high), row-major pixels."""
    eye, target, up = (np.asarray(v, np.float64) for v in (eye, target, up))
    fwd = (target - eye) / np.linalg.norm(target - eye)
    right = np.cross(fwd, up)
    right = right / np.linalg.norm(right)
    up = np.cross(right, fwd)
    fwd, right, up = (torch.from_numpy(v).to(DEV) for v in (fwd, right, up))
    tan = math.tan(math.radians(30.0))
    x = (2 * (torch.arange(w, device=DEV, dtype=torch.float64) + 0.5) / w - 1) * tan * w / h
    y = (1 - 2 * (torch.arange(h, device=DEV, dtype=torch.float64) + 0.5) / h) * tan
    d = fwd + x[None, :, None] * right + y[:, None, None] * up
    d = (d / d.norm(dim=2, keepdim=True)).reshape(-1, 3).float().contiguous()
    o = torch.from_numpy(eye).to(DEV).float().expand(w * h, 3).contiguous()
    return o, d


def _one_camera(layout, w, h):
    if layout == "ground":
        return _camera((0, -7, 3.5), (0, 0, 0.5), (0, 0, 1), w, h)
    return _camera((0, 0, -3 if layout == "box" else -4), (0, 0, 0), (0, 1, 0), w, h)


def _cameras(placed):
    """Rays of several cameras back to back and their view table; placed: [(eye, target, up, w, h)]."""
    os_, ds, views, off = [], [], [], 0
    for eye, target, up, w, h in placed:
        o, d = _camera(eye, target, up, w, h)
        os_.append(o)
        ds.append(d)
        views.append((off, w, h))
        off += w * h
    return torch.cat(os_), torch.cat(ds), views


def _around(count, sizes):
    """Cameras spread over a sphere of radius 4, looking at its centre."""
    placed = []
    for i in range(count):
        z = 1 - 2 * (i + 0.5) / count
        r, phi = math.sqrt(max(0.0, 1 - z * z)), math.pi * (3 - math.sqrt(5)) * i
        up = (0, 0, 1) if abs(z) <= 0.95 else (0, 1, 0)
        placed.append(((4 * r * math.cos(phi), 4 * r * math.sin(phi), 4 * z), (0, 0, 0), up) + sizes[i])
    return placed


def _ring(count, w, h):
    placed = []
    for i in range(count):
        a = 2 * math.pi * i / count + 0.25 * math.pi
        placed.append(((6 * math.cos(a), 6 * math.sin(a), 3), (0, 0, 0.5), (0, 0, 1), w, h))
    return placed


def _grid(cells):
    """Vertices (u, v) in [-1, 1]^2 and triangles of a square grid."""
    s = np.linspace(-1, 1, cells + 1)
    u, v = (a.ravel() for a in np.meshgrid(s, s))
    k = (np.arange(cells)[:, None] * (cells + 1) + np.arange(cells)[None, :]).ravel()
    a, b, c, d = k, k + 1, k + cells + 1, k + cells + 2
    return u, v, np.concatenate([np.stack([a, b, d], 1), np.stack([a, d, c], 1)])


def _cube(cells):
    """A closed cube [-1, 1]^3 of gridded faces, wound outwards."""
    u, v, t = _grid(cells)
    verts, tris = [], []
    for axis in range(3):
        for sign in (1, -1):
            p = np.empty((len(u), 3))
            p[:, axis], p[:, (axis + 1) % 3], p[:, (axis + 2) % 3] = sign, u, v
            verts.append(p)
            tris.append((t if sign > 0 else t[:, ::-1]) + len(u) * (len(verts) - 1))
    return np.concatenate(verts), np.concatenate(tris)


def _mesh(glass):
    """A mirror floor with a sphere above it (diffuse, or glass beside a glass box)."""
    u, v, pt = _grid(50)
    parts = [(np.stack([3 * u, 3 * v, 0 * u], 1), pt, 1)]
    sv, st = _cube(21)
    parts.append((0.6 * sv / np.linalg.norm(sv, axis=1, keepdims=True) + (0, 0, 0.8), st, 2 if glass else 0))
    if glass:
        bv, bt = _cube(1)
        parts.append((0.4 * bv + (1.3, -1.2, 0.45), bt, 2))
    verts, tris, mat, off = [], [], [], 0
    for pv, t, m in parts:
        verts.append(pv)
        tris.append(t + off)
        mat.append(np.full(len(t), m))
        off += len(pv)
    dev = lambda a, dt: torch.from_numpy(np.ascontiguousarray(np.concatenate(a).astype(dt))).to(DEV)
    return R.Mesh(dev(verts, np.float32), dev(tris, np.int32), dev(mat, np.int32))


def _photo(w, h, gen):
    """A target image [h * w, 3]: smooth shapes with a little noise, in [0, 1]."""
    low = torch.rand(1, 3, max(2, h // 24), max(2, w // 24), generator=gen, device=DEV)
    img = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear", align_corners=False)
    img = img + 0.02 * torch.randn(img.shape, generator=gen, device=DEV)
    return img.clamp(0, 1)[0].permute(1, 2, 0).reshape(-1, 3).contiguous()


def _gradient(rays, gen):
    """An L1 loss's gradient: a sign per channel over the count of values."""
    s = torch.randint(0, 2, (rays, 3), generator=gen, device=DEV).float() * 2 - 1
    return s / (3.0 * rays)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kind, s = case["kind"], dict(case)
    if kind == "loss":
        w, h = case["width"], case["height"]
        s["target"] = _photo(w, h, gen)
        s["img"] = (s["target"] + 0.1 * torch.randn(w * h, 3, generator=gen, device=DEV)).clamp(0, 1)
        s["ws"] = R.loss_workspace(w, h)
        return s
    scene = _scene(case["layout"], case["n"], gen)
    s["scene"] = scene
    w, h = case["width"], case["height"]
    if kind == "view":
        o, d = _one_camera(case["layout"], w, h)
        s["rays"] = R.Rays(o, d, views=[(0, w, h)])
        s["g"] = R.Gaussians(*scene)
        s["params"] = R.Params(flags=RS_BUILD_LBVH if case["lbvh"] else 0)
        s["ws"] = torch.empty(R.workspace_bytes(case["n"]), dtype=torch.uint8, device=DEV)
        if not case["rebuild"]:
            s["bvh"] = R.build_bvh(s["g"], s["params"], workspace=s["ws"])
    elif kind == "train":
        s["o"], s["d"] = _one_camera(case["layout"], w, h)
        s["leaves"] = [a.requires_grad_(True) for a in scene]
        s["target"] = _photo(w, h, gen)
        s["params"] = R.Params(hit_list=case["hit_list"], flags=RS_PAPER_GRADIENT if case["paper"] else 0,
                               eps2=1e-3 if case["paper"] else 1e-4)
    elif kind == "batch":
        sizes = [(w, h)] * case["views"] + [(case["small_width"], case["small_height"])] * case["small_views"]
        o, d, views = _cameras(_around(len(sizes), sizes))
        s["rays"] = R.Rays(o, d, views=views)
        s["g"] = R.Gaussians(*scene)
        s["params"] = R.Params(hit_list=case["hit_list"], flags=RS_PERSISTENT)
        s["ws"] = torch.empty(R.workspace_bytes(case["n"]), dtype=torch.uint8, device=DEV)
        s["state"] = R.new_state(s["rays"].n, s["params"], DEV)
        s["out"] = torch.empty(s["rays"].n, 3, device=DEV)
        s["grad"] = _gradient(s["rays"].n, gen)
        s["grads"] = tuple(torch.empty_like(a) for a in scene)
    else:
        s["o"], s["d"], s["views"] = _cameras(_ring(case["views"], w, h))
        s["mesh"] = _mesh(case["glass"])
        s["mbvh"] = R.build_mesh_bvh(s["mesh"])
        s["shading"] = R.Shading(max_bounces=case["bounces"])
        s["params"] = R.Params(hit_list=case["hit_list"])
        s["leaves"] = [a.requires_grad_(case["backward"]) for a in scene]
        s["grad"] = _gradient(s["o"].shape[0], gen)
        if not case["backward"]:
            s["g"] = R.Gaussians(*scene)
            s["rays"] = R.Rays(s["o"], s["d"], views=s["views"])
            s["frame"] = R.mesh_frame(s["rays"].n, s["params"], DEV, s["shading"])
            s["ws"] = torch.empty(R.workspace_bytes(case["n"]), dtype=torch.uint8, device=DEV)
    return s


# -------------------------------------------------------------------- run

def run(s):
    kind = s["kind"]
    if kind == "loss":
        loss, grad = R.image_loss(s["img"], s["target"], s["width"], s["height"], grad=s["grad"], ws=s["ws"])
        return dict(loss=loss, grad=grad) if s["grad"] else dict(loss=loss)
    if kind == "view":
        bvh = s["bvh"] if not s["rebuild"] else R.build_bvh(s["g"], s["params"], workspace=s["ws"])
        out, _ = R.render_fwd(bvh, s["g"], s["rays"], s["params"], want_state=False)
        return dict(image=out)
    if kind == "train":
        w, h = s["width"], s["height"]
        img = R.render(*s["leaves"], s["o"], s["d"], s["params"], [(0, w, h)])
        if s["loss"] == "paper":
            loss = R.ImageLoss.apply(img, s["target"], w, h)
        else:
            loss = (img - s["target"]).abs().mean()
        return dict(image=img.detach(), loss=loss.detach(), grads=torch.autograd.grad(loss, s["leaves"]))
    if kind == "batch":
        bvh = R.build_bvh(s["g"], s["params"], workspace=s["ws"])
        R.render_fwd(bvh, s["g"], s["rays"], s["params"], out=s["out"], state=s["state"])
        R.render_bwd(bvh, s["g"], s["rays"], s["params"], s["grad"], s["state"], grads=s["grads"])
        return dict(image=s["out"], grads=s["grads"])
    if s["backward"]:
        img = R.MeshRender.apply(*s["leaves"], s["o"], s["d"], s["mesh"], s["mbvh"], s["shading"], s["params"],
                                 s["views"])
        return dict(image=img.detach(), grads=torch.autograd.grad(img, s["leaves"], s["grad"]))
    bvh = R.build_bvh(s["g"], s["params"], workspace=s["ws"])
    out, _ = R.render_mesh_fwd(bvh, s["mbvh"], s["g"], s["mesh"], s["shading"], s["rays"], s["params"],
                               frame=s["frame"])
    return dict(image=out)


# ------------------------------------------------------------------- work

def _rays(case):
    if case["kind"] == "batch":
        return case["width"] * case["height"] * case["views"] \
            + case["small_width"] * case["small_height"] * case["small_views"]
    return case["width"] * case["height"] * (case["views"] if case["kind"] == "mesh" else 1)


def _hits(case):
    """Hits that a ray composites on average, about: 40 in the 1M ground scene, fewer the fewer Gaussians there
    are (the hits of a ray go with the Gaussians' count until an opaque surface ends it)."""
    full, at = {"box": (6, 1000), "clusters": (40, 100000), "ground": (40, 1000000)}[case["layout"]]
    return full * min(1.0, case["n"] / at)


def work(case):
    """Inputs read once, outputs written once; per composited hit the ray-ellipsoid test, alpha and Eq. 3 (110
    operations) and its adjoint (265 with the chain to the parameters)."""
    if case["kind"] == "loss":
        n = case["width"] * case["height"]
        # two 11-tap passes over the five moments and, for the gradient, over the three maps, per channel
        return dict(bytes=n * (36 if case["grad"] else 24), flops=n * 3 * 44 * (8 if case["grad"] else 5))
    rays, n = _rays(case), case["n"]
    backward = case["kind"] in ("train", "batch") or case.get("backward", False)
    b, f = rays * 36 + n * 56, rays * _hits(case) * 110
    if backward:
        b, f = b + rays * 12 + n * 56, f + rays * _hits(case) * 265
    if case["kind"] == "mesh":
        f *= 2
    return dict(bytes=b, flops=f)


# ------------------------------------------------------------------ exact

PAIRS = 2_000_000_000  # ray-Gaussian pairs that the reference below tests within some seconds


def exact(case, seed):
    if case["kind"] == "loss":
        s = prepare(case, seed)
        img = s["img"].double().requires_grad_(True)
        loss = _loss64(img, s["target"].double(), case["width"], case["height"])
        if not case["grad"]:
            return dict(loss=loss.detach().reshape(1))
        return dict(loss=loss.detach().reshape(1), grad=torch.autograd.grad(loss, img)[0])
    if case["kind"] not in ("view", "train") or case.get("paper") or _rays(case) * case["n"] > PAIRS:
        return None
    gen = torch.Generator(device=DEV).manual_seed(seed)
    p = [a.double().requires_grad_(case["kind"] == "train") for a in _scene(case["layout"], case["n"], gen)]
    w, h = case["width"], case["height"]
    o, d = (a.double() for a in _one_camera(case["layout"], w, h))
    img = _render64(*p, o, d)
    if case["kind"] == "view":
        return dict(image=img)
    target = _photo(w, h, gen).double()
    loss = _loss64(img, target, w, h) if case["loss"] == "paper" else (img - target).abs().mean()
    return dict(image=img.detach(), loss=loss.detach(), grads=torch.autograd.grad(loss, p))


def _rotation64(q):
    a, b, c, d = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (c * c + d * d), 2 * (b * c - a * d), 2 * (b * d + a * c),
                        2 * (b * c + a * d), 1 - 2 * (b * b + d * d), 2 * (c * d - a * b),
                        2 * (b * d - a * c), 2 * (c * d + a * b), 1 - 2 * (b * b + c * c)], 1).reshape(-1, 3, 3)


def _meet64(x, d, Rm, s):
    """Whitened line-to-centre distance squared and the nearer root's depth; x = o - mean, the last axis is xyz."""
    ow, dw = ((v.unsqueeze(-1) * Rm).sum(-2) / s for v in (x, d))
    a, b = (dw * dw).sum(-1), (ow * dw).sum(-1)
    u = torch.linalg.cross(ow, dw)
    h2 = (u * u).sum(-1) / a
    return h2, -b / a - torch.sqrt((_Q - h2).clamp(min=0) / a)


_Q = float(np.float32(11.3449))
_EPS1, _MAX_HITS = float(np.float32(1e-4)), 512


def _render64(mean, scale, quat, opacity, rgb, o, d):
    """Every ray against every Gaussian, the hits of a ray sorted by depth and composited front to back."""
    n, rays = mean.shape[0], o.shape[0]
    Rm = _rotation64(quat)
    with torch.no_grad():
        found = []
        step = max(1, 20_000_000 // n)
        for k in range(0, rays, step):
            h2, t = _meet64(o[k:k + step, None] - mean, d[k:k + step, None].expand(-1, n, 3), Rm, scale)
            r, g = torch.nonzero((h2 <= _Q) & (t >= 0), as_tuple=True)
            found.append((r + k, g, t[r, g]))
        ray, gid, t = (torch.cat(v) for v in zip(*found))
        at = torch.argsort(t, stable=True)
        at = at[torch.argsort(ray[at], stable=True)]
        ray, gid = ray[at], gid[at]
        count = torch.bincount(ray, minlength=rays)
        slot = torch.arange(ray.numel(), device=ray.device) - (torch.cumsum(count, 0) - count)[ray]
        most = max(1, int(count.max()))
    h2, _ = _meet64(o[ray] - mean[gid], d[ray], Rm[gid], scale[gid])
    alpha = opacity[gid] * torch.exp(-0.5 * h2)
    A = torch.zeros(rays, most, dtype=alpha.dtype, device=alpha.device).index_put((ray, slot), alpha)
    with torch.no_grad():  # a ray stops behind the hit that takes T below eps1, and after max_hits
        before = torch.cumprod(torch.cat([torch.ones_like(A[:, :1]), 1 - A[:, :-1]], 1), 1)
        keep = (before >= _EPS1) & (torch.arange(most, device=A.device) < _MAX_HITS)
    A = A * keep
    T = torch.exp(torch.cumsum(torch.cat([torch.zeros_like(A[:, :1]), torch.log1p(-A[:, :-1])], 1), 1))
    weight = (T * A)[ray, slot]
    return torch.zeros(rays, 3, dtype=alpha.dtype, device=alpha.device).index_add(0, ray, weight[:, None] * rgb[gid])


def _loss64(img, target, w, h, lam=0.2, radius=5, sigma=1.5):
    """(1 - lam) L2 + lam (1 - SSIM) / 2, SSIM from moments of a Gaussian window that is zero outside the image."""
    x, y = (v.reshape(h, w, 3).permute(2, 0, 1).unsqueeze(1) for v in (img, target))
    m = torch.arange(-radius, radius + 1, dtype=torch.float64, device=img.device)
    k = torch.exp(-m * m / (2 * sigma * sigma))
    k = k / k.sum()

    def blur(v):
        v = torch.nn.functional.pad(v, (radius,) * 4)
        v = sum(k[i] * v[:, :, :, i:i + w] for i in range(2 * radius + 1))
        return sum(k[i] * v[:, :, i:i + h] for i in range(2 * radius + 1))

    mx, my = blur(x), blur(y)
    vx, vy, cov = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    c1, c2 = 0.01 ** 2, 0.03 ** 2
    ssim = (2 * mx * my + c1) * (2 * cov + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2))
    return (1 - lam) * ((x - y) ** 2).mean() + lam * (1 - ssim.mean()) / 2
