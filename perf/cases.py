"""Workloads that this rasterizer is timed on, through its public entry points.

A case is a dict of plain values. ``listed()`` holds the workloads a user has the framework do:
rendering a view, a forward + backward step in each texture layout, a whole optimisation step,
single-image fitting and densification, from 1k splats at 128 x 128 to 3M splats on four 1080p
views (the named workloads of ``scenegen`` and ``bench.py``, and two odd-sized ones).
``draw(rng)`` gives more cases of the same ranges. ``prepare`` makes what a program holds before
the call (splats, a planned rasterizer, gradient buffers), ``run`` is one pass, ``work`` counts
what the pass cannot do without and ``exact`` is a plain float64 torch rendering of the smaller
cases.

Kinds of case:
  view    forward render (``Rasterizer.forward``), as a viewer does
  step    forward + backward into kept buffers (``Rasterizer.forward`` / ``backward``)
  autograd  the differentiable ``render()`` with torch's autograd, default checks on
  train   one ``Trainer.step``: activations, render, L1 or MSE loss, backward, Adam
  densify ``TrainState.densify``: clone, split and prune with the optimiser state
"""
import math

import numpy as np
import torch

import paper_2412_12734_amd as gb
from paper_2412_12734_amd import train as gbt

SIGMA, ALPHA_MIN, ALPHA_MAX, T_MIN, LP_VAR = 0.5, 1.0 / 255.0, 0.99, 1e-4, 0.5


def _case(kind, P, N, res, views=1, orbit=False, dist=8.0, half=4.0, s_lo=0.02, s_hi=0.2,
          bf16=False, sides="", sh=-1, loss="l1", name=None):
    c = dict(kind=kind, P=P, N=N, res=res, views=views, orbit=orbit, dist=dist, half=half,
             s_lo=s_lo, s_hi=s_hi, bf16=bf16, sides=sides, sh=sh, loss=loss)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a thumbnail of a small object, where launches and latency count
        _case("view", 1000, 4, "128x128", dist=3.0, half=1.0, name="view_1k_128"),
        # a viewer's frame of a large scene (bfloat16 colour grids, as a trained scene is stored)
        _case("view", 1_000_000, 8, "1920x1080", bf16=True, name="view_1m_bf16_1080p"),
        # a mid-sized object at a common training resolution
        _case("step", 100_000, 8, "800x800", dist=5.0, half=2.0, s_lo=0.005, s_hi=0.1,
              name="step_100k_800"),
        # the headline workload: 1M splats, 8 x 8 grids, one 1080p view
        _case("step", 1_000_000, 8, "1920x1080", name="step_1m_1080p"),
        # the same with the largest grids
        _case("step", 1_000_000, 16, "1920x1080", name="step_1m_n16_1080p"),
        # the same with grids of several sides in one call
        _case("step", 1_000_000, 8, "1920x1080", sides="2,4,8", name="step_1m_mixed_1080p"),
        # many views of uneven size in one call
        _case("step", 1_000_000, 4, "640x480,1024x768,1280x720,1600x1060", views=16, orbit=True,
              name="step_1m_16_views"),
        # the largest call: many small splats, bfloat16 grids, a batch of four 1080p views
        _case("step", 3_000_000, 8, "1920x1080", views=4, orbit=True, s_lo=0.002, s_hi=0.05,
              bf16=True, name="step_3m_4x1080p"),
        # a user's own torch loop: autograd, view-dependent colour, odd sizes, checks on
        _case("autograd", 20_011, 2, "613x397,317x241", views=2, orbit=True, dist=5.0, half=2.0,
              s_lo=0.01, s_hi=0.1, sh=3, name="autograd_20k_sh3_odd"),
        # an optimisation step of a scene on a batch of four 720p views
        _case("train", 500_000, 8, "1280x720", views=4, orbit=True, bf16=True,
              name="train_500k_4x720p"),
        # an optimisation step of single-image fitting
        _case("train", 10_000, 4, "1920x871", loss="mse", name="fit_10k_1920x871"),
        # densification between optimisation steps
        _case("densify", 500_000, 8, "1280x720", name="densify_500k"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _res(rng, lo, hi):
    """A frame of lo..hi pixels (spread over the logarithm), of 4:3 to 16:9, mostly odd."""
    px, ratio = _log(rng, lo, hi), rng.uniform(1.0, 1.9)
    w = int(round(math.sqrt(px * ratio)))
    return "%dx%d" % (w, max(8, px // w))


def draw(rng):
    kind = rng.choice(["view", "view", "step", "step", "step", "step", "autograd", "train",
                       "train", "densify"])
    if kind == "densify":
        return _case("densify", _log(rng, 3000, 500_000), rng.choice([1, 2, 4, 8]), "1280x720")
    if kind == "train" and rng.random() < 0.5:
        return _case("train", _log(rng, 2000, 150_000), rng.choice([2, 4, 8]),
                     _res(rng, 50_000, 2_000_000), loss="mse")
    P = _log(rng, 1000, 1_000_000 if kind != "autograd" else 100_000)
    n = rng.choice([1, 1, 1, 2, 3, 4])
    res = ",".join(_res(rng, 12_000, 2_000_000 if P < 300_000 else 1_000_000) for _ in range(n))
    # the splats of a scene shrink as their number grows: s_hi covers the frame some tens of times
    s_hi = min(0.2, 3.0 / math.sqrt(P) * math.exp(rng.uniform(math.log(2.0), math.log(30.0))))
    s_lo = s_hi / rng.uniform(5.0, 25.0)
    N, sides, sh, bf16 = rng.choice([1, 2, 4, 4, 8, 8, 8, 16]), "", -1, rng.random() < 0.4
    if kind == "step" and rng.random() < 0.2:
        N, sides = rng.choice([(8, "2,4,8"), (8, "1,3,8"), (16, "4,8,16")])
    if kind in ("step", "autograd") and not sides and rng.random() < 0.3:
        sh = rng.choice([0, 1, 2, 3])
    if kind == "autograd":
        bf16 = False
    if kind == "train":
        N, sh, bf16 = rng.choice([2, 4, 8]), -1, rng.random() < 0.5
    return _case(kind, P, N, res, views=n, orbit=True, s_lo=s_lo, s_hi=s_hi, bf16=bf16,
                 sides=sides, sh=sh)


# ---- inputs ------------------------------------------------------------------------------------
class _View:
    """A pinhole camera: x right, y down, z forward, 60 degrees wide, float32 values."""

    def __init__(self, pos, width, height):
        f = np.zeros(3) - pos
        f /= np.linalg.norm(f)
        up = np.array([0.0, 1.0, 0.0]) if abs(f[1]) < 0.99 else np.array([1.0, 0.0, 0.0])
        r = np.cross(f, up)
        r /= np.linalg.norm(r)
        R = np.stack([r, np.cross(f, r), f])
        self.width, self.height = width, height
        self.fx = self.fy = float(np.float32(width / 2.0 / math.tan(math.radians(30.0))))
        self.cx, self.cy = width / 2.0, height / 2.0
        self.R, self.t = R.astype(np.float32), (-R @ pos).astype(np.float32)
        self.z_near = float(np.float32(0.01))


def _sizes(case):
    res = [tuple(int(x) for x in r.split("x")) for r in case["res"].split(",")]
    return [res[i % len(res)] for i in range(case["views"])]


def _views(case, seed, n=None):
    rng, out = np.random.default_rng(seed + 1), []
    sizes = _sizes(case)
    for i in range(n or case["views"]):
        d = rng.standard_normal(3)
        d = d / np.linalg.norm(d) if case["orbit"] else np.array([0.0, 0.0, -1.0])
        out.append(_View(case["dist"] * d, *sizes[i % len(sizes)]))
    return out


def _pixels(case):
    return sum(w * h for w, h in _sizes(case))


class _Draws:
    """Seeded float32 draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uniform(self, shape, lo=0.0, hi=1.0):
        x = torch.empty(shape, dtype=torch.float32, device="cuda")
        return x.uniform_(lo, hi, generator=self.g)

    def normal(self, shape, scale=1.0):
        x = torch.empty(shape, dtype=torch.float32, device="cuda")
        return x.normal_(0.0, scale, generator=self.g)

    def permutation(self, n):
        return torch.randperm(n, generator=self.g, device="cuda")


def _raw(case, seed):
    """Raw parameters of a scene (quaternions, log-scales, logits): centres in a box, scales
    uniform over their logarithm, opacities 0.05 to 0.95, texels 0 to 1."""
    d, P, N = _Draws(seed), case["P"], case["N"]
    raw = dict(means=d.uniform((P, 3), -case["half"], case["half"]), quats=d.normal((P, 4)),
               log_scales=d.uniform((P, 2), math.log(case["s_lo"]), math.log(case["s_hi"])))
    o = d.uniform((P,), 0.05, 0.95)
    raw["opacity_logits"] = torch.log(o / (1.0 - o))
    if not case["sides"]:
        raw["textures"] = d.uniform((P, N, N, 3))
    return raw, d


def _tangents(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    u = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y + w * z), 2 * (x * z - w * y)], 1)
    v = torch.stack([2 * (x * y - w * z), 1 - 2 * (x * x + z * z), 2 * (y * z + w * x)], 1)
    return u, v


def _scene(case, seed):
    """Activated parameters, as a dict of tensors in the argument order of ``gb.Splats``."""
    raw, d = _raw(case, seed)
    u, v = _tangents(raw["quats"])
    s = dict(means=raw["means"], tan_u=u.contiguous(), tan_v=v.contiguous(),
             scales=raw["log_scales"].exp(), opacity=torch.sigmoid(raw["opacity_logits"]))
    if case["sides"]:
        # equal shares of the sides, in random order
        sides = torch.tensor([int(x) for x in case["sides"].split(",")], device="cuda")
        n = sides[d.permutation(case["P"]) % len(sides)]
        s["textures"] = d.uniform((int((n * n).sum()), 3))
        s["tex_side"], s["layout_side"] = n.to(torch.int32), case["N"]
        s["tex_offset"] = (torch.cumsum(n * n, 0) - n * n).to(torch.int64)
    else:
        s["textures"] = raw["textures"]
    if case["bf16"]:
        s["textures"] = s["textures"].to(torch.bfloat16)
    if case["sh"] >= 0:
        s["sh"] = d.normal((case["P"], (case["sh"] + 1) ** 2, 3), 0.2)
    return s, d


class _Raw:
    """Raw parameters as the arrays that ``TrainState`` takes."""

    def __init__(self, raw):
        for k, v in raw.items():
            setattr(self, k, v.cpu().numpy())


def _image(d, w, h):
    """A smooth random picture with some fine texture, [h * w, 3] in 0..1."""
    low = d.uniform((1, 3, 9, 12))
    img = torch.nn.functional.interpolate(low, size=(h, w), mode="bicubic", align_corners=True)
    img = img[0].permute(1, 2, 0).reshape(-1, 3) + d.normal((h * w, 3), 0.03)
    return img.clamp_(0.0, 1.0).contiguous()


def _fit_raw(case, seed, view):
    """Single-image fitting: splats on the plane z = 1 before an identity camera, rotated about z
    only, their scales such that together they cover the picture about once."""
    d, P, N = _Draws(seed), case["P"], case["N"]
    half_w, half_h = view.width / 2 / view.fx, view.height / 2 / view.fy
    means = torch.ones((P, 3), device="cuda")
    means[:, 0] = d.uniform((P,), -half_w, half_w)
    means[:, 1] = d.uniform((P,), -half_h, half_h)
    a, zero = d.uniform((P,), 0.0, math.pi), torch.zeros(P, device="cuda")
    px = math.sqrt(view.width * view.height / P) / view.fx
    o = d.uniform((P,), 0.3, 0.9)
    return dict(means=means, quats=torch.stack([a.cos(), zero, zero, a.sin()], 1),
                log_scales=(d.uniform((P, 2), 0.5, 1.5) * px).log(),
                opacity_logits=torch.log(o / (1.0 - o)), textures=d.uniform((P, N, N, 3))), d


def _prepare_train(case, seed):
    if case["loss"] == "mse":
        w, h = _sizes(case)[0]
        view = _View(np.array([0.0, 0.0, -1.0]), w, h)
        view.R, view.t = np.eye(3, dtype=np.float32), np.zeros(3, dtype=np.float32)
        raw, d = _fit_raw(case, seed, view)
        state = gbt.TrainState(_Raw(raw), bf16=case["bf16"], rotz_only=True)
        trainer = gbt.Trainer(state, [view], _image(d, w, h)[None], loss="mse")
        batches = [[0]]
    else:
        raw, d = _raw(case, seed)
        views = _views(case, seed, 2 * case["views"])
        most = max(v.width * v.height for v in views)
        targets = torch.zeros((len(views), most, 3), device="cuda")
        for t, v in zip(targets, views):
            t[:v.width * v.height] = _image(d, v.width, v.height)
        state = gbt.TrainState(_Raw(raw), bf16=case["bf16"])
        trainer = gbt.Trainer(state, views, targets)
        n = case["views"]
        batches = [list(range(n)), list(range(n, 2 * n))]
    trainer.plan(batches, headroom=2.0)
    return dict(trainer=trainer, batches=batches, at=0)


def _prepare_densify(case, seed):
    """A training state with moments and an accumulated statistic: a tenth of the splats over
    the threshold, most of those large enough to split, one in fifty too transparent to keep."""
    raw, d = _raw(case, seed)
    P = case["P"]
    mixed = d.permutation(P)
    gone, dense = mixed[:P // 50], mixed[P // 50:P // 50 + P // 10]
    o = d.uniform((P,), 0.08, 0.95)
    o[gone] = d.uniform((len(gone),), 0.01, 0.06)
    raw["opacity_logits"] = torch.log(o / (1.0 - o))
    state = gbt.TrainState(_Raw(raw), bf16=True)
    state.m = {k: d.normal(tuple(t.shape), 1e-3) for k, t in state.m.items()}
    state.v = {k: d.uniform(tuple(t.shape), 0.0, 1e-6) for k, t in state.v.items()}
    vis = d.uniform((P,), 1.0, 40.0).floor()
    mean = d.uniform((P,), 0.0, 1.9e-4)
    mean[dense] = d.uniform((len(dense),), 2.1e-4, 6e-4)
    return dict(state=state, accum=vis * mean, vis=vis, noise=d.normal((P, 2, 2)),
                options=gbt.DensifyOptions(dense_scale=0.04, min_opacity=0.07),
                before=(state.params, state.m, state.v, P))


def prepare(case, seed):
    if case["kind"] == "train":
        return dict(_prepare_train(case, seed), kind="train")
    if case["kind"] == "densify":
        return dict(_prepare_densify(case, seed), kind="densify")
    scene, d = _scene(case, seed)
    views = _views(case, seed)
    g = d.normal((_pixels(case), 3))
    if case["kind"] == "autograd":
        params = {k: v.requires_grad_() for k, v in scene.items()}
        rast = gb.Rasterizer(views)
        rast.plan(gb.Splats(**{k: v.detach() for k, v in scene.items()}))
        return dict(kind="autograd", rast=rast, params=params, g=g)
    sp = gb.Splats(**scene)
    rast = gb.Rasterizer(views, check_overflow=False)
    rast.plan(sp)
    rgb, T = torch.empty_like(g), torch.empty(g.shape[0], device="cuda")
    state = dict(kind=case["kind"], rast=rast, sp=sp, g=g, rgb=rgb, T=T)
    if case["kind"] == "step":
        grads = {k: torch.empty(scene[k].shape, device="cuda")
                 for k in ("means", "tan_u", "tan_v", "scales", "opacity", "textures")}
        if case["sh"] >= 0:
            grads["sh"] = torch.empty_like(scene["sh"])
        state["grads"] = grads
    return state


def run(state):
    kind = state["kind"]
    if kind == "view":
        return state["rast"].forward(state["sp"], state["rgb"], state["T"])
    if kind == "step":
        r, sp, grads = state["rast"], state["sp"], state["grads"]
        rgb, T = r.forward(sp, state["rgb"], state["T"], zero_grads=grads)
        return rgb, T, r.backward(sp, T, state["g"], grads)
    if kind == "autograd":
        params = state["params"]
        rgb, T = gb.render(state["rast"], **params)
        grads = torch.autograd.grad(rgb, list(params.values()), state["g"])
        return rgb.detach(), T, dict(zip(params, grads))
    if kind == "train":
        trainer, batches = state["trainer"], state["batches"]
        loss = trainer.step(batches[state["at"] % len(batches)])
        state["at"] += 1
        return dict(loss=loss, grads=dict(trainer.state.raw_grads), params=trainer.state.params)
    s = state["state"]
    s.params, s.m, s.v, s.P = state["before"]
    n = s.densify(state["accum"], state["vis"], state["options"], state["noise"])
    return dict(n=n, params=s.params, m=s.m, v=s.v)


# ---- work ----------------------------------------------------------------------------------------
def _blended(case):
    """An estimate of the (pixel, splat) pairs a render blends: the splats' area above the
    opacity threshold at the scene's distance, seen at a mean tilt of one half, up to the about
    70 pairs per pixel after which a pixel is opaque."""
    w = math.log(case["s_hi"] / case["s_lo"])
    mean_s = (case["s_hi"] - case["s_lo"]) / w  # mean of a scale that is log-uniform
    area = 0.0
    for width, height in _sizes(case):
        if case["loss"] == "mse" and case["kind"] == "train":
            area += 15.0 * width * height
            continue
        f = width / 2 / math.tan(math.radians(30.0)) / case["dist"]
        per_splat = math.pi * 2 * math.log(255.0 * 0.4) * 0.5 * (mean_s * f) ** 2 + 6.0
        frame = (2 * case["half"] * f) ** 2  # the box's face, in pixels
        inside = min(1.0, width * height / frame)
        area += min(70.0 * width * height, case["P"] * inside * per_splat)
    return area


def work(case):
    P, N, px = case["P"], case["N"], _pixels(case)
    if case["sides"]:
        sides = [int(x) for x in case["sides"].split(",")]
        texels = P * sum(n * n for n in sides) / len(sides)
    else:
        texels = P * N * N
    per = 13 + 3 * texels / P  # floats of a splat's raw or activated parameters, about
    if case["kind"] == "densify":
        return {"bytes": 2 * 3 * 4.0 * P * per, "flops": 10.0 * P * per}
    tex_bytes = texels * 3 * (2 if case["bf16"] else 4)
    sh = 12.0 * (case["sh"] + 1) ** 2 * P
    fwd = 48.0 * P + tex_bytes + sh + 16.0 * px
    pairs = _blended(case)
    if case["kind"] == "view":
        return {"bytes": fwd, "flops": 78.0 * pairs}
    bwd = 48.0 * P + 12.0 * texels + sh + 28.0 * px
    total, flops = fwd + bwd, (78.0 + 177.0) * pairs
    if case["kind"] == "train":
        # the loss reads the targets; Adam reads and writes parameters and moments
        total += 24.0 * px + P * per * (28.0 + (2 if case["bf16"] else 0))
        flops += 12.0 * P * per
    return {"bytes": total, "flops": flops}


# ---- float64 -------------------------------------------------------------------------------------
def _sh_basis(d):
    """Real spherical harmonics of degree <= 3 with signs (-1)^m, at unit directions [n, 3]."""
    x, y, z = d.unbind(1)
    xx, yy, zz = x * x, y * y, z * z
    c = lambda v: math.sqrt(v / math.pi)
    out = [torch.full_like(x, 0.5 * c(1.0)), -c(0.75) * y, c(0.75) * z, -c(0.75) * x,
           c(15 / 4) * x * y, -c(15 / 4) * y * z, c(5 / 16) * (2 * zz - xx - yy),
           -c(15 / 4) * x * z, c(15 / 16) * (xx - yy),
           -c(35 / 32) * y * (3 * xx - yy), c(105 / 4) * x * y * z,
           -c(21 / 32) * y * (4 * zz - xx - yy), c(7 / 16) * z * (2 * zz - 3 * xx - 3 * yy),
           -c(21 / 32) * x * (4 * zz - xx - yy), c(105 / 16) * z * (xx - yy),
           -c(35 / 32) * x * (xx - 3 * yy)]
    return torch.stack(out, 1)


def _exact_cell(s, view, x, y, N, sh):
    """Colour and transmittance at pixel centres x, y (float64) of depth-ordered splats."""
    R = torch.tensor(view.R, dtype=torch.float64, device="cuda")
    t = torch.tensor(view.t, dtype=torch.float64, device="cuda")
    a = (s["scales"][:, :1] * s["tan_u"]) @ R.T
    b = (s["scales"][:, 1:] * s["tan_v"]) @ R.T
    p = s["means"] @ R.T + t
    K = lambda q: (view.fx * q[:, 0] + view.cx * q[:, 2], view.fy * q[:, 1] + view.cy * q[:, 2],
                   q[:, 2])
    M = [torch.stack(c, 1) for c in zip(K(a), K(b), K(p))]  # rows of the screen matrix, [n, 3]
    hx = x[:, None, None] * M[2] - M[0]
    hy = y[:, None, None] * M[2] - M[1]
    rho = torch.linalg.cross(hx, hy)
    ok = rho[..., 2] != 0
    r2 = torch.where(ok, rho[..., 2], torch.ones_like(rho[..., 2]))
    u, v = rho[..., 0] / r2, rho[..., 1] / r2
    c2x, c2y = M[0][:, 2] / M[2][:, 2], M[1][:, 2] / M[2][:, 2]
    q_uv = 0.5 * (u * u + v * v)
    q_lp = ((x[:, None] - c2x) ** 2 + (y[:, None] - c2y) ** 2) / (2 * LP_VAR)
    q = torch.where(q_uv <= q_lp, q_uv, q_lp)
    alpha = (s["opacity"] * torch.exp(-q)).clamp(max=float(np.float32(ALPHA_MAX)))
    mask = ok & (alpha.detach() >= float(np.float32(ALPHA_MIN)))
    alpha = torch.where(mask, alpha, torch.zeros_like(alpha))
    cum = torch.cumsum(torch.log1p(-alpha), 1)
    keep = mask & (torch.exp(cum.detach()) >= float(np.float32(T_MIN)))
    alpha = torch.where(keep, alpha, torch.zeros_like(alpha))
    cum = torch.cumsum(torch.log1p(-alpha), 1)
    before = torch.exp(cum - torch.log1p(-alpha))
    tex = s["textures"]
    if N == 1:
        col = tex[:, 0, 0][None].expand(len(x), -1, -1)
    else:
        grid = lambda w: ((w + SIGMA) * ((N - 1) / (2 * SIGMA))).clamp(0, N - 1)
        gu, gv = grid(u), grid(v)
        iu = gu.detach().floor().clamp(max=N - 2).long()
        iv = gv.detach().floor().clamp(max=N - 2).long()
        fu, fv = (gu - iu)[..., None], (gv - iv)[..., None]
        k, flat = torch.arange(len(tex), device="cuda")[None], tex.reshape(-1, 3)
        at = lambda i, j: flat[(k * N + iu + i) * N + iv + j]
        col = (1 - fu) * ((1 - fv) * at(0, 0) + fv * at(0, 1)) + \
            fu * ((1 - fv) * at(1, 0) + fv * at(1, 1))
    if sh >= 0:
        d = s["means"] + t @ R
        d = d / d.norm(dim=1, keepdim=True)
        n = (sh + 1) ** 2
        col = col + (_sh_basis(d)[:, :n, None] * s["sh"]).sum(1)
    rgb = ((alpha * before)[..., None] * col).sum(1)
    return rgb, torch.exp(cum[:, -1])


def _exact_render(scene, views, N, sh, g=None):
    """rgb, T and, with g, the gradients of sum(g * rgb): float64 torch autograd over cells of
    32 x 32 pixels and the splats whose bounds touch them."""
    full = {k: v.detach().double() for k, v in scene.items()}
    grads = {k: torch.zeros_like(v) for k, v in full.items()} if g is not None else None
    rgbs, Ts, base, side = [], [], 0, 32
    for view in views:
        R = torch.tensor(view.R, dtype=torch.float64, device="cuda")
        t = torch.tensor(view.t, dtype=torch.float64, device="cuda")
        p = full["means"] @ R.T + t
        a = 3.33 * (full["scales"][:, :1] * full["tan_u"]) @ R.T
        b = 3.33 * (full["scales"][:, 1:] * full["tan_v"]) @ R.T
        q = torch.stack([p + a + b, p + a - b, p - a + b, p - a - b, p])
        near = (q[..., 2] <= view.z_near).any(0)
        px = view.fx * q[..., 0] / q[..., 2] + view.cx
        py = view.fy * q[..., 1] / q[..., 2] + view.cy
        x0, x1, y0, y1 = px.amin(0) - 3, px.amax(0) + 3, py.amin(0) - 3, py.amax(0) + 3
        seen = (p[:, 2] > view.z_near) & (full["opacity"] >= float(np.float32(ALPHA_MIN)))
        order = torch.argsort(p[:, 2], stable=True)
        order = order[seen[order]]
        rgb = torch.zeros((view.height, view.width, 3), dtype=torch.float64, device="cuda")
        T = torch.ones((view.height, view.width), dtype=torch.float64, device="cuda")
        gv = None if g is None else \
            g[base:base + view.width * view.height].double().view(view.height, view.width, 3)
        base += view.width * view.height
        for j in range(0, view.height, side):
            for i in range(0, view.width, side):
                jj, ii = min(j + side, view.height), min(i + side, view.width)
                hit = near | ((x1 >= i) & (x0 <= ii) & (y1 >= j) & (y0 <= jj))
                idx = order[hit[order]]
                if not len(idx):
                    continue
                yy, xx = torch.meshgrid(
                    torch.arange(j, jj, dtype=torch.float64, device="cuda") + 0.5,
                    torch.arange(i, ii, dtype=torch.float64, device="cuda") + 0.5, indexing="ij")
                # rows of a cell in pieces that keep the temporaries at a few million values
                rows = max(1, (1 << 21) // (len(idx) * (ii - i)))
                for r in range(0, jj - j, rows):
                    part = {k: v[idx].requires_grad_(g is not None) for k, v in full.items()}
                    x, y = xx[r:r + rows].reshape(-1), yy[r:r + rows].reshape(-1)
                    c, tr = _exact_cell(part, view, x, y, N, sh)
                    r1 = min(j + r + rows, jj)
                    rgb[j + r:r1, i:ii] = c.detach().view(-1, ii - i, 3)
                    T[j + r:r1, i:ii] = tr.detach().view(-1, ii - i)
                    if g is not None:
                        gc = gv[j + r:r1, i:ii].reshape(-1, 3)
                        got = torch.autograd.grad(c, list(part.values()), gc)
                        for k, d in zip(part, got):
                            grads[k].index_add_(0, idx, d)
        rgbs.append(rgb.view(-1, 3))
        Ts.append(T.view(-1))
    return torch.cat(rgbs), torch.cat(Ts), grads


def _exact_densify(case, seed):
    st = _prepare_densify(case, seed)
    par, m, v, P = st["before"]
    o, noise = st["options"], st["noise"].double()
    ls = par["log_scales"].amax(1)
    dense = st["accum"] / st["vis"].clamp(min=1) >= np.float32(o.grad_threshold)
    gone = par["opacity_logits"] < np.float32(math.log(o.min_opacity / (1 - o.min_opacity)))
    split = dense & (ls > np.float32(math.log(o.dense_scale)))
    n = torch.where(gone, 0, torch.where(dense, 2, 1))
    parent = torch.repeat_interleave(torch.arange(P, device="cuda"), n)
    start = torch.cumsum(n, 0) - n
    second = torch.arange(len(parent), device="cuda") - start[parent]
    child, kept = split[parent], ~split[parent] & (second == 0)
    out = {k: t.double()[parent] for k, t in par.items()}
    z = noise[parent, second]
    tu, tv = _tangents(out["quats"])
    s = out["log_scales"].exp()
    moved = out["means"] + s[:, :1] * z[:, :1] * tu + s[:, 1:] * z[:, 1:] * tv
    out["means"] = torch.where(child[:, None], moved, out["means"])
    shrunk = out["log_scales"] - math.log(o.split_shrink)
    out["log_scales"] = torch.where(child[:, None], shrunk, out["log_scales"])
    N, idx = case["N"], torch.nonzero(child)[:, 0]
    if N > 1:
        at = torch.linspace(-SIGMA, SIGMA, N, dtype=torch.float64, device="cuda")
        for part in idx.split(1 << 16):
            g = (z[part][:, :, None] + at / o.split_shrink + SIGMA) * ((N - 1) / (2 * SIGMA))
            g = g.clamp(0, N - 1)
            i = g.floor().clamp(max=N - 2).long()
            f = (g - i)[..., None]
            tex, row = out["textures"][part], torch.arange(len(part), device="cuda")[:, None]
            rows = (1 - f[:, 0, :, None]) * tex[row, i[:, 0]] + f[:, 0, :, None] * tex[row, i[:, 0] + 1]
            rows = rows.transpose(1, 2)
            cols = (1 - f[:, 1, :, None]) * rows[row, i[:, 1]] + f[:, 1, :, None] * rows[row, i[:, 1] + 1]
            out["textures"][part] = cols.transpose(1, 2)
    rows = lambda t: t.double()[parent] * kept.view(-1, *[1] * (t.dim() - 1))
    return dict(n=None, params=out, m={k: rows(t) for k, t in m.items()},
                v={k: rows(t) for k, t in v.items()})


def exact(case, seed):
    """float64 results of renders of up to about 100k splats and of densification; None for the
    larger renders and the optimisation steps (which end in Adam's division by a tiny root)."""
    if case["kind"] == "densify":
        return _exact_densify(case, seed) if case["P"] * case["N"] ** 2 <= 500_000 * 64 else None
    if case["kind"] == "train" or case["sides"] or case["P"] * case["views"] > 100_000:
        return None
    if _blended(case) > 3e8 or _pixels(case) > 1_500_000:
        return None
    scene, d = _scene(case, seed)
    g = d.normal((_pixels(case), 3))
    rgb, T, grads = _exact_render(scene, _views(case, seed), case["N"], case["sh"],
                                  None if case["kind"] == "view" else g)
    return (rgb, T) if grads is None else (rgb, T, grads)
