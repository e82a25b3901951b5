"""Performance cases of the Gaussian ray marcher.

Each case is one piece of work that a program does with the framework, through
its public entry points (`Renderer`, `render`, `TrainStep`, `Adam`,
`isotropic_loss`): frames of a scene whose structure is already built, a
preview after the parameters changed, training steps (rebuild, forward, loss,
backward) from a debugging size up to a million Gaussians, a graph-captured
step, the densification statistic and the optimizer.  Scenes follow the
recipes of `paper_2509_07782_amd/inputs.py` (uniform, clustered, outdoor
layout), drawn on the GPU; every number of an input follows from the seed.

A case holds
  path        frame | preview | train | captured | densify | optimizer
  scene       uniform | cluster | outdoor
  n           Gaussians
  deg, n_sg   SH degree, spherical-Gaussian lobes per Gaussian
  views, width, height
  adaptive    Eq. 5 step sizes, else the fixed step `dt`
  n_s         samples per segment
  persistent  one persistent launch over all tiles
  lean        record no per-sample sums (half the record pool)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2509_07782_amd import inputs
from paper_2509_07782_amd.render import (Adam, RenderOptions, Renderer, TrainStep, isotropic_loss,
                                         render)

SIGMA_EPS = 0.01
T_EPS = 1e-4
ADAPTIVE = dict(dt_min=0.005, dt_max=0.02, beta=1024.0)
SH_C0 = 0.28209479177387814
KEYS = ("means", "log_scales", "quats", "density", "sh")

# Distinct Gaussians a ray meets, as a share of the scene (statistics pass of
# the three layouts), for the operations of work().
RAY_SHARE = {"uniform": 1e-2, "cluster": 2.5e-4, "outdoor": 5e-4}


def _case(path, scene, n, deg, views, width, height, adaptive=True, dt=0.0025, n_s=8, n_sg=0,
          persistent=True, lean=False):
    return dict(path=path, scene=scene, n=n, deg=deg, n_sg=n_sg, views=views, width=width,
                height=height, adaptive=adaptive, dt=dt, n_s=n_s, persistent=persistent, lean=lean)


def listed():
    c = {
        # the smallest frame: a thumbnail of a toy scene, where launches and
        # one tile's latency are all there is
        "frame_64": _case("frame", "uniform", 1_000, 0, 1, 64, 64, adaptive=False, dt=0.01,
                          persistent=False),
        # a debugging-size training step on a ragged view (the size of the
        # gradient tests); every step rebuilds the structure
        "train_67x45": _case("train", "cluster", 2_000, 3, 1, 67, 45, persistent=False),
        # a test view of a synthetic object: uniform step, one 800x800 frame
        "frame_object": _case("frame", "cluster", 100_000, 3, 1, 800, 800, adaptive=False),
        # a full-HD frame of a trained scene, as an interactive viewer asks for
        "frame_hd": _case("frame", "cluster", 1_000_000, 3, 1, 1920, 1080),
        # an outdoor test view: the camera stands inside the dense part
        "frame_outdoor": _case("frame", "outdoor", 3_000_000, 3, 1, 1297, 840),
        # a small preview of a large scene after its parameters changed (the
        # viewer beside a training run): the rebuild is most of it
        "preview_5m": _case("preview", "cluster", 5_000_000, 3, 1, 257, 193),
        # the headline training step: rebuild, four views, loss, backward
        "train_1m": _case("train", "cluster", 1_000_000, 3, 4, 1024, 768),
        # outdoor training step on one view, the batch most trainers use
        "train_outdoor": _case("train", "outdoor", 3_000_000, 3, 1, 1297, 840),
        # the 9 SH + 7 SG appearance model on a ragged half-size view
        "train_lobes": _case("train", "cluster", 100_000, 2, 1, 401, 299, n_sg=7),
        # the graph-captured step over a batch of small views
        "captured_views": _case("captured", "outdoor", 300_000, 3, 6, 320, 213),
        # the step before a densification: per-view mean-gradient statistic
        "densify_8": _case("densify", "cluster", 100_000, 3, 8, 160, 121),
        # isotropic scale loss and the Adam update of a million Gaussians
        "optimizer_1m": _case("optimizer", "cluster", 1_000_000, 3, 1, 1, 1),
    }
    return [dict(v, name=k) for k, v in c.items()]


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm,
    odd ones among them, no costlier than the largest listed one."""
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["frame", "frame", "preview", "train", "train", "captured", "densify",
                       "optimizer"])
    scene = rng.choice(["uniform", "cluster", "cluster", "outdoor"])
    if path == "optimizer":
        return _case(path, "cluster", logu(1_000, 3_000_000), rng.choice([0, 1, 2, 3]), 1, 1, 1)
    n = logu(1_000, {"uniform": 10_000, "cluster": 2_000_000, "outdoor": 3_000_000}[scene])
    if path == "preview":
        n = logu(2_000, 5_000_000)
        scene = "cluster"
    width = logu(33, 1920)
    height = max(17, min(1080, int(width * rng.uniform(0.5, 1.0))))
    views = 1
    if path in ("train", "captured", "densify"):
        views = rng.choice([1, 1, 2, 3, 4, 8])
        most = 1_000_000 if scene != "outdoor" else 400_000
        while views * width * height > most:
            width, height = max(33, int(width * 0.8)), max(17, int(height * 0.8))
    if path == "preview":
        width, height = min(width, 640), min(height, 480)
    n_sg = rng.choice([0, 0, 0, 3, 7]) if n <= 200_000 and path in ("frame", "train") else 0
    deg = rng.choice([0, 1, 2, 3, 3, 3])
    adaptive = rng.random() < 0.7
    # fixed steps are the synthetic scenes' mode; an outdoor ray is 128 long
    if scene == "outdoor":
        adaptive = True
    dt = rng.choice([0.0025, 0.005, 0.01])
    n_s = 8 if n_sg else rng.choice([4, 8, 8, 8, 16])
    return _case(path, scene, n, deg, views, width, height, adaptive=adaptive, dt=dt, n_s=n_s,
                 n_sg=n_sg, persistent=rng.random() < 0.6,
                 lean=path in ("train", "captured") and rng.random() < 0.25)


# ----------------------------------------------------------------------------
# inputs


def _ball_mixture(g, n, dev):
    """32 isotropic normals (sd 0.2) centred in the unit ball; points outside
    the unit ball are drawn again."""
    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev, dtype=torch.float64)

    c = normal(32, 3)
    c /= c.norm(dim=1, keepdim=True)
    c *= torch.rand(32, 1, generator=g, device=dev, dtype=torch.float64) ** (1.0 / 3.0)
    out = torch.empty(n, 3, device=dev, dtype=torch.float64)
    todo = torch.arange(n, device=dev)
    while todo.numel():
        comp = torch.randint(0, 32, (todo.numel(),), generator=g, device=dev)
        x = c[comp] + 0.2 * normal(todo.numel(), 3)
        ok = (x * x).sum(1) <= 1.0
        out[todo[ok]] = x[ok]
        todo = todo[~ok]
    return out


def _scene(case, g, dev):
    """Parameter tensors (float32, device) of the case's scene."""
    n, deg = int(case["n"]), int(case["deg"])

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev, dtype=torch.float64)

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, generator=g, device=dev, dtype=torch.float64)

    if case["scene"] == "uniform":
        means = uniform(-1.0, 1.0, n, 3)
        ls = -3.0 + 0.3 * normal(n, 3)
    elif case["scene"] == "cluster":
        means = _ball_mixture(g, n, dev)
        ls = -4.0 + 0.5 * normal(n, 3)
    else:
        n_in = int(round(0.7 * n))
        r = uniform(2.0, 50.0, n - n_in)
        u = normal(n - n_in, 3)
        shell = u / u.norm(dim=1, keepdim=True) * r[:, None]
        means = torch.cat([_ball_mixture(g, n_in, dev), shell])
        ls = -4.0 + 0.5 * normal(n, 3)
        ls[n_in:] += r.log()[:, None]
    q = normal(n, 4)
    q /= q.norm(dim=1, keepdim=True)
    density = 10.0 * torch.nn.functional.softplus(normal(n))
    k = (deg + 1) ** 2
    if case["scene"] == "uniform" and deg == 0:
        sh = uniform(0.0, 1.0, n, 1, 3) / SH_C0
    else:
        sh = 0.2 * torch.randn(n, k, 3, generator=g, device=dev, dtype=torch.float32)
    p = dict(means=means, log_scales=ls, quats=q, density=density, sh=sh)
    if case["n_sg"]:
        m = int(case["n_sg"])
        ax = normal(n, m, 3)
        ax *= uniform(0.5, 2.0, n, m, 1) / ax.norm(dim=2, keepdim=True)
        p["sg"] = torch.cat([0.2 * normal(n, m, 3), ax, uniform(1.0, 30.0, n, m, 1)], dim=2)
    return {k: v.to(torch.float32).contiguous() for k, v in p.items()}


def _cameras(case, seed):
    """Views on an orbit (radius 3, or 0.5 and inside the ball outdoors), the
    first azimuth drawn from the seed."""
    rng = np.random.default_rng(seed)
    out, (w, h) = [], (int(case["width"]), int(case["height"]))
    radius, t_far = (0.5, 128.0) if case["scene"] == "outdoor" else (3.0, 6.0)
    az0 = rng.uniform(0.0, 2.0 * math.pi)
    for v in range(int(case["views"])):
        a = az0 + 2.0 * math.pi * v / int(case["views"])
        eye = np.array([radius * math.sin(a), 0.0, radius * math.cos(a)])
        fwd = -eye / np.linalg.norm(eye)
        right = np.cross(fwd, (0.0, 1.0, 0.0))
        right /= np.linalg.norm(right)
        c2w = np.stack([right, np.cross(fwd, right), fwd, eye], axis=1).astype(np.float32)
        f = float(np.float32(w / (2.0 * math.tan(math.radians(30.0)))))
        out.append(inputs.Camera(w, h, f, f, w / 2.0, h / 2.0, c2w, 0.0, t_far))
    return out


def _options(case):
    return RenderOptions(adaptive=bool(case["adaptive"]), dt=float(case["dt"]),
                         n_s=int(case["n_s"]), t_eps=T_EPS, ess=1,
                         persistent=bool(case["persistent"]), no_sample_record=bool(case["lean"]),
                         **ADAPTIVE)


def _rays(case):
    return int(case["views"]) * int(case["width"]) * int(case["height"])


def _inputs(case, seed):
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    params = _scene(case, g, dev)
    if case["path"] == "optimizer":
        grads = {k: 1e-3 * torch.randn(v.shape, generator=g, device=dev) for k, v in params.items()}
        return params, grads, None
    target = torch.rand(_rays(case), 3, generator=g, device=dev)
    return params, target, _cameras(case, seed)


# ----------------------------------------------------------------------------
# the cases


def prepare(case, seed):
    params, other, cams = _inputs(case, seed)
    path = case["path"]
    s = dict(path=path, params=params, deg=int(case["deg"]), renderer=Renderer(0))
    if path == "optimizer":
        for k, p in params.items():
            p.grad = other[k]
        s["adam"] = Adam(s["renderer"], params)
        s["ls"] = params["log_scales"].clone().requires_grad_(True)
        return s
    s.update(cams=cams, opts=_options(case), target=other)
    if path == "frame":
        s["renderer"].build(params, s["deg"])
    elif path in ("train", "captured"):
        for p in params.values():
            p.requires_grad_(True)
    if path == "captured":
        target = other
        s["step"] = TrainStep(s["renderer"], params, s["deg"], cams, s["opts"],
                              lambda rgb, T: ((rgb - target) ** 2).mean())
    elif path == "densify":
        s["state"] = s["renderer"].new_state()
    return s


def run(s):
    path, r, params = s["path"], s["renderer"], s["params"]
    if path == "frame":
        rgb, T = r.forward(s["cams"], s["opts"])
        return {"rgb": rgb, "T": T}
    if path == "preview":
        r.build(params, s["deg"], force=True)
        rgb, T = r.forward(s["cams"], s["opts"])
        return {"rgb": rgb, "T": T}
    if path == "train":
        for p in params.values():
            p.grad = None
        r.build(params, s["deg"], force=True)      # the last update changed the parameters
        rgb, T = render(params, s["deg"], r, s["cams"], s["opts"])
        loss = ((rgb - s["target"]) ** 2).mean()
        loss.backward()
        return {"loss": loss.detach(), "rgb": rgb.detach(), "T": T.detach(),
                "grads": {k: p.grad for k, p in params.items()}}
    if path == "captured":
        step = s["step"]
        loss = step.replay()
        return {"loss": loss, "rgb": step.rgb, "T": step.T, "grads": dict(step.grads)}
    if path == "densify":
        r.build(params, s["deg"], force=True)
        rgb, T = r.forward(s["cams"], s["opts"], state=s["state"])
        n = params["density"].shape[0]
        stat = torch.zeros(n, device=rgb.device)
        seen = torch.zeros(n, device=rgb.device, dtype=torch.int32)
        grad_rgb = (rgb - s["target"]) * (2.0 / rgb.numel())
        grads = r.backward(s["state"], rgb, T, grad_rgb, None, params, stat, seen)
        return {"rgb": rgb, "T": T, "grads": grads, "densify": stat, "views": seen}
    # optimizer: the scale loss with its gradient, and one Adam step
    s["ls"].grad = None
    loss = isotropic_loss(s["ls"], r)
    loss.backward()
    s["adam"].step()
    return {"loss": loss.detach(), "grad": s["ls"].grad, "params": dict(params),
            "m": dict(s["adam"].m), "v": dict(s["adam"].v)}


def work(case):
    """Bytes: parameters read once, gradients or moments written once, pixels
    in and out once.  Operations: per (ray, Gaussian) pair the chord (45), the
    colour (6 per coefficient) and the N_s samples' weights and sums (13
    each), three times that with a backward; per Gaussian about 300 for a
    rebuild."""
    n, k = float(case["n"]), (int(case["deg"]) + 1) ** 2
    rec = 4.0 * (11 + 3 * k + 7 * int(case["n_sg"]))
    path, rays = case["path"], float(_rays(case))
    if path == "optimizer":
        return {"bytes": n * rec * 7 + n * 24, "flops": n * (rec / 4 * 12 + 40)}
    pairs = rays * n * RAY_SHARE[case["scene"]]
    per = 45 + 6 * k + 10 * int(case["n_sg"]) + 13 * int(case["n_s"])
    if path == "frame":
        return {"bytes": n * rec + rays * 16, "flops": pairs * per}
    if path == "preview":
        return {"bytes": n * rec + rays * 16, "flops": pairs * per + 300 * n}
    return {"bytes": 2 * n * rec + rays * 28 + (8 * n if path == "densify" else 0),
            "flops": 3 * pairs * per + 300 * n}


# ----------------------------------------------------------------------------
# the same in 64 bits, in plain torch: every ray against every Gaussian


def _sh_basis64(deg, d):
    """Real spherical harmonics (Condon-Shortley phase), index l^2 + l + m."""
    x, y, z = d.unbind(1)
    out = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if deg >= 1:
        c = math.sqrt(3.0 / (4.0 * math.pi))
        out += [-c * y, c * z, -c * x]
    if deg >= 2:
        c = 0.5 * math.sqrt(15.0 / math.pi)
        out += [c * x * y, -c * y * z, 0.25 * math.sqrt(5.0 / math.pi) * (3 * z * z - 1),
                -c * x * z, 0.5 * c * (x * x - y * y)]
    if deg >= 3:
        a, b = 0.25 * math.sqrt(35.0 / (2.0 * math.pi)), 0.25 * math.sqrt(21.0 / (2.0 * math.pi))
        c = 0.5 * math.sqrt(105.0 / math.pi)
        out += [-a * y * (3 * x * x - y * y), c * x * y * z, -b * y * (5 * z * z - 1),
                0.25 * math.sqrt(7.0 / math.pi) * z * (5 * z * z - 3), -b * x * (5 * z * z - 1),
                0.5 * c * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(out, 1)


def _geometry64(p):
    """M = S^-1 R^T and k^2 of every Gaussian (differentiable)."""
    q = p["quats"] / p["quats"].norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                    1).view(-1, 3, 3)
    return R.transpose(1, 2) * torch.exp(-p["log_scales"])[:, :, None]


def _rays64(cam, dev):
    c2w = torch.from_numpy(np.asarray(cam.cam_to_world, np.float64)).to(dev)
    v, u = torch.meshgrid(torch.arange(cam.height, device=dev, dtype=torch.float64),
                          torch.arange(cam.width, device=dev, dtype=torch.float64), indexing="ij")
    local = torch.stack([(u.reshape(-1) + 0.5 - cam.cx) / cam.fx,
                         (v.reshape(-1) + 0.5 - cam.cy) / cam.fy,
                         torch.ones(cam.width * cam.height, device=dev, dtype=torch.float64)], 1)
    d = local @ c2w[:, :3].T
    return c2w[:, 3], d / d.norm(dim=1, keepdim=True)


def _f32(x):
    return float(np.float32(x))


def _march64(case, p, cam, o, d):
    """(rgb, T) of the rays, Algorithm 1 in 64 bits; differentiable in p (the
    sample schedule and the truncation are constants)."""
    dev, r, n_s = d.device, d.shape[0], int(case["n_s"])
    eps = _f32(SIGMA_EPS)
    dt_min, dt_max = _f32(ADAPTIVE["dt_min"]), _f32(ADAPTIVE["dt_max"])
    tn, tf = float(cam.t_near), float(cam.t_far)
    M, sig = _geometry64(p), p["density"]
    with torch.no_grad():
        active = sig > eps
        k2 = 2.0 * torch.log(torch.where(active, sig, 1.0) / eps)
        op = (M @ (o - p["means"])[:, :, None])[:, :, 0]
        S = M.transpose(1, 2) @ M
        six = torch.stack([S[:, 0, 0], S[:, 1, 1], S[:, 2, 2], 2 * S[:, 0, 1], 2 * S[:, 0, 2],
                           2 * S[:, 1, 2]], 0)
        bvec = (M.transpose(1, 2) @ op[:, :, None])[:, :, 0].T.contiguous()
        c2 = (op * op).sum(1)
        x, y, z = d.unbind(1)
        dd = torch.stack([x * x, y * y, z * z, x * y, x * z, y * z], 1)
        # every ray against every Gaussian, some rays at a time
        pr, pg, pin, pout = [], [], [], []
        step = max(1, int(2e8 // sig.shape[0]))
        for r0 in range(0, r, step):
            A, B = dd[r0:r0 + step] @ six, d[r0:r0 + step] @ bvec
            w2 = (k2 - c2 + B * B / A) / A
            i, j = torch.nonzero((w2 >= 0) & active, as_tuple=True)
            ts, w = -B[i, j] / A[i, j], w2[i, j].sqrt()
            keep = (ts + w >= tn) & (ts - w <= tf)
            pr.append(i[keep] + r0); pg.append(j[keep])
            pin.append((ts - w)[keep]); pout.append((ts + w)[keep])
            del A, B, w2
        pr, pg, pin, pout = (torch.cat(v) for v in (pr, pg, pin, pout))
        big = torch.full((r,), math.inf, device=dev, dtype=torch.float64)

        def closest(lo, ask):
            m = ask[pr] & (pout >= lo[pr])
            return big.clone().scatter_reduce_(0, pr[m], torch.maximum(pin[m], lo[pr[m]]), "amin")

    Y = _sh_basis64(int(case["deg"]), d)
    ks = torch.arange(n_s, device=dev, dtype=torch.float64)
    adaptive, dt0 = bool(case["adaptive"]), _f32(case["dt"])
    T = torch.ones(r, device=dev, dtype=torch.float64)
    C = torch.zeros(r, 3, device=dev, dtype=torch.float64)
    a = torch.full((r,), tn, device=dev, dtype=torch.float64)
    alive = torch.ones(r, device=dev, dtype=torch.bool)
    ask, lo = alive.clone(), a.clone()
    while True:
        with torch.no_grad():
            best = closest(lo, ask)
            alive = alive & ~(ask & torch.isinf(best))
            at = best
            if not adaptive:
                seg = dt0 * n_s
                at = tn + torch.maximum(((a - tn) / seg).round(), ((best - tn) / seg).floor()) * seg
            a = torch.where(ask & alive, at, a)
            alive = alive & (a < tf) & (T > _f32(T_EPS))
            if not bool(alive.any()):
                return C, T
            dt = torch.full_like(a, dt0)
            if adaptive:
                dt = (torch.clamp(a / ADAPTIVE["beta"], min=dt_min) *
                      T.clamp(min=1e-300) ** (-1.0 / 3.0)).clamp(max=dt_max)
            b = a + n_s * dt
            m = torch.nonzero(alive[pr] & (pin <= b[pr]) & (pout >= a[pr]))[:, 0]
            ri, gi = pr[m], pg[m]
            t = a[:, None] + (ks + 0.5) * dt[:, None]
        if m.numel():
            xs = (o - p["means"][gi])[:, None, :] + t[ri][:, :, None] * d[ri][:, None, :]
            q = (xs @ M[gi].transpose(1, 2)).square().sum(2)
            w = sig[gi][:, None] * torch.exp(-0.5 * q) * ((q <= k2[gi][:, None]) & (t[ri] < tf))
            col = (p["sh"][gi] * Y[ri][:, :, None]).sum(1)
            if "sg" in p:
                L = p["sg"][gi]
                ax = L[:, :, 3:6] / L[:, :, 3:6].norm(dim=2, keepdim=True)
                lobe = torch.exp(L[:, :, 6] * ((ax * d[ri][:, None, :]).sum(2) - 1.0))
                col = col + (L[:, :, :3] * lobe[:, :, None]).sum(1)
            sk = torch.zeros(r, n_s, device=dev, dtype=torch.float64).index_add(0, ri, w)
            W = torch.zeros(r, n_s, 3, device=dev, dtype=torch.float64).index_add(
                0, ri, w[:, :, None] * col[:, None, :])
            for k in range(n_s):
                s = sk[:, k]
                e = torch.exp(-s * dt)
                on = s > 0
                phi = torch.where(on, -torch.expm1(-s * dt) / torch.where(on, s, 1.0), dt)
                C = C + torch.where(on, T * phi, 0.0)[:, None] * W[:, k]
                T = T * e
        with torch.no_grad():
            hit = torch.zeros(r, device=dev, dtype=torch.bool)
            hit[ri] = True
            ask, lo = alive & ~hit, b
            a = torch.where(alive, b, a)


def exact(case, seed):
    n, rays, path = int(case["n"]), _rays(case), case["path"]
    params, other, cams = _inputs(case, seed)
    p = {k: v.double() for k, v in params.items()}
    if path == "optimizer":
        return _optimizer64(p, {k: v.double() for k, v in other.items()})
    grad = path in ("train", "captured", "densify")
    # what plain torch does within seconds
    if n * float(rays) > (2e10 if grad else 8e10) or \
            RAY_SHARE[case["scene"]] * n * rays > (2e7 if grad else 5e7):
        return None
    if grad:
        for v in p.values():
            v.requires_grad_(True)
            v.grad = torch.zeros_like(v)
    dev = other.device
    size = 16384 if not grad else 4096
    rgbs, Ts, at = [], [], 0
    stat = torch.zeros(n, device=dev, dtype=torch.float64)
    before = torch.zeros(n, 3, device=dev, dtype=torch.float64)
    loss = 0.0
    for cam in cams:
        o, d = _rays64(cam, dev)
        for r0 in range(0, d.shape[0], size):
            with torch.set_grad_enabled(grad):
                rgb, T = _march64(case, p, cam, o, d[r0:r0 + size])
                if grad:
                    err = rgb - other[at:at + rgb.shape[0]].double()
                    part = (err * err).sum() / (3.0 * rays)
                    if part.requires_grad:             # else no ray of the chunk met anything
                        part.backward()
                    loss += float(part.detach())
            rgbs.append(rgb.detach()); Ts.append(T.detach())
            at += rgb.shape[0]
        if path == "densify":
            g = p["means"].grad - before
            before = p["means"].grad.clone()
            stat += (p["means"].detach() - o).norm(dim=1) / cam.fx * g.norm(dim=1)
    out = {"rgb": torch.cat(rgbs), "T": torch.cat(Ts)}
    if not grad:
        return out
    # (a captured step's gradients are those of the five common tensors)
    out["grads"] = {k: v.grad for k, v in p.items() if path != "captured" or k in KEYS}
    if path == "densify":
        return dict(out, densify=stat, views=None)
    return dict(out, loss=torch.tensor(loss, dtype=torch.float64))


def _optimizer64(p, g):
    ls = p["log_scales"].clone().requires_grad_(True)
    ratio = 2.0 / (math.pi * math.sqrt(3.0)) * torch.exp(2 * ls).sum(1) ** 1.5 / torch.exp(ls.sum(1))
    loss = (torch.clamp(ratio, min=10.0) - 10.0).mean()
    loss.backward()
    lr = dict(means=1.6e-4, log_scales=5e-3, quats=1e-3, density=5e-2, sh=2.5e-3)
    b1, b2 = _f32(0.9), _f32(0.999)
    m = {k: (1 - b1) * g[k] for k in KEYS}
    v = {k: (1 - b2) * g[k] ** 2 for k in KEYS}
    new = {k: p[k] - _f32(lr[k]) * (m[k] / (1 - b1)) / ((v[k] / (1 - b2)).sqrt() + 1e-15)
           for k in KEYS}
    return {"loss": loss.detach(), "grad": ls.grad, "params": new, "m": m, "v": v}
