"""The work that the framework is timed on: a mapping loop's calls through the
public entry points, over the range of sizes that its users run.

A case is a dict of plain values.  `op` names the path:

  render    render_forward, and with back = "full" or "pose" render_backward
            (all gradients with the pose's, or the pose gradient alone)
  loss      mapping_loss, value and gradients
  merge     voxel_merge (closed form or L-BFGS solver)
  patches   patch_grid_sample
  adam      adam_step

`listed` gives the fixed cases, `draw` others of the same ranges, `prepare`
what a program holds before the call, `run` one pass, `work` the bytes and
operations a pass cannot do without, and `exact` the outputs in 64 bits from
plain torch, where that takes seconds.
"""
import math
import random

import torch

from paper_2509_13536_amd import (AdamState, GaussianMap, View, Workspace, adam_step, mapping_loss,
                                  patch_grid_sample, render_backward, render_forward, voxel_merge)

DEV = "cuda"
GROUPS = ("means", "scales", "quats", "opac", "sh")
ADAM_LR = {"means": 1.6e-4, "scales": 5e-3, "quats": 1e-3, "opac": 5e-2, "sh": 2.5e-3}
LAMBDA_SSIM = 0.2


# ---------------------------------------------------------------- the cases
def _render(name, scene, n, w, h, f, views=1, back="none", sh=0, mixed=False):
    return {"name": name, "op": "render", "scene": scene, "n": n, "w": w, "h": h, "f": float(f), "views": views,
            "back": back, "sh": sh, "mixed": mixed}


def listed():
    return [
        # the smallest call: a preview of a small map, where launches and the read-back count
        _render("preview_10k", "box", 10_000, 320, 240, 300.0),
        # one batch of a render server: one resident map, requests at three resolutions
        _render("serve_mixed_300k", "room", 300_000, 1200, 680, 600.0, views=3, mixed=True),
        # a tracking iteration on a map of the size a SLAM run holds, at an odd resolution
        _render("track_100k", "room", 100_000, 611, 457, 517.0, back="pose"),
        # a mapping iteration on one keyframe
        _render("keyframe_200k", "surface", 200_000, 640, 480, 525.0, back="full"),
        # a mapping iteration over a window of keyframes
        _render("window_500k", "room", 500_000, 1200, 680, 600.0, views=8, back="full"),
        # one view of the largest map, with view-dependent colour
        _render("large_3M_sh3", "room", 3_000_000, 1200, 680, 600.0, back="full", sh=3),
        # the loss of one monocular frame, at an odd resolution
        {"name": "loss_frame", "op": "loss", "w": 641, "h": 479, "views": 1, "depth": False, "n": 0},
        # the loss of the window: colour, depth and the scales' isotropy
        {"name": "loss_window", "op": "loss", "w": 1200, "h": 680, "views": 8, "depth": True, "n": 500_000},
        # the merge that follows a window, over the whole map
        {"name": "merge_500k", "op": "merge", "n": 500_000, "voxel": 0.05, "solver": "closed", "masked": False},
        # the merge of a local map under the eligibility mask, by the iterative solver
        {"name": "merge_lbfgs_100k", "op": "merge", "n": 100_000, "voxel": 0.05, "solver": "lbfgs", "masked": True},
        # new Gaussians of a monocular keyframe
        {"name": "patches_1200x680", "op": "patches", "w": 1200, "h": 680, "f": 600.0, "kp": 2000, "rgbd": False},
        # the optimiser step that ends a mapping iteration
        {"name": "adam_500k", "op": "adam", "n": 500_000, "sh": 0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["render", "render", "render", "loss", "loss", "merge", "merge", "patches", "adam"])
    if op == "render":
        scene = rng.choice(["box", "surface", "room", "room"])
        w = _log(rng, 160, 1200)
        h = max(120, int(w * rng.uniform(0.55, 0.8)))
        views = rng.choice([1, 1, 2, 3, 5, 8])
        # at most the window's Gaussians and pixels in all; the box and the surface are seen whole by every view
        n = min(_log(rng, 5_000, 500_000), 500_000 if scene == "room" else 400_000 // views)
        while views > 1 and views * w * h > 6_500_000:
            views -= 1
        return {"op": op, "scene": scene, "n": n, "w": w, "h": h, "f": round(w * rng.uniform(0.5, 0.95), 1),
                "views": views, "back": rng.choice(["none", "pose", "full", "full"]),
                "sh": rng.choice([0, 0, 1, 2, 3]), "mixed": views > 1 and rng.random() < 0.3}
    if op == "loss":
        w = _log(rng, 96, 1200)
        depth = rng.random() < 0.5
        return {"op": op, "w": w, "h": max(64, int(w * rng.uniform(0.55, 0.8))), "views": rng.choice([1, 1, 2, 3, 8]),
                "depth": depth, "n": _log(rng, 5_000, 500_000) if depth else 0}
    if op == "merge":
        solver = rng.choice(["closed", "closed", "lbfgs"])
        return {"op": op, "n": _log(rng, 5_000, 500_000 if solver == "closed" else 100_000),
                "voxel": rng.choice([0.03, 0.05, 0.05, 0.08]), "solver": solver, "masked": rng.random() < 0.5}
    if op == "patches":
        w = _log(rng, 320, 1200)
        return {"op": op, "w": w, "h": int(w * rng.uniform(0.55, 0.8)), "f": round(w * rng.uniform(0.5, 0.95), 1),
                "kp": _log(rng, 200, 6000), "rgbd": rng.random() < 0.5}
    return {"op": op, "n": _log(rng, 5_000, 500_000), "sh": rng.choice([0, 0, 1, 3])}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2 + 1)
    return g


def _u(g, *shape, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device=DEV)


def _n(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _attributes(g, n, sh):
    """Scales of about 3 cm, any rotation, opacities in (0.05, 0.95), colours in [0, 1] with small higher orders."""
    k = (sh + 1) ** 2
    coef = 0.2 * _n(g, n, k, 3)
    coef[:, 0] = _u(g, n, 3, lo=-math.sqrt(math.pi), hi=math.sqrt(math.pi))
    quats = _n(g, n, 4)
    return [torch.exp(-3.5 + 0.5 * _n(g, n, 3)), quats / quats.norm(dim=1, keepdim=True),
            _u(g, n, lo=0.05, hi=0.95), coef]


def _look_at(pos, target):
    """World to camera (rows right, down, forward), z up in the world."""
    f = torch.tensor(target, dtype=torch.float64) - torch.tensor(pos, dtype=torch.float64)
    f = f / f.norm()
    r = torch.linalg.cross(f, torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64))
    r = r / r.norm()
    R = torch.stack([r, torch.linalg.cross(f, r), f])
    return torch.cat([R, -(R @ torch.tensor(pos, dtype=torch.float64))[:, None]], dim=1)


def _room(g, rnd, n, sh, dup=0.3):
    """Gaussians on the walls and on fifty boxes of an 8 x 6 x 3 m room; the last `dup` of them near-duplicates."""
    X, Y, Z = 8.0, 6.0, 3.0
    faces = [((0, 0, 0), (X, 0, 0), (0, Y, 0)), ((0, 0, Z), (X, 0, 0), (0, Y, 0)), ((0, 0, 0), (0, Y, 0), (0, 0, Z)),
             ((X, 0, 0), (0, Y, 0), (0, 0, Z)), ((0, 0, 0), (X, 0, 0), (0, 0, Z)), ((0, Y, 0), (X, 0, 0), (0, 0, Z))]
    for _ in range(50):
        sx, sy, sz = (rnd.uniform(0.2, 1.0) for _ in range(3))
        cx, cy, yaw = rnd.uniform(0.6, X - 0.6), rnd.uniform(0.6, Y - 0.6), rnd.uniform(0, 2 * math.pi)
        ex, ey, ez = (sx * math.cos(yaw), sx * math.sin(yaw), 0.0), (-sy * math.sin(yaw), sy * math.cos(yaw), 0.0), (0, 0, sz)
        o = (cx - 0.5 * (ex[0] + ey[0]), cy - 0.5 * (ex[1] + ey[1]), 0.0)
        faces += [((o[0], o[1], sz), ex, ey), (o, ex, ez), (o, ey, ez),
                  ((o[0] + ey[0], o[1] + ey[1], 0.0), ex, ez), ((o[0] + ex[0], o[1] + ex[1], 0.0), ey, ez)]
    F = torch.tensor(faces, dtype=torch.float32, device=DEV)  # [faces, 3, 3]: origin and two edges
    area = torch.linalg.cross(F[:, 1], F[:, 2]).norm(dim=1)
    n_dup = int(n * dup)
    m = n - n_dup
    edges = torch.cumsum(area, 0) / area.sum()
    face = F[torch.searchsorted(edges, _u(g, m)).clamp(max=len(faces) - 1)]
    means = face[:, 0] + _u(g, m, 1) * face[:, 1] + _u(g, m, 1) * face[:, 2]
    parts = [means, *_attributes(g, m, sh)]
    src = torch.randint(0, m, (n_dup,), generator=g, device=DEV)
    more = [p[src] for p in parts]
    more[0] = more[0] + _u(g, n_dup, 3, lo=-0.005, hi=0.005)
    more[1] = more[1] * _u(g, n_dup, 3, lo=0.95, hi=1.05)
    return [torch.cat(p) for p in zip(parts, more)]


def _depth_surface(rnd):
    z0, gx, gy = rnd.uniform(1.5, 2.5), rnd.uniform(-1.5e-3, 1.5e-3), rnd.uniform(-1.5e-3, 1.5e-3)
    waves = []
    for _ in range(3):
        a, k = rnd.uniform(0, 2 * math.pi), 2 * math.pi * rnd.uniform(1 / 400, 1 / 80)
        waves.append((rnd.uniform(0.05, 0.3), k * math.cos(a), k * math.sin(a), rnd.uniform(0, 2 * math.pi)))

    def z(u, v):
        out = z0 + gx * u + gy * v
        for amp, ku, kv, ph in waves:
            out = out + amp * torch.sin(ku * u + kv * v + ph)
        return out.clamp(0.5, 4.0)
    return z


def _trajectory(rnd, case, count):
    """Keyframes on an ellipse through the room, looking along the path."""
    th0, out = rnd.uniform(0, 2 * math.pi), []
    for k in range(count):
        th = th0 + 0.3 * k
        pos = (4.0 + 2.5 * math.cos(th), 3.0 + 1.5 * math.sin(th), 1.5 + 0.2 * math.sin(2 * th))
        psi = math.atan2(1.5 * math.cos(th), -2.5 * math.sin(th)) + rnd.uniform(-0.3, 0.3)
        out.append(_look_at(pos, (pos[0] + math.cos(psi), pos[1] + math.sin(psi), pos[2] - 0.15)))
    return out


def _nearby(rnd, count):
    """Poses within a few centimetres and degrees of the identity."""
    out = []
    for k in range(count):
        a = [0.0 if k == 0 else rnd.uniform(-0.05, 0.05) for _ in range(6)]
        W = torch.tensor([[0, -a[5], a[4]], [a[5], 0, -a[3]], [-a[4], a[3], 0]], dtype=torch.float64)
        out.append(torch.cat([torch.linalg.matrix_exp(W), torch.tensor(a[:3], dtype=torch.float64)[:, None]], dim=1))
    return out


def _scene(case, seed):
    """The map's arrays and the views of a render case."""
    g, rnd = _gen(seed), random.Random(int(seed))
    n, w, h, f = case["n"], case["w"], case["h"], case["f"]
    if case["scene"] == "room":
        parts = _room(g, rnd, n, case["sh"], 0.0 if n > 1_000_000 else 0.3)
        poses = _trajectory(rnd, case, case["views"])
    else:
        if case["scene"] == "box":
            means = torch.stack([_u(g, n, lo=-1, hi=1), _u(g, n, lo=-1, hi=1), _u(g, n, lo=1, hi=3)], dim=1)
        else:
            u, v = _u(g, n, hi=w), _u(g, n, hi=h)
            z = _depth_surface(rnd)(u, v)
            means = torch.stack([(u - w / 2) * z / f, (v - h / 2) * z / f, z], dim=1) + _u(g, n, 3, lo=-0.02, hi=0.02)
        parts = [means, *_attributes(g, n, case["sh"])]
        poses = _nearby(rnd, case["views"])
    views = []
    for k, T in enumerate(poses):
        d = (1, 2, 4)[k % 3] if case["mixed"] else 1
        views.append(View(max(1, w // d), max(1, h // d), f / d, f / d, w / d / 2, h / d / 2,
                          T.to(torch.float32).numpy()))
    return [p.to(torch.float32).contiguous() for p in parts], views, g


def _loss_inputs(case, seed):
    g = _gen(seed)
    P = case["views"] * case["w"] * case["h"]
    gt = _u(g, 3 * P)
    rgb = (gt + 0.05 * _n(g, 3 * P)).clamp(min=0.0)
    depth = gtd = scales = None
    if case["depth"]:
        gtd = _u(g, P, lo=0.5, hi=4.0)
        depth = gtd + 0.01 * _n(g, P)
        gtd = torch.where(_u(g, P) < 0.2, torch.zeros_like(gtd), gtd)
    if case["n"]:
        scales = torch.exp(-3.5 + 0.5 * _n(g, case["n"], 3))
    return rgb, gt, depth, gtd, scales


def _patch_inputs(case, seed):
    """Keypoints crowded into a quarter of the 32-pixel patches, a tenth of them
    scattered one to a patch elsewhere; three in ten have a depth."""
    g, rnd = _gen(seed), random.Random(int(seed))
    w, h, n = case["w"], case["h"], case["kp"]
    z = _depth_surface(rnd)
    nx = math.ceil(w / 32)
    cells = torch.randperm(nx * math.ceil(h / 32), generator=g, device=DEV)
    dense = min(len(cells) // 4, n // 8)
    alone = min(n // 10, len(cells) - dense)
    crowd = torch.cat([torch.arange(dense, device=DEV).repeat(4),
                       torch.randint(0, dense, (n - alone - 4 * dense,), generator=g, device=DEV)])
    cell = cells[torch.cat([crowd, torch.arange(dense, dense + alone, device=DEV)])]
    cell = cell[torch.randperm(n, generator=g, device=DEV)]
    low = 32.0 * torch.stack([cell % nx, cell // nx], dim=1)
    size = torch.minimum(torch.tensor([w, h], device=DEV) - low, torch.tensor(32.0, device=DEV))
    kp = low - 0.49 + (size - 0.02) * _u(g, n, 2)
    kd = torch.where(_u(g, n) < 0.3, z(kp[:, 0], kp[:, 1]) + 0.01 * _n(g, n), torch.zeros(n, device=DEV))
    depth = None
    if case["rgbd"]:
        v, u = torch.meshgrid(torch.arange(h, device=DEV).float(), torch.arange(w, device=DEV).float(), indexing="ij")
        depth = torch.where(_u(g, h, w) < 0.05, torch.zeros(h, w, device=DEV), z(u, v)).contiguous()
    view = View(w, h, case["f"], case["f"], w / 2, h / 2, _trajectory(rnd, case, 1)[0].to(torch.float32).numpy())
    return view, kp.contiguous(), kd.contiguous(), _u(g, 3, h, w), depth


def _adam_inputs(case, seed):
    g = _gen(seed)
    n, k = case["n"], (case["sh"] + 1) ** 2
    p = [_u(g, n, 3, hi=8.0), *_attributes(g, n, case["sh"])]
    grads = [1e-4 * _n(g, *t.shape) for t in p]
    m = [1e-4 * _n(g, *t.shape) for t in p]
    v = [1e-8 * (0.1 + _n(g, *t.shape).square()) for t in p]
    return p, grads, m, v


def prepare(case, seed):
    s = {"case": case}
    if case["op"] == "render":
        parts, s["views"], g = _scene(case, seed)
        s["map"], s["ws"] = GaussianMap(*parts, case["sh"]), Workspace(DEV)
        if case["back"] != "none":
            P = sum(v.W * v.H for v in s["views"])
            s["g_rgb"], s["g_depth"] = _n(g, 3 * P) / P, _n(g, P) / P
    elif case["op"] == "loss":
        s["in"], s["sizes"], s["ws"] = _loss_inputs(case, seed), [(case["w"], case["h"])] * case["views"], Workspace(DEV)
    elif case["op"] == "merge":
        g = _gen(seed)
        s["map"], s["ws"] = GaussianMap(*_room(g, random.Random(int(seed)), case["n"], 0), 0), Workspace(DEV)
        s["mask"] = (_u(g, case["n"]) < 0.9).to(torch.uint8) if case["masked"] else None
        s["out"] = GaussianMap(*(torch.zeros_like(getattr(s["map"], k)) for k in GROUPS), 0)
    elif case["op"] == "patches":
        s["in"], s["ws"] = _patch_inputs(case, seed), Workspace(DEV)
    else:
        p, grads, m, v = _adam_inputs(case, seed)
        s["map"], s["grads"] = GaussianMap(*p, case["sh"]), dict(zip(GROUPS, grads))
        s["state"] = AdamState(GaussianMap(*m, case["sh"]), GaussianMap(*v, case["sh"]), 10)
    return s


# ---------------------------------------------------------------- one pass
def _arrays(m):
    return [getattr(m, k) for k in GROUPS]


def run(s):
    case = s["case"]
    if case["op"] == "render":
        back = case["back"]
        st = render_forward([s["map"]], s["views"], need_backward=back != "none", ws=s["ws"])
        out = {"rgb": st.rgb, "depth": st.depth, "T": st.T}
        if back == "full":
            grads, out["pose"] = render_backward(st, s["g_rgb"], s["g_depth"])
            out["grads"] = [grads[0][k] for k in GROUPS]
        elif back == "pose":
            _, out["pose"] = render_backward(st, s["g_rgb"], s["g_depth"], want=())
        return out
    if case["op"] == "loss":
        rgb, gt, depth, gtd, scales = s["in"]
        r = mapping_loss(s["sizes"], rgb, gt, depth, gtd, scales, lambda_ssim=LAMBDA_SSIM, w_depth=1.0, w_iso=1.0,
                         ws=s["ws"])
        return {"loss": r.loss, "d_rgb": r.d_rgb, "d_depth": r.d_depth, "d_scales": r.d_scales}
    if case["op"] == "merge":
        r = voxel_merge(s["map"], s["mask"], voxel_size=case["voxel"], solver=case["solver"], ws=s["ws"],
                        out=s["out"])
        return {"map": _arrays(s["out"]), "n": r.n_out, "old_to_new": r.old_to_new}
    if case["op"] == "patches":
        view, kp, kd, image, depth = s["in"]
        r = patch_grid_sample(view, kp, kd, image, depth, ws=s["ws"])
        return {"map": _arrays(r.map), "n": r.n_out, "source": r.source}
    st = adam_step(s["map"], s["grads"], s["state"], ADAM_LR)
    return {"params": _arrays(s["map"]), "m": _arrays(st.exp_avg), "v": _arrays(st.exp_avg_sq)}


# ---------------------------------------------------------------- the least work of a pass
def work(case):
    op = case["op"]
    if op == "render":
        per = 4 * (11 + 3 * (case["sh"] + 1) ** 2)  # bytes of a Gaussian
        d = [(1, 2, 4)[k % 3] if case["mixed"] else 1 for k in range(case["views"])]
        P = sum((case["w"] // x) * (case["h"] // x) for x in d)
        b, f = per * case["n"] + 20 * P, 60 * case["n"] * case["views"] + 64 * 30 * P  # about 64 blended Gaussians a pixel
        if case["back"] != "none":
            b, f = b + per * case["n"] + 20 * P, f + 64 * 70 * P
        if case["back"] == "full":
            b += per * case["n"]
        return {"bytes": b, "flops": f}
    if op == "loss":
        P = case["views"] * case["w"] * case["h"]
        # per channel and pixel: four moments and three derivative maps through a separable 11-tap window, and the formula
        return {"bytes": P * (36 + (12 if case["depth"] else 0)) + 24 * case["n"], "flops": 3 * P * (7 * 2 * 2 * 11 + 60)}
    if op == "merge":  # the map in, about as much out, the index; a merge of every second Gaussian
        return {"bytes": case["n"] * (56 + 40 + 4), "flops": case["n"] * (700 if case["solver"] == "closed" else 30_000)}
    if op == "patches":
        cells = math.ceil(case["w"] / 32) * math.ceil(case["h"] / 32) * 4
        out = case["kp"] + cells
        return {"bytes": 12 * case["kp"] + out * (12 + 56 + 4 + (4 if case["rgbd"] else 0)),
                "flops": out * (30 + (0 if case["rgbd"] else 5 * 0.3 * case["kp"]))}
    return {"bytes": 28 * case["n"] * (11 + 3 * (case["sh"] + 1) ** 2),
            "flops": 14 * case["n"] * (11 + 3 * (case["sh"] + 1) ** 2)}


# ---------------------------------------------------------------- the same in 64 bits
def _sh_basis(deg, d):
    x, y, z = d.unbind(1)
    B = [torch.full_like(x, 0.28209479177387814)]
    if deg > 0:
        c = 0.4886025119029199
        B += [-c * y, c * z, -c * x]
    if deg > 1:
        a, xx, yy, zz = 1.0925484305920792, x * x, y * y, z * z
        B += [a * x * y, -a * y * z, 0.31539156525252005 * (2 * zz - xx - yy), -a * x * z, 0.5462742152960396 * (xx - yy)]
    if deg > 2:
        B += [-0.5900435899266435 * y * (3 * xx - yy), 2.890611442640554 * x * y * z,
              -0.4570457994644658 * y * (4 * zz - xx - yy), 0.3731763325901154 * z * (2 * zz - 3 * xx - 3 * yy),
              -0.4570457994644658 * x * (4 * zz - xx - yy), 1.445305721320277 * z * (xx - yy),
              -0.5900435899266435 * x * (xx - 3 * yy)]
    return torch.stack(B, dim=1)


def _project(parts, view, deg, xi):
    """Per Gaussian: u, v, conic, opacity, colour, depth (differentiable), and its tile rectangle."""
    m, sc, q, o, sh = parts
    T = torch.as_tensor(view.Tcw, dtype=torch.float64, device=DEV)
    Z = torch.zeros((), dtype=torch.float64, device=DEV)
    W = torch.eye(3, dtype=torch.float64, device=DEV) + torch.stack(
        [torch.stack([Z, -xi[5], xi[4]]), torch.stack([xi[5], Z, -xi[3]]), torch.stack([-xi[4], xi[3], Z])])
    R, t = W @ T[:, :3], W @ T[:, 3] + xi[:3]
    p = m @ R.T + t
    z = p[:, 2]
    qn = q / q.norm(dim=1, keepdim=True)
    a, b, c, d = qn.unbind(1)
    Rq = torch.stack([1 - 2 * (c * c + d * d), 2 * (b * c - a * d), 2 * (b * d + a * c),
                      2 * (b * c + a * d), 1 - 2 * (b * b + d * d), 2 * (c * d - a * b),
                      2 * (b * d - a * c), 2 * (c * d + a * b), 1 - 2 * (b * b + c * c)], dim=1).view(-1, 3, 3)
    M = R @ Rq * sc[:, None, :]
    lx, ly = 1.3 * (0.5 * view.W / view.fx), 1.3 * (0.5 * view.H / view.fy)
    xn, yn = p[:, 0] / z, p[:, 1] / z
    O = torch.zeros_like(z)
    J = torch.stack([view.fx / z, O, -view.fx * xn.clamp(-lx, lx) / z, O, view.fy / z, -view.fy * yn.clamp(-ly, ly) / z],
                    dim=1).view(-1, 2, 3)
    JM = J @ M
    S = JM @ JM.transpose(1, 2)
    A, B, C = S[:, 0, 0] + 0.3, S[:, 0, 1], S[:, 1, 1] + 0.3
    det = A * C - B * B
    u, v = view.fx * xn + view.cx, view.fy * yn + view.cy
    dirs = m + R.T @ t
    col = (_sh_basis(deg, dirs / dirs.norm(dim=1, keepdim=True))[:, :, None] * sh).sum(1) + 0.5
    out = torch.cat([torch.stack([u, v, C / det, -B / det, A / det, o], dim=1), col.clamp(min=0), z[:, None]], dim=1)
    with torch.no_grad():
        mid = 0.5 * (A + C)
        r = torch.ceil(3 * torch.sqrt(mid + torch.sqrt((mid * mid - det).clamp(min=0.1))))
        tx, ty = math.ceil(view.W / 16), math.ceil(view.H / 16)
        rect = torch.stack([torch.floor((u - r) / 16).clamp(0, tx), torch.floor((v - r) / 16).clamp(0, ty),
                            (torch.floor((u + r) / 16) + 1).clamp(0, tx), (torch.floor((v + r) / 16) + 1).clamp(0, ty)], dim=1)
        rect[~((z > view.near) & (det > 0))] = 0
    return out, torch.nan_to_num(rect).long()


def _exact_view(parts, view, deg, xi, g_rgb, g_depth):
    """Images of one view; its gradients go to the leaves of parts and to xi."""
    G, rect = _project(parts, view, deg, xi)
    tx = math.ceil(view.W / 16)
    with torch.no_grad():
        order = torch.argsort(G[:, 9], stable=True)
        rc = rect[order]
        nx, ny = (rc[:, 2] - rc[:, 0]).clamp(min=0), (rc[:, 3] - rc[:, 1]).clamp(min=0)
        cnt = nx * ny
        who = torch.repeat_interleave(torch.arange(len(cnt), device=DEV), cnt)
        k = torch.arange(len(who), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[who]
        tile = (rc[who, 1] + k // nx[who]) * tx + rc[who, 0] + k % nx[who]
        tile, at = torch.sort(tile, stable=True)
        lists = order[who[at]]
        first = torch.searchsorted(tile, torch.arange(tx * math.ceil(view.H / 16) + 1, device=DEV)).tolist()
    rgb = torch.zeros(3, view.H, view.W, dtype=torch.float64, device=DEV)
    dep, Tr = torch.zeros_like(rgb[0]), torch.ones_like(rgb[0])
    dG, Gd = torch.zeros_like(G), G.detach()
    for t in range(len(first) - 1):
        sel = lists[first[t]:first[t + 1]]
        if not len(sel):
            continue
        y0, x0 = t // tx * 16, t % tx * 16
        y1, x1 = min(y0 + 16, view.H), min(x0 + 16, view.W)
        yy, xx = torch.meshgrid(torch.arange(y0, y1, device=DEV).double(), torch.arange(x0, x1, device=DEV).double(), indexing="ij")
        with torch.enable_grad():
            e = Gd[sel].requires_grad_(g_rgb is not None)
            c = [e[:, i:i + 1] for i in range(6)]
            dx, dy = c[0] - xx.reshape(1, -1), c[1] - yy.reshape(1, -1)
            al = (c[5] * torch.exp(-0.5 * (c[2] * dx * dx + c[4] * dy * dy) - c[3] * dx * dy)).clamp(max=0.99)
            lg = torch.log1p(-torch.where(al >= 1 / 255, al, torch.zeros_like(al)))
            keep = (al >= 1 / 255) & (torch.exp(torch.cumsum(lg, 0)) >= 1e-4)
            al = torch.where(keep, al, torch.zeros_like(al))
            lg = torch.log1p(-al)
            w = al * torch.exp(torch.cumsum(lg, 0) - lg)
            img = e[:, 6:10].T @ w
        rgb[:, y0:y1, x0:x1] = img[:3].detach().view(3, y1 - y0, x1 - x0)
        dep[y0:y1, x0:x1] = img[3].detach().view(y1 - y0, x1 - x0)
        Tr[y0:y1, x0:x1] = torch.exp(lg.detach().sum(0)).view(y1 - y0, x1 - x0)
        if g_rgb is not None:
            gr = torch.cat([g_rgb[:, y0:y1, x0:x1].reshape(3, -1), g_depth[y0:y1, x0:x1].reshape(1, -1)])
            dG.index_add_(0, sel, torch.autograd.grad((img * gr).sum(), e)[0])
    if g_rgb is not None:
        seen = rect[:, 0] < rect[:, 2]  # a culled Gaussian has no gradient
        torch.autograd.backward(G[seen], dG[seen])
    return rgb.view(-1), dep.view(-1), Tr.view(-1)


def _exact_render(case, seed):
    if case["views"] * case["w"] * case["h"] > 400_000 or case["n"] * case["views"] > 400_000:
        return None  # minutes of tile loops
    parts, views, g = _scene(case, seed)
    full = case["back"] == "full"
    parts = [p.double().requires_grad_(full) for p in parts]
    P = sum(v.W * v.H for v in views)
    gr = gd = None
    if case["back"] != "none":
        gr, gd = (_n(g, 3 * P) / P).double(), (_n(g, P) / P).double()
    xi = torch.zeros(len(views), 6, dtype=torch.float64, device=DEV, requires_grad=gr is not None)
    imgs, o = [], 0
    for k, v in enumerate(views):
        n = v.W * v.H
        imgs.append(_exact_view(parts, v, case["sh"], xi[k], None if gr is None else gr[3 * o:3 * (o + n)].view(3, v.H, v.W),
                                None if gd is None else gd[o:o + n].view(v.H, v.W)))
        o += n
    out = {k: torch.cat([im[i] for im in imgs]) for i, k in enumerate(("rgb", "depth", "T"))}
    if gr is not None:
        out["pose"] = xi.grad
    if full:
        out["grads"] = [p.grad for p in parts]
    return out


def _window(x):
    """The 11 x 11 Gaussian window (sigma 1.5) over [c, h, w], zeros outside."""
    k = torch.exp(-(torch.arange(11, dtype=torch.float64) - 5) ** 2 / (2 * 1.5 * 1.5))
    k = (k / k.sum()).tolist()
    for dim in (1, 2):
        pad = [5, 5, 0, 0] if dim == 2 else [0, 0, 5, 5]
        y = torch.nn.functional.pad(x, pad)
        x = sum(k[i] * y.narrow(dim, i, x.shape[dim]) for i in range(11))
    return x


def _exact_loss(case, seed):
    rgb, gt, depth, gtd, scales = _loss_inputs(case, seed)
    w, h = case["w"], case["h"]
    n, terms, total, d_rgb, d_depth = w * h, [], 0.0, [], []
    for v in range(case["views"]):
        x = rgb[3 * n * v:3 * n * (v + 1)].double().view(3, h, w).requires_grad_(True)
        y = gt[3 * n * v:3 * n * (v + 1)].double().view(3, h, w)
        mx, my = _window(x), _window(y)
        vx, vy, cov = _window(x * x) - mx * mx, _window(y * y) - my * my, _window(x * y) - mx * my
        c1, c2 = 1e-4, 9e-4
        ssim = ((2 * mx * my + c1) * (2 * cov + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2))).mean()
        l1 = (x - y).abs().mean()
        lv, ld, leaves = (1 - LAMBDA_SSIM) * l1 + LAMBDA_SSIM * (1 - ssim), torch.zeros_like(l1), [x]
        if depth is not None:
            d, t = depth[n * v:n * (v + 1)].double().requires_grad_(True), gtd[n * v:n * (v + 1)].double()
            ld = torch.where(t > 0, (d - t).abs(), torch.zeros_like(t)).mean()
            lv, leaves = lv + ld, [x, d]
        grads = torch.autograd.grad(lv, leaves)
        d_rgb.append(grads[0].reshape(-1))
        d_depth += [grads[1]] if depth is not None else []
        terms += [float(l1), float(ssim), float(ld), float(lv)]
        total += float(lv)
    iso, d_scales = 0.0, None
    if scales is not None:
        s = scales.double().requires_grad_(True)
        li = (s - s.mean(1, keepdim=True)).abs().mean()
        d_scales, iso = torch.autograd.grad(li, s)[0], float(li)
    return {"loss": torch.tensor(terms + [iso, total + iso], dtype=torch.float64), "d_rgb": torch.cat(d_rgb),
            "d_depth": torch.cat(d_depth) if d_depth else None, "d_scales": d_scales}


def _exact_patches(case, seed):
    view, kp, kd, image, dmap = _patch_inputs(case, seed)
    w, h, P, s = case["w"], case["h"], 32, 2
    px = torch.floor(kp + 0.5).long()
    on = (px[:, 0] >= 0) & (px[:, 0] < w) & (px[:, 1] >= 0) & (px[:, 1] < h)
    nx, ny = math.ceil(w / P), math.ceil(h / P)
    count = torch.bincount((px[on, 1] // P) * nx + px[on, 0] // P, minlength=nx * ny)
    patch = torch.arange(nx * ny, device=DEV).repeat_interleave(s * s)
    lat = torch.arange(s * s, device=DEV).repeat(nx * ny)
    x0, y0 = P * (patch % nx), P * (patch // nx)
    sx = x0 + ((2 * (lat % s) + 1) * (w - x0).clamp(max=P)) // (2 * s)
    sy = y0 + ((2 * (lat // s) + 1) * (h - y0).clamp(max=P)) // (2 * s)
    xy = torch.cat([kp.double(), torch.stack([sx, sy], dim=1).double()])
    pix = torch.cat([px, torch.stack([sx, sy], dim=1)])
    keep = torch.cat([on, (count < 4)[patch]])
    own = kd > 0
    z = torch.cat([torch.where(own, kd, torch.zeros_like(kd)).double(), torch.zeros(len(lat), dtype=torch.float64, device=DEV)])
    pix = torch.where(keep[:, None], pix, torch.zeros_like(pix))
    if dmap is not None:
        z = torch.where(z > 0, z, dmap[pix[:, 1], pix[:, 0]].double().clamp(min=0))
    near = torch.cdist(xy, kp[own].double(), compute_mode="donot_use_mm_for_euclid_dist").argmin(1)
    z = torch.where(z > 0, z, kd[own].double()[near])
    at = torch.nonzero(keep)[:, 0]
    xy, pix, z = xy[at], pix[at], z[at]
    T = torch.as_tensor(view.Tcw, dtype=torch.float64, device=DEV)
    pc = torch.stack([z * (xy[:, 0] - view.cx) / view.fx, z * (xy[:, 1] - view.cy) / view.fy, z], dim=1)
    quat = torch.zeros(len(at), 4, dtype=torch.float64, device=DEV)
    quat[:, 0] = 1
    sh = (image[:, pix[:, 1], pix[:, 0]].T.double() - 0.5) / 0.28209479177387814
    return {"map": [(pc - T[:, 3]) @ T[:, :3], (0.5 * P / s / view.fx * z)[:, None].expand(-1, 3), quat,
                    torch.full((len(at),), 0.5, dtype=torch.float64, device=DEV), sh[:, None]],
            "n": len(at), "source": at.to(torch.int32)}


def _exact_adam(case, seed):
    p, grads, m, v = ([t.double() for t in x] for x in _adam_inputs(case, seed))
    f32 = lambda x: float(torch.tensor(x, dtype=torch.float32))  # noqa: E731
    b1, b2, step = f32(0.9), f32(0.999), 11
    m = [b1 * a + (1 - b1) * g for a, g in zip(m, grads)]
    v = [b2 * a + (1 - b2) * g * g for a, g in zip(v, grads)]
    new = [t - f32(ADAM_LR[k]) * (a / (1 - b1 ** step)) / (torch.sqrt(b / (1 - b2 ** step)) + 1e-15)
           for k, t, a, b in zip(GROUPS, p, m, v)]
    return {"params": new, "m": m, "v": v}


def exact(case, seed):
    """None for the merges: a voxel's members merge one after another, minutes in plain numpy."""
    if case["op"] == "merge":
        return None
    return {"render": _exact_render, "loss": _exact_loss, "patches": _exact_patches, "adam": _exact_adam}[case["op"]](case, seed)
