"""Workloads of the renderer as a user's program runs them, each through the package's public entry points.

A case names its path (what the program does), the number of Gaussians, the image, and the options in use:

  forward   a viewer: ``WSRContext.forward``
  step      forward and backward with buffers the program keeps: project, bin, render_fwd, render_bwd
  autograd  the differentiable ``render()`` and ``torch.autograd.grad`` through it
  graph     the step captured once (``GraphStep``) and replayed
  train     ``TrainStep.step``: forward, l1 + D-SSIM loss, backward, Adam
  sorted    sorted alpha blending of the same splats (Eq. 6), the comparison the paper draws

``exact`` evaluates the same quantities from their definitions in float64 with plain torch operations.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2410_18931_amd import WSRContext, globals_tensor, render
from paper_2410_18931_amd.graph import GraphStep
from paper_2410_18931_amd.train import TrainStep, default_lrs
from wsr_synth import DC_HALF_RANGE, Settings, look_at_camera

KEYS = ("means", "log_scales", "quats", "sh", "opacity_logit", "lc_v")
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
TRAINED = 1000       # Adam step at which the training cases start: moments are in place, rates have decayed
LR_SCALE = 0.01      # learning rates late in training, relative to the first step's


def _case(name, path, n, width, height, **kw):
    c = {"path": path, "n": n, "width": width, "height": height, "views": 1, "scene": "blobs", "degree": 3,
         "weight": "lc", "opacity": "sh", "storage": "f32", "oit": False, "alpha_cut": 0.0, "alpha_min": 0.0,
         "t_min": 0.0, "grow": False}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    small = {"scene": "cloud", "degree": 0, "weight": "exp", "opacity": "logit"}
    return [
        # a thumbnail or a quick preview: 4,096 Gaussians, called with the defaults (the pair count is read back)
        _case("forward_4k_128", "forward", 4096, 128, 128, grow=True, **small),
        # a small fit driven by autograd, nothing a multiple of a tile or a wave
        _case("autograd_5k_odd", "autograd", 5003, 201, 133, grow=True, **dict(small, degree=1)),
        # one 720p view of a mid-sized scene, buffers kept
        _case("step_200k_720p", "step", 200_000, 1280, 720, scene="cloud"),
        # gradients into a 16-bit scene through autograd, at a ragged size
        _case("autograd_300k_bf16", "autograd", 300_007, 1001, 747, degree=2, storage="bf16", grow=True),
        # serving: forward only from half-precision attributes
        _case("forward_1m_f16", "forward", 1_000_000, 1920, 1080, storage="f16"),
        # the benchmark's step: 1 M Gaussians, one 1080p view
        _case("step_1m_1080p", "step", 1_000_000, 1920, 1080),
        # the same with the two options that change the raster kernels
        _case("step_1m_oit", "step", 1_000_000, 1920, 1080, oit=True),
        _case("step_1m_earlyout", "step", 1_000_000, 1920, 1080, alpha_cut=1.0 / 255.0),
        # the sorted comparison with the usual skip and early stop
        _case("sorted_1m_1080p", "sorted", 1_000_000, 1920, 1080, weight="dir", alpha_min=1.0 / 255.0, t_min=1e-4),
        # training: a small scene seen by three odd-sized views with the defaults, and the benchmark's size
        _case("train_30k_3views", "train", 30_011, 407, 301, views=3, scene="cloud", grow=True),
        _case("train_1m_1080p", "train", 1_000_000, 1920, 1080),
        # the batched benchmark: 16 views of uneven size, the step replayed as one graph
        _case("graph_1m_16views", "graph", 1_000_000, 1920, 1080, views=16),
    ]


def draw(rng: random.Random):
    """A case of the same ranges: images from 96 to 1920 pixels wide, 1,000 Gaussians to half a million."""
    def log_uniform(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    path = rng.choice(["forward", "step", "step", "autograd", "graph", "train", "sorted"])
    width = log_uniform(96, 1920)
    height = max(64, int(width * rng.uniform(0.5, 0.8)))
    n = log_uniform(1000, max(2000, min(500_000, width * height // 2)))
    kw = {"views": 1 if path == "sorted" else rng.choice([1, 1, 2, 3]), "scene": rng.choice(["cloud", "blobs"]),
          "degree": rng.choice([0, 1, 2, 3, 3]), "grow": path != "graph" and rng.random() < 0.3}
    if path == "sorted":
        kw["weight"] = "dir"
        if rng.random() < 0.5:
            kw.update(alpha_min=1.0 / 255.0, t_min=1e-4)
    else:
        kw["weight"] = rng.choice(["dir", "exp", "lc", "lc"])
        option = rng.choice(["none", "none", "oit", "cut"])
        kw["oit"] = option == "oit"
        kw["alpha_cut"] = 1.0 / 255.0 if option == "cut" else 0.0
    kw["opacity"] = rng.choice(["logit", "sh"])
    kw["storage"] = "f32" if path == "train" else rng.choice(["f32", "f32", "f16", "bf16"])
    return _case(None, path, n, width, height, **kw)


# ------------------------------------------------------------------------------------------------ inputs

def _settings(case):
    s = {"exp": 0.1, "lc": 10.0, "dir": 0.1}[case["weight"]]
    return Settings(weight_kind=case["weight"], opacity_mode=case["opacity"], sigma=s, beta=0.8, oit=case["oit"],
                    alpha_cut=case["alpha_cut"])


def _cameras(case, seed):
    """View v's size is fixed by the case, its position by the seed (the first looks along z from distance 4)."""
    r = random.Random(seed)
    cams = [look_at_camera((0.0, 0.0, -4.0), case["width"], case["height"])]
    for v in range(1, case["views"]):
        f = 1 / 3 + 2 / 3 * ((5 * v) % case["views"]) / case["views"]
        w, h = max(16, int(case["width"] * f)), max(16, int(case["height"] * f))
        d = [r.gauss(0.0, 1.0) for _ in range(3)]
        s = r.uniform(4.0, 6.0) / math.sqrt(sum(x * x for x in d))
        cams.append(look_at_camera([x * s for x in d], w, h))
    return cams


def _scene(case, seed, device, n=None):
    """The attribute distributions of the synthetic benchmark scenes, drawn on the device."""
    g = torch.Generator(device=device).manual_seed(seed)
    n = case["n"] if n is None else n

    def normal(*shape):
        return torch.randn(shape, generator=g, device=device)

    def uniform(a, b, *shape):
        return a + (b - a) * torch.rand(shape, generator=g, device=device)

    k = (case["degree"] + 1) ** 2
    if case["scene"] == "blobs":
        blob = torch.randint(0, 32, (n,), generator=g, device=device)
        means = (2.0 * normal(3, 32))[:, blob] + normal(3, n) * uniform(0.2, 0.6, 32)[blob]
        logs = -4.0 + 0.7 * normal(3, n)
    else:
        big = case["degree"] == 3
        means = (2.0 if big else 1.0) * normal(3, n)
        logs = (-4.0 if big else -3.0) + (0.7 if big else 0.5) * normal(3, n)
    quats = normal(4, n)
    sh = 0.1 * normal(k, n, 4)
    sh[0] = uniform(-DC_HALF_RANGE, DC_HALF_RANGE, n, 4)
    s = {"means": means, "log_scales": logs, "quats": quats / quats.norm(dim=0), "sh": sh,
         "opacity_logit": normal(n), "lc_v": uniform(0.5, 1.5, n)}
    dt = DTYPES[case["storage"]]
    return {key: (t.to(dt) if key in ("means", "log_scales", "quats", "sh") else t).contiguous()
            for key, t in s.items()}


def _upstream(case, pixels, seed, device):
    g = torch.Generator(device=device).manual_seed(seed + 7)
    return torch.randn((pixels, 3), generator=g, device=device)


def _moments(case, pixels, shapes, seed, device):
    """Adam's moments in the middle of a run: first moments of the gradients' size, second moments above it."""
    g = torch.Generator(device=device).manual_seed(seed + 13)
    r = 1.0 / pixels
    m = {k: r * torch.randn(s, generator=g, device=device) for k, s in shapes.items()}
    v = {k: r * r * (1.0 + torch.rand(s, generator=g, device=device)) for k, s in shapes.items()}
    return m, v


def _shapes(case):
    n, k = case["n"], (case["degree"] + 1) ** 2
    return {"means": (3, n), "log_scales": (3, n), "quats": (4, n), "sh": (k, n, 4), "opacity_logit": (n,),
            "lc_v": (n,), "globals": (6,)}


def _lrs():
    return {k: LR_SCALE * v for k, v in default_lrs().items()}


def _target(scene):
    """The image a training case fits: the same scene with its degree-0 colour shifted."""
    t = dict(scene)
    t["sh"] = scene["sh"].clone()
    t["sh"][0, :, :3] += 0.1
    return t


def prepare(case, seed):
    dev = "cuda"
    st, cams, scene = _settings(case), _cameras(case, seed), _scene(case, seed, "cuda")
    g = globals_tensor(st)
    ctx = WSRContext(case["n"], cams, st)
    s = {"case": case, "ctx": ctx, "scene": scene, "g": g}
    path = case["path"]
    if path != "graph":
        source = _target(scene) if path == "train" else scene
        image = ctx.forward(source, g)[0]         # sizes the pair buffer
        if not case["grow"]:
            ctx._alloc_pairs(int(ctx.last_pairs * (1.3 if path == "train" else 1.1)) + 1024)
    P = ctx.total_pixels
    if path in ("step", "autograd", "graph"):
        s["dL"] = _upstream(case, P, seed, dev)
    if path == "step":
        s["out"] = (torch.empty((P, 3), device=dev), torch.empty((P,), device=dev))
        s["grads"] = ctx.alloc_grads(scene)
    elif path == "graph":
        s["graph"] = GraphStep(ctx, scene, g, s["dL"])
    elif path == "train":
        t = TrainStep(ctx, scene, g.clone(), image.clone(), lrs=_lrs(), grow=case["grow"])
        t.it = TRAINED
        m, v = _moments(case, P, _shapes(case), seed, dev)
        for key in t.m:
            t.m[key].copy_(m[key])
            t.v[key].copy_(v[key])
        s["train"] = t
    elif path == "autograd":
        s["leaves"] = [g.requires_grad_()] + [scene[k].requires_grad_() for k in KEYS]
    return s


def run(state):
    case, ctx, scene, g = state["case"], state["ctx"], state["scene"], state["g"]
    path = case["path"]
    if path == "forward":
        return list(ctx.forward(scene, g, grow=case["grow"]))
    if path == "step":
        ctx.project(scene, g)
        ctx.bin(grow=case["grow"])
        rgb, den = ctx.render_fwd(g, out=state["out"])
        return [rgb, den, ctx.render_bwd(scene, g, state["dL"], rgb, den, grads=state["grads"])]
    if path == "autograd":
        rgb, den = render(scene, g, ctx)
        grads = torch.autograd.grad(rgb, state["leaves"], state["dL"])
        return [rgb.detach(), den, dict(zip(("globals",) + KEYS, grads))]
    if path == "graph":
        s = state["graph"]
        s.replay()
        return [s.rgb, s.den, s.grads]
    if path == "train":
        t = state["train"]
        return {"loss": t.step(), "scene": t.scene, "globals": t.globals_, "m": t.m, "v": t.v}
    ctx.project(scene, g)
    ctx.bin(grow=case["grow"])
    return list(ctx.render_sorted(g, alpha_min=case["alpha_min"], t_min=case["t_min"]))


# ------------------------------------------------------------------------------------------------ the work of a pass

def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the in-support (pixel, Gaussian) pairs, whose
    number is the image share of the splats' support ellipses (from a sample of the scene)."""
    n, nv = case["n"], case["views"]
    st = _settings(case)
    sample = min(n, max(2000, 20_000 // nv))
    p = {k: t.double() for k, t in _scene(case, 0, "cpu", n=sample).items()}
    glob = globals_tensor(st, device="cpu").double()
    pixels, pairs = 0, 0.0
    for cam in _cameras(case, 0):
        with torch.no_grad():
            s = _splats(p, glob, cam, st)
        W, H = cam["width"], cam["height"]
        pixels += W * H
        inside = s["alive"] & (s["mux"] >= 0) & (s["mux"] < W) & (s["muy"] >= 0) & (s["muy"] < H)
        area = math.pi * s["cut"] / torch.sqrt((s["A"] * s["C"] - s["B"] ** 2).clamp(min=1e-30))
        pairs += float(area[inside].clamp(max=W * H).sum()) * n / sample
    k = (case["degree"] + 1) ** 2
    size = 4 if case["storage"] == "f32" else 2
    attr = n * ((10 + 4 * k) * size + 4)
    image = pixels * 16
    if case["path"] in ("forward", "sorted"):
        return {"bytes": attr + image, "flops": 20 * pairs}
    flops = (23 + 56 if case["oit"] else 20 + 48) * pairs
    if case["path"] == "train":
        return {"bytes": 24 * n * (10 + 4 * k + 2) + pixels * 12, "flops": flops}
    out = n * ((10 + 4 * k) * (size if case["path"] == "autograd" else 4) + 8)
    return {"bytes": attr + image + pixels * 12 + out, "flops": flops}


# ------------------------------------------------------------------------------------------------ float64 definitions

def _basis(degree, d):
    """Real spherical harmonics up to degree 3 of the unit vectors d [3][n] -> [K][n]."""
    x, y, z = d
    f = math.sqrt
    pi = math.pi
    out = [torch.full_like(x, f(1 / (4 * pi)))]
    if degree >= 1:
        c = f(3 / (4 * pi))
        out += [c * y, c * z, c * x]
    if degree >= 2:
        c = f(15 / (4 * pi))
        out += [c * x * y, c * y * z, f(5 / (16 * pi)) * (3 * z * z - 1), c * x * z, c / 2 * (x * x - y * y)]
    if degree >= 3:
        a, b = f(35 / (32 * pi)), f(105 / (4 * pi))
        c, e = f(21 / (32 * pi)), f(7 / (16 * pi))
        out += [a * y * (3 * x * x - y * y), b * x * y * z, c * y * (5 * z * z - 1), e * z * (5 * z * z - 3),
                c * x * (5 * z * z - 1), b / 2 * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(out)


def _splats(p, glob, cam, st):
    """Every Gaussian's projected centre, conic, colour, opacity, depth weight and support cutoff for one view."""
    dev = p["means"].device
    view = torch.tensor(cam["viewmat"], dtype=torch.float64, device=dev)
    R, T = view[:, :3], view[:, 3:]
    W, H, fx, fy = cam["width"], cam["height"], cam["fx"], cam["fy"]
    t = R @ p["means"] + T
    tz = t[2]
    vis = tz > st.near
    z = torch.where(vis, tz, torch.ones_like(tz))
    qn = p["quats"].norm(dim=0)
    w, x, y, q = p["quats"] / qn
    rot = torch.stack([1 - 2 * (y * y + q * q), 2 * (x * y - w * q), 2 * (x * q + w * y),
                       2 * (x * y + w * q), 1 - 2 * (x * x + q * q), 2 * (y * q - w * x),
                       2 * (x * q - w * y), 2 * (y * q + w * x), 1 - 2 * (x * x + y * y)]).reshape(3, 3, -1)
    M = rot * p["log_scales"].exp()[None]                   # Sigma = M M^T
    limx, limy = 1.3 * 0.5 * W / fx, 1.3 * 0.5 * H / fy
    rx, ry = (t[0] / z).clamp(-limx, limx), (t[1] / z).clamp(-limy, limy)
    a = (fx / z) * (R[0][:, None] - rx * R[2][:, None])     # rows of J W
    b = (fy / z) * (R[1][:, None] - ry * R[2][:, None])
    aM, bM = (a[:, None] * M).sum(0), (b[:, None] * M).sum(0)
    c00, c01, c11 = (aM * aM).sum(0) + st.dilation, (aM * bM).sum(0), (bM * bM).sum(0) + st.dilation
    det = c00 * c11 - c01 * c01
    vis = vis & (det > 0)
    mux, muy = fx * t[0] / z + cam["cx"], fy * t[1] / z + cam["cy"]
    vis = vis & (mux.abs() < 2 ** 22) & (muy.abs() < 2 ** 22)
    d = p["means"] + (R.T @ T)
    basis = _basis(int(round(math.sqrt(p["sh"].shape[0]))) - 1, d / d.norm(dim=0))
    raw = (basis[:, :, None] * p["sh"]).sum(0)
    rgb = (raw[:, :3] + 0.5).clamp(min=0.0)
    u = raw[:, 3] + st.opacity_offset if st.opacity_mode == "sh" else torch.sigmoid(p["opacity_logit"])
    if st.weight_kind == "dir":
        wd = torch.ones_like(z)
    elif st.weight_kind == "exp":
        wd = torch.exp(-glob[0] * z ** glob[1])
    else:
        wd = (1 - z / glob[0]).clamp(min=0.0) * p["lc_v"]
    cut = torch.full_like(z, st.tau)
    alive = vis
    if st.alpha_cut > 0:
        least = float(torch.tensor(st.alpha_cut, dtype=torch.float32))
        alive = vis & (u > least)
        cut = torch.where(alive, torch.minimum(cut, 2 * torch.log((u / least).clamp(min=1.0))), cut).detach()
    return {"alive": alive, "mux": mux, "muy": muy, "A": c11 / det, "B": -c01 / det, "C": c00 / det, "rgb": rgb,
            "u": u, "amp": u * wd, "cut": cut, "depth": tz.detach().float(),
            "ex": torch.sqrt(cut * c00).detach(), "ey": torch.sqrt(cut * c11).detach()}


_T = 16


def _tile_lists(s, cam):
    """(Gaussian, tile) pairs grouped by tile, each tile's Gaussians in (depth, id) order, as batches of tiles of
    similar list length: (tile ids [t], Gaussian ids [t][L], valid [t][L])."""
    W, H = cam["width"], cam["height"]
    tx, ty = -(-W // _T), -(-H // _T)

    def span(mu, e, size):
        lo, hi = torch.ceil(mu - e - 0.5) - 1, torch.floor(mu + e - 0.5) + 1
        return lo, hi, (lo.clamp(0, size - 1) // _T).long(), (hi.clamp(0, size - 1) // _T).long() + 1

    lx, hx, x0, x1 = span(s["mux"].detach(), s["ex"], W)
    ly, hy, y0, y1 = span(s["muy"].detach(), s["ey"], H)
    on = s["alive"] & (hx >= 0) & (lx <= W - 1) & (hy >= 0) & (ly <= H - 1)
    order = torch.argsort(s["depth"], stable=True)
    order = order[on[order]]
    w = (x1 - x0)[order]
    cnt = w * (y1 - y0)[order]
    g = torch.repeat_interleave(order, cnt)
    first = torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
    k = torch.arange(g.numel(), device=g.device) - first
    ww = torch.repeat_interleave(w, cnt)
    tile = (y0[g] + k // ww) * tx + x0[g] + k % ww
    tile, by = torch.sort(tile, stable=True)
    g = g[by]
    length = torch.bincount(tile, minlength=tx * ty)
    start = length.cumsum(0) - length
    by_len = torch.argsort(length, descending=True, stable=True)
    lens = length[by_len].tolist()
    k = 0
    while k < len(lens):
        L = max(1, lens[k])
        t = max(1, min(len(lens) - k, 32_768 // L))
        ids = by_len[k:k + t]
        pos = torch.arange(L, device=g.device)[None]
        valid = pos < length[ids][:, None]
        at = (start[ids][:, None] + pos).clamp(max=max(g.numel() - 1, 0))
        yield ids, (g[at] if g.numel() else torch.zeros_like(at)), valid
        k += t


def _falloff(s, ids, gid, valid, cam):
    """(G [t][L][256], pixel index [t][256] (-1 outside the image), pixel offsets from the tile's centre [256][2])."""
    W, H = cam["width"], cam["height"]
    tx = -(-W // _T)
    dev = gid.device
    k = torch.arange(_T * _T, device=dev)
    ox, oy = (k % _T).double() + 0.5 - _T / 2, (k // _T).double() + 0.5 - _T / 2
    cx, cy = (ids % tx * _T + _T // 2)[:, None].double(), (ids // tx * _T + _T // 2)[:, None].double()
    mx, my = s["mux"][gid] - cx, s["muy"][gid] - cy
    A, B, C = s["A"][gid], s["B"][gid], s["C"][gid]
    coef = torch.stack([A, 2 * B, C, -2 * (A * mx + B * my), -2 * (C * my + B * mx),
                        A * mx * mx + 2 * B * mx * my + C * my * my], dim=-1)
    q = coef @ torch.stack([ox * ox, ox * oy, oy * oy, ox, oy, torch.ones_like(ox)])
    keep = (q <= s["cut"][gid][..., None]) & valid[..., None]
    G = torch.where(keep, torch.exp(-0.5 * q), torch.zeros_like(q))
    px, py = (cx + ox - 0.5).long(), (cy + oy - 0.5).long()
    pix = torch.where((px < W) & (py < H), py * W + px, torch.full_like(px, -1))
    return G, pix, torch.stack([ox, oy], dim=-1), mx, my


def _put(dst, pix, values):
    ok = pix >= 0
    dst[pix[ok]] = values[ok]


def _render_exact(s, glob, cam, st):
    """rgb [P][3], den [P], coverage P and the weighted average (OIT) of one view."""
    P = cam["width"] * cam["height"]
    dev = glob.device
    sums = torch.zeros((P, 4), dtype=torch.float64, device=dev)
    cov = torch.ones((P,), dtype=torch.float64, device=dev)
    feat = torch.cat([s["rgb"] * s["amp"][:, None], s["amp"][:, None]], dim=1)
    for ids, gid, valid in _tile_lists(s, cam):
        G, pix, _, _, _ = _falloff(s, ids, gid, valid, cam)
        _put(sums, pix, G.transpose(1, 2).contiguous() @ (feat[gid] * valid[..., None]))
        if st.oit:
            _put(cov, pix, (1 - (s["u"][gid][..., None] * G).clamp(0, 1)).prod(dim=1))
    N, D = sums[:, :3], sums[:, 3]
    if st.oit:
        avg = torch.where(D[:, None] != 0, N / D[:, None], torch.zeros_like(N))
        return cov[:, None] * glob[3:] + (1 - cov[:, None]) * avg, D, cov, avg
    D = D + glob[2]
    return torch.where(D[:, None] != 0, (N + glob[2] * glob[3:]) / D[:, None], glob[3:].expand_as(N)), D, cov, N


def _backward_exact(s, glob, cam, st, dL, rgb, den, cov, avg):
    """Gradients with respect to the splats' mux, muy, A, B, C, rgb, amp, u and to (w_B, c_B) of one view."""
    dev = glob.device
    n = s["mux"].numel()
    safe = torch.where(den != 0, den, torch.ones_like(den))
    gback = torch.zeros(6, dtype=torch.float64, device=dev)
    if st.oit:
        gbar = torch.where(den != 0, (1 - cov) / safe, torch.zeros_like(den))[:, None] * dL
        sp = (gbar * avg).sum(1)
        kc = cov * (dL * (glob[3:] - avg)).sum(1)
        gback[3:] = (cov[:, None] * dL).sum(0)
    else:
        gbar = torch.where(den != 0, 1 / safe, torch.zeros_like(den))[:, None] * dL
        sp = (gbar * rgb).sum(1)
        kc = torch.zeros_like(den)
        zero = den == 0
        gback[2] = (gbar * (glob[3:] - rgb)).sum()
        gback[3:] = glob[2] * gbar.sum(0) + dL[zero].sum(0)
    out = torch.zeros((n, 10), dtype=torch.float64, device=dev)
    for ids, gid, valid in _tile_lists(s, cam):
        G, pix, o, mx, my = _falloff(s, ids, gid, valid, cam)
        ok = (pix >= 0)[..., None]
        at = pix.clamp(min=0)
        gb = torch.where(ok, gbar[at], torch.zeros_like(gbar[at]))                 # [t][256][3]
        ss = torch.where(ok[..., 0], sp[at], torch.zeros_like(sp[at]))
        dLda = s["rgb"][gid] @ gb.transpose(1, 2).contiguous() - ss[:, None]
        amp = s["amp"][gid]
        e = amp[..., None] * G * dLda
        du = torch.zeros_like(amp)
        if st.oit:
            al = s["u"][gid][..., None] * G
            kk = torch.where(ok[..., 0], kc[at], torch.zeros_like(kc[at]))[:, None]
            dal = torch.where((al > 0) & (al < 1), -kk / (1 - al).clamp(min=1e-300), torch.zeros_like(al))
            e = e + al * dal
            du = (G * dal).sum(-1)
        ox, oy = o[:, 0], o[:, 1]
        m = e @ torch.stack([torch.ones_like(ox), ox, oy, ox * ox, ox * oy, oy * oy], dim=1)
        S, X, Y, XX, XY, YY = m.unbind(-1)
        dx, dy = X - mx * S, Y - my * S
        dxx, dyy = XX - 2 * mx * X + mx * mx * S, YY - 2 * my * Y + my * my * S
        dxy = XY - mx * Y - my * X + mx * my * S
        A, B, C = s["A"][gid], s["B"][gid], s["C"][gid]
        cols = torch.stack([A * dx + B * dy, B * dx + C * dy, -0.5 * dxx, -dxy, -0.5 * dyy], dim=-1)
        cols = torch.cat([cols, amp[..., None] * (G @ gb), (G * dLda).sum(-1, keepdim=True), du[..., None]], dim=-1)
        out.index_add_(0, gid[valid], cols[valid])
    return out, gback


def _loss_exact(x, y, cams, lam=0.2):
    """Mean over views of (1 - lam) mean|x - y| + lam (1 - mean SSIM), 11-tap Gaussian windows, zero padding."""
    k = torch.arange(11, dtype=torch.float64, device=x.device) - 5
    w = torch.exp(-k * k / (2 * 1.5 ** 2))
    w = w / w.sum()

    def blur(a):
        for dim, pad in ((1, (0, 0, 5, 5)), (2, (5, 5, 0, 0))):
            b = torch.nn.functional.pad(a, pad)
            a = sum(w[j] * b.narrow(dim, j, a.shape[dim]) for j in range(11))
        return a

    total, o = 0.0, 0
    for c in cams:
        P = c["width"] * c["height"]
        a, b = (t[o:o + P].T.reshape(3, c["height"], c["width"]) for t in (x, y))
        o += P
        u, v = blur(a), blur(b)
        saa, sbb, sab = blur(a * a) - u * u, blur(b * b) - v * v, blur(a * b) - u * v
        c1, c2 = 0.01 ** 2, 0.03 ** 2
        ssim = (2 * u * v + c1) * (2 * sab + c2) / ((u * u + v * v + c1) * (saa + sbb + c2))
        total = total + (1 - lam) * (a - b).abs().mean() + lam * (1 - ssim.mean())
    return total / len(cams)


def _sorted_exact(s, glob, cam, alpha_min, t_min, alpha_max=0.99):
    P = cam["width"] * cam["height"]
    rgb = torch.zeros((P, 3), dtype=torch.float64, device=glob.device)
    T = torch.zeros((P,), dtype=torch.float64, device=glob.device)
    for ids, gid, valid in _tile_lists(s, cam):
        G, pix, _, _, _ = _falloff(s, ids, gid, valid, cam)
        al = (s["amp"][gid][..., None] * G).clamp(max=alpha_max)
        al = torch.where((G > 0) & (al >= alpha_min), al, torch.zeros_like(al))
        before = torch.cat([torch.ones_like(al[:, :1]), torch.cumprod(1 - al, dim=1)[:, :-1]], dim=1)
        al = torch.where(before >= t_min, al, torch.zeros_like(al))
        w = al * before
        left = (1 - al).prod(dim=1)
        _put(T, pix, left)
        _put(rgb, pix, w.transpose(1, 2).contiguous() @ s["rgb"][gid] + left[..., None] * glob[3:])
    return rgb, T


def exact(case, seed):
    st, cams, scene = _settings(case), _cameras(case, seed), _scene(case, seed, "cuda")
    glob = globals_tensor(st).double()
    p = {k: t.double() for k, t in scene.items()}
    path = case["path"]
    if path == "sorted":
        s = _splats(p, glob, cams[0], st)
        return list(_sorted_exact(s, glob, cams[0], case["alpha_min"], case["t_min"]))

    def images(q):
        with torch.no_grad():
            return [_render_exact(_splats(q, glob, c, st), glob, c, st) for c in cams]

    imgs = images(p)
    rgb, den = torch.cat([i[0] for i in imgs]), torch.cat([i[1] for i in imgs])
    if path == "forward":
        return [rgb, den]
    pixels = rgb.shape[0]
    if path == "train":
        target = torch.cat([i[0] for i in images({k: t.double() for k, t in _target(scene).items()})])
        target = target.float().double()          # the program holds its target images in float32
        x = rgb.clone().requires_grad_()
        loss = _loss_exact(x, target, cams)
        dL = torch.autograd.grad(loss, x)[0]
    else:
        dL = _upstream(case, pixels, seed, "cuda").double()
    grads = {k: torch.zeros_like(t) for k, t in p.items()}
    grads["globals"] = torch.zeros(6, dtype=torch.float64, device=glob.device)
    o = 0
    for cam, (c_rgb, c_den, c_cov, c_avg) in zip(cams, imgs):
        P = c_den.numel()
        leaves = {k: t.detach().requires_grad_() for k, t in p.items()}
        gl = glob.detach().requires_grad_()
        s = _splats(leaves, gl, cam, st)
        with torch.no_grad():
            d, gback = _backward_exact({k: t.detach() for k, t in s.items()}, glob, cam, st, dL[o:o + P], c_rgb,
                                       c_den, c_cov, c_avg)
        grads["globals"] += gback
        keep = s["alive"][:, None]
        d = torch.where(keep, d, torch.zeros_like(d))
        outs = [s["mux"], s["muy"], s["A"], s["B"], s["C"], s["rgb"], s["amp"], s["u"]]
        seeds = [d[:, 0], d[:, 1], d[:, 2], d[:, 3], d[:, 4], d[:, 5:8], d[:, 8], d[:, 9]]
        got = torch.autograd.grad(outs, list(leaves.values()) + [gl], seeds, allow_unused=True)
        for k, t in zip(list(leaves) + ["globals"], got):
            if t is not None:
                grads[k] += t
        o += P
    if path != "train":
        return [rgb, den, grads]
    m, v = _moments(case, pixels, _shapes(case), seed, "cuda")
    m = {k: 0.9 * m[k].double() + 0.1 * grads[k] for k in m}
    v = {k: 0.999 * v[k].double() + 0.001 * grads[k] ** 2 for k in v}
    lrs, step = _lrs(), TRAINED + 1
    new = {}
    for k, t in {**p, "globals": glob}.items():
        lr = lrs.get(k)
        if k == "sh":
            lr = torch.full((t.shape[0], 1, 1), lrs["shN"], dtype=torch.float64, device=t.device)
            lr[0] = lrs["sh0"]
        new[k] = t - lr * (m[k] / (1 - 0.9 ** step)) / (torch.sqrt(v[k] / (1 - 0.999 ** step)) + 1e-15)
    return {"loss": loss.detach().reshape(1), "scene": {k: new[k] for k in KEYS}, "globals": new["globals"], "m": m,
            "v": v}
