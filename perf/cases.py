"""The work this library is timed on, as a program that uses it would ask for it.

Each case is one call (or the few calls that go together) of the public entry
points on one batch, over the range of sizes that a barn camera installation
meets: one live frame of some hundred birds, batches of recorded video, a
whole house of 30000 birds in one frame, a minute of video at once.

  listed()        the cases that are always timed
  draw(rng)       another case of the same ranges
  prepare         a batch in device memory, and the output buffers a serving
                  loop keeps
  run             one pass through the entry points
  work            bytes and flops that a pass cannot do without
  tolerance       what another correct implementation may differ by
  exact           the floating-point outputs in 64 bits, in plain torch

Inputs are synthetic and made on the GPU from the seed alone: birds in
Gaussian groups over a uniform background (groups differ from frame to frame),
or one flock walking from frame to frame; smooth heatmaps; probability maps
with one soft ellipse per bird and single-pixel false positives.
"""

from __future__ import annotations

import math

import torch

import paper_2512_07009_amd as flock

QUANTA = 16  # positions are in 1/16 px


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _birds(frames, birds, width, height, **more):
    """A batch of `frames` frames with at most `birds` birds each."""
    case = {"frames": frames, "birds": birds, "width": width, "height": height,
            "ragged": 0,       # 0: every frame full; r: counts from birds / r to birds, some frames empty
            "bounded": True,   # whether the caller knows the largest frame
            "walk": False,     # one flock walking on from frame to frame
            "groups": 6, "group_lo": 80.0, "group_hi": 200.0, "uniform": 0.1,  # where the birds are
            "eps": 40.0, "min_pts": 4, "grid_w": 128, "grid_h": 72, "sigma": 30.0}
    case.update(more)
    return case


def listed():
    return [
        # a live camera: one small frame, clustered and mapped as it arrives,
        # results in new tensors
        dict(_birds(1, 500, 1920, 1080, uniform=1.0, grid_w=64, grid_h=36), kind="live", name="live 1x500"),
        # about two seconds of recorded 30 fps video
        dict(_birds(64, 2000, 1920, 1080), kind="cluster", name="cluster 64x2000"),
        # a minute of video at once
        dict(_birds(1800, 5000, 1920, 1080, walk=True), kind="cluster", name="cluster 1800x5000"),
        # a whole house in one frame
        dict(_birds(1, 30000, 3840, 2160, groups=20, group_lo=40.0, group_hi=40.0, uniform=0.7, eps=25.0, min_pts=6),
             kind="cluster", name="cluster 1x30000"),
        # cameras of different pens in one batch, frame sizes not known to the
        # caller: small frames, large ones, empty ones
        dict(_birds(96, 20000, 3840, 2160, ragged=64, bounded=False, groups=12, group_lo=60.0, group_hi=300.0,
                    uniform=0.05, eps=60.0, min_pts=5), kind="cluster", name="cluster ragged"),
        dict(_birds(64, 2000, 1920, 1080), kind="density", name="density 64x2000"),
        # 4K video on a fine grid
        dict(_birds(256, 8800, 3840, 2160, ragged=1.2, groups=12, group_lo=60.0, group_hi=300.0, uniform=0.0,
                    grid_w=256, grid_h=144, sigma=45.0), kind="density", name="density 256x8000 4k"),
        # a grid whose cells are no whole number of 1/16 px
        dict(_birds(48, 3000, 1280, 720, ragged=4, grid_w=97, grid_h=61, sigma=25.0), kind="density",
             name="density odd grid"),
        {"kind": "heatmap", "name": "heatmap 64x128x72", "frames": 64, "grid_w": 128, "grid_h": 72, "connectivity": 8},
        # the whole-house grid
        {"kind": "heatmap", "name": "heatmap 1x512x288", "frames": 1, "grid_w": 512, "grid_h": 288, "connectivity": 8},
        # the counts of a minute of video: birds along the wall, birds at the
        # drinker lines
        dict(_birds(1800, 5000, 1920, 1080, walk=True), kind="zones", vertices=5, lines=2, reach=20.0,
             name="zones 1800x5000"),
        # a segmentation network's batch
        {"kind": "masks", "name": "masks 8x1280x720", "frames": 8, "width": 1280, "height": 720, "birds": 2000,
         "connectivity": 8, "labels": True},
    ]


_CAMERAS = [(1280, 720), (1920, 1080), (2592, 1944), (3840, 2160)]


def _log_int(rng, lo, hi):
    return max(int(lo), min(int(hi), int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_birds(rng, most_frames=1800, most_birds=30000, most_total=2_000_000):
    birds = _log_int(rng, 20, most_birds)
    frames = min(_log_int(rng, 1, most_frames), max(1, most_total // birds))
    width, height = rng.choice(_CAMERAS)
    lo = rng.uniform(0.01, 0.05) * width
    cell = rng.choice([7.5, 10.0, 12.0, 15.0, 20.0, 30.0])
    grid_w, grid_h = max(8, int(width / cell)), max(8, int(height / cell))
    if rng.random() < 0.4:  # a grid of any size
        grid_w, grid_h = _log_int(rng, 16, 400), _log_int(rng, 16, 300)
    return _birds(frames, birds, width, height, ragged=rng.choice([0, 1.2, 4, 64]), bounded=rng.random() < 0.7,
                  groups=rng.randint(1, 20), group_lo=lo, group_hi=lo * rng.uniform(1.0, 3.0),
                  uniform=rng.choice([0.0, 0.1, 0.3, 0.7, 1.0]), eps=rng.randint(10 * QUANTA, 70 * QUANTA) / QUANTA,
                  min_pts=rng.randint(2, 10), grid_w=grid_w, grid_h=grid_h, sigma=round(rng.uniform(10.0, 60.0), 1))


def draw(rng):
    kind = rng.choice(["live", "cluster", "cluster", "density", "density", "heatmap", "zones", "masks"])
    if kind == "live":
        return dict(_draw_birds(rng, most_frames=1, most_birds=3000), kind=kind)
    if kind == "cluster":
        return dict(_draw_birds(rng), kind=kind)
    if kind == "density":
        case = dict(_draw_birds(rng, most_frames=512), kind=kind)
        cells = case["grid_w"] * case["grid_h"]
        case["frames"] = max(1, min(case["frames"], 9_000_000 // cells))  # grids of at most the largest listed case's size
        return case
    if kind == "heatmap":
        grid_w, grid_h = _log_int(rng, 16, 640), _log_int(rng, 16, 360)
        frames = min(_log_int(rng, 1, 512), max(1, 9_000_000 // (grid_w * grid_h)))
        return {"kind": kind, "frames": frames, "grid_w": grid_w, "grid_h": grid_h, "connectivity": rng.choice([4, 8])}
    if kind == "zones":
        return dict(_draw_birds(rng, most_total=8_000_000), kind=kind, vertices=rng.randint(3, 12), lines=rng.randint(1, 8),
                    reach=rng.randint(5 * QUANTA, 60 * QUANTA) / QUANTA)
    width, height = rng.choice([(640, 360), (641, 479), (1280, 720), (1920, 1080)])
    return {"kind": "masks", "frames": rng.randint(1, 8) if width < 1920 else rng.randint(1, 4), "width": width, "height": height,
            "birds": _log_int(rng, 50, 2500), "connectivity": rng.choice([4, 8]), "labels": rng.random() < 0.7}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _counts(case, g):
    """Birds per frame: spread evenly over the logarithm from birds / ragged to
    birds, one frame in twenty empty, in random order (the same total for
    every seed)."""
    F, n, r = case["frames"], case["birds"], case["ragged"]
    if not r:
        return torch.full((F,), n, dtype=torch.int64, device="cuda")
    u = (torch.arange(F, device="cuda", dtype=torch.float64) + 0.5) / F
    c = torch.round(n * torch.exp(-u * math.log(r))).to(torch.int64).clamp(1, n)
    if F >= 8 and r > 1.5:
        c[7::20] = 0
    return c[torch.randperm(F, generator=g, device="cuda")]


def _inside(v, extent):
    """Positions outside [0, extent) mirrored at the border."""
    v = v.abs()
    return torch.clamp(extent - (extent - v).abs(), 0.0, extent)


def _quanta(x, y, width, height):
    q = torch.stack([torch.floor(x * QUANTA), torch.floor(y * QUANTA)], dim=-1).to(torch.int32)
    q[..., 0].clamp_(0, QUANTA * width - 1)
    q[..., 1].clamp_(0, QUANTA * height - 1)
    return q


def _flock(case, frame, F, g):
    """x and y of one bird per entry of `frame` (its frame), F frames of groups."""
    W, H, k, n = case["width"], case["height"], case["groups"], frame.numel()
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    gx, gy = rand(F, k) * W, rand(F, k) * H
    sd = case["group_lo"] + rand(F, k) * (case["group_hi"] - case["group_lo"])
    at = frame * k + torch.randint(0, k, (n,), generator=g, device="cuda")
    sd = sd.reshape(-1)[at]
    x = gx.reshape(-1)[at] + sd * torch.randn(n, generator=g, device="cuda")
    y = gy.reshape(-1)[at] + sd * torch.randn(n, generator=g, device="cuda")
    alone = rand(n) < case["uniform"]
    x = torch.where(alone, rand(n) * W, _inside(x, W))
    y = torch.where(alone, rand(n) * H, _inside(y, H))
    return x, y


def _batch(case, seed):
    """(xy int32[T, 2], offsets int32[F + 1], largest frame)"""
    g = _generator(seed)
    F, W, H = case["frames"], case["width"], case["height"]
    if case["walk"]:
        n = case["birds"]
        x, y = _flock(case, torch.zeros(n, dtype=torch.int64, device="cuda"), 1, g)
        xy = torch.empty((F, n, 2), dtype=torch.int32, device="cuda")
        for t in range(F):
            if t:
                step = 2.0 * torch.randn((2, n), generator=g, device="cuda")
                new = torch.rand((3, n), generator=g, device="cuda")
                x = torch.where(new[0] < 0.01, new[1] * W, _inside(x + step[0], W))
                y = torch.where(new[0] < 0.01, new[2] * H, _inside(y + step[1], H))
            xy[t] = _quanta(x, y, W, H)
        offsets = torch.arange(F + 1, device="cuda", dtype=torch.int32) * n
        return xy.reshape(-1, 2), offsets, n
    counts = _counts(case, g)
    frame = torch.repeat_interleave(torch.arange(F, device="cuda"), counts)
    x, y = _flock(case, frame, F, g)
    offsets = torch.zeros(F + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = torch.cumsum(counts, 0).to(torch.int32)
    return _quanta(x, y, W, H).contiguous(), offsets, int(counts.max())


def _heatmaps(case, seed):
    """Smooth grids float32[F, h, w] in birds per px^2, exact zeros far from every bird."""
    g = _generator(seed)
    F, gw, gh, k = case["frames"], case["grid_w"], case["grid_h"], 48
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    home = torch.randint(0, 6, (F, k), generator=g, device="cuda")
    cx = torch.gather(rand(F, 6), 1, home) + 0.07 * torch.randn(F, k, generator=g, device="cuda")
    cy = torch.gather(rand(F, 6), 1, home) + 0.07 * torch.randn(F, k, generator=g, device="cuda")
    s = (0.01 + 0.03 * rand(F, k)) * max(gw, gh)
    a = 1e-4 + 1e-3 * rand(F, k)
    xs = torch.arange(gw, device="cuda") + 0.5
    ys = torch.arange(gh, device="cuda") + 0.5
    out = torch.zeros((F, gh, gw), device="cuda")
    for i in range(k):
        z = -0.5 / (s[:, i] * s[:, i])
        fx = torch.exp((xs[None] - cx[:, i, None] * gw) ** 2 * z[:, None])
        fy = torch.exp((ys[None] - cy[:, i, None] * gh) ** 2 * z[:, None])
        out += (a[:, i, None] * fy)[:, :, None] * fx[:, None, :]
    out[out < 1e-9] = 0.0
    return out


def _masks(case, seed):
    """Probability maps float32[F, H, W]."""
    g = _generator(seed)
    F, W, H, n = case["frames"], case["width"], case["height"], case["birds"]
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    out = rand(F, H, W) * 0.1
    flock_of = {"width": W, "height": H, "groups": 6, "group_lo": W / 24.0, "group_hi": W / 9.6, "uniform": 0.1}
    scale = W / 1280.0
    r = int(math.ceil(11.0 * scale)) + 1
    d = torch.arange(-r, r + 1, device="cuda")
    for f in range(F):
        x, y = _flock(flock_of, torch.zeros(n, dtype=torch.int64, device="cuda"), 1, g)
        a, b, th = (7.0 + 3.0 * rand(n)) * scale, (4.0 + 2.0 * rand(n)) * scale, rand(n) * math.pi
        px = (x.long()[:, None, None] + d[None, None, :]).expand(n, 2 * r + 1, 2 * r + 1)
        py = (y.long()[:, None, None] + d[None, :, None]).expand(n, 2 * r + 1, 2 * r + 1)
        dx, dy = px + 0.5 - x[:, None, None], py + 0.5 - y[:, None, None]
        co, si = torch.cos(th)[:, None, None], torch.sin(th)[:, None, None]
        u, v = (dx * co + dy * si) / a[:, None, None], (dy * co - dx * si) / b[:, None, None]
        p = (1.15 - 0.6 * (u * u + v * v)).clamp(0.0, 1.0)
        ok = (px >= 0) & (px < W) & (py >= 0) & (py < H)
        out[f].view(-1).scatter_reduce_(0, (py * W + px)[ok], p[ok], "amax")
    speckle = rand(F, H, W)
    return torch.where(speckle < 2e-4, 0.5 + speckle * 2.4e3, out)


def _threshold(case, density):
    """Hot cells: twice the average density."""
    return 2.0 * float(density.double().mean())


def _area(case):
    return (1920.0 / case["grid_w"]) * (1080.0 / case["grid_h"])


def _polygon(case, seed):
    """A region along the left wall: the closed polygon's corners in 1/16 px,
    its edge to the right ragged."""
    W, H, v = QUANTA * case["width"], QUANTA * case["height"], case["vertices"]
    r = torch.Generator()
    r.manual_seed(int(seed))
    u = torch.rand(v, generator=r).tolist()
    edge = [[int(W * (0.08 + 0.12 * u[i])), H * i // max(1, v - 3)] for i in range(v - 2)]
    return [[0, 0]] + edge + [[0, H]]


def _lines(case, seed):
    """Drinker lines across the frame (segments in 1/16 px)."""
    W, H, k = QUANTA * case["width"], QUANTA * case["height"], case["lines"]
    r = torch.Generator()
    r.manual_seed(int(seed) + 1)
    u = (torch.rand(k, generator=r) * 0.04).tolist()
    return [[W // 10, int(H * ((2 * i + 1) / (2 * k) + u[i])), 9 * W // 10, int(H * ((2 * i + 1) / (2 * k) - u[i]))]
            for i in range(k)]


def _new(*shape, dtype=torch.int32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "heatmap":
        s["density"] = _heatmaps(case, seed)
        s["threshold"] = _threshold(case, s["density"])
        F, gh, gw = s["density"].shape
        s["out"] = {"labels": _new(F, gh, gw), "n_components": _new(F), "entropy": _new(F, dtype=torch.float64),
                    "degree": _new(F, dtype=torch.float64), "comp_cells": _new(F, gh, gw),
                    "comp_mass": _new(F, gh, gw, dtype=torch.float64)}
        return s
    if kind == "masks":
        F, W, H = case["frames"], case["width"], case["height"]
        s["prob"] = _masks(case, seed)
        C = s["capacity"] = F * (2 * case["birds"] + 1024)
        s["out"] = {"labels": _new(F, H, W) if case["labels"] else None, "n_components": _new(F), "offsets": _new(F + 1),
                    "label": _new(C), "area": _new(C), "box": _new(C, 4), "centroid": _new(C, 2, dtype=torch.float64),
                    "xy": _new(C, 2), "score": _new(C, dtype=torch.float32)}
        return s
    s["xy"], s["offsets"], largest = _batch(case, seed)
    s["bound"] = largest if case["bounded"] else 0
    F, T = case["frames"], s["xy"].shape[0]
    if kind == "cluster":
        s["out"] = (_new(T), _new(T, dtype=torch.uint8), _new(F))
    elif kind == "density":
        s["out"] = _new(F, case["grid_h"], case["grid_w"], dtype=torch.float32)
    elif kind == "zones":
        s["polygon"], s["lines"] = _polygon(case, seed), _lines(case, seed)
        s["roi"] = {"counts": _new(F), "xy": _new(T, 2), "offsets": _new(F + 1), "index": _new(T)}
        s["near"] = {"drinking": _new(T, dtype=torch.uint8), "line": _new(T), "counts": _new(F)}
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "cluster":
        return flock.cluster_frames(state["xy"], state["offsets"], case["eps"], case["min_pts"], state["bound"],
                                    out=state["out"])
    if kind == "density":
        return flock.density_frames(state["xy"], state["offsets"], case["width"], case["height"], case["grid_w"],
                                    case["grid_h"], case["sigma"], state["bound"], out=state["out"])
    if kind == "live":
        clusters = flock.cluster_frames(state["xy"], state["offsets"], case["eps"], case["min_pts"], state["bound"])
        density = flock.density_frames(state["xy"], state["offsets"], case["width"], case["height"], case["grid_w"],
                                       case["grid_h"], case["sigma"], state["bound"])
        return {"clusters": clusters, "density": density}
    if kind == "heatmap":
        return flock.heatmap_frames(state["density"], _area(case), state["threshold"], case["connectivity"],
                                    out=state["out"])
    if kind == "zones":
        roi = flock.roi_filter_frames(state["xy"], state["offsets"], state["polygon"], out=state["roi"])
        near = flock.drinker_proximity_frames(state["xy"], state["offsets"], state["lines"],
                                              int(case["reach"] * QUANTA), out=state["near"])
        return {"roi": roi, "near": near}
    return flock.mask_components_frames(state["prob"], 0.5, case["connectivity"], capacity=state["capacity"],
                                        out=state["out"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _total(case):
    """Birds of the batch, about."""
    n, r = case["birds"], case["ragged"]
    mean = n if not r or r <= 1 else n * (1 - 1 / r) / math.log(r)
    return case["frames"] * mean


def work(case):
    kind = case["kind"]
    if kind == "heatmap":
        return {"bytes": case["frames"] * (20.0 * case["grid_w"] * case["grid_h"] + 20), "flops": 0}
    if kind == "masks":
        px = float(case["frames"] * case["width"] * case["height"])
        comps = case["frames"] * 0.25 * case["birds"] + 2e-4 * px
        return {"bytes": (8 if case["labels"] else 4) * px + 52 * comps, "flops": 0}
    T, F = _total(case), case["frames"]
    clusters = 13 * T + 8 * F  # xy in, labels and kinds out
    grid = 8 * T + 4.0 * F * (case["grid_w"] * case["grid_h"] + 1)
    # every bird adds to the cells within about 6 sigma of it
    reach = [min(n, 12 * case["sigma"] * n / extent + 1) for n, extent in
             ((case["grid_w"], case["width"]), (case["grid_h"], case["height"]))]
    flops = 2 * T * reach[0] * reach[1]
    if kind == "cluster":
        return {"bytes": clusters, "flops": 0}
    if kind == "density":
        return {"bytes": grid, "flops": flops}
    if kind == "live":
        return {"bytes": clusters + grid, "flops": flops}
    # zones: xy in twice; kept birds (about 14 % of the frame lies in the
    # region) and their indices; flag and line of every bird
    return {"bytes": 2 * 8 * T + 12 * 0.14 * T + 5 * T + 20 * F, "flops": 0}


# ---------------------------------------------------------------------------
# Tolerances and 64-bit results
# ---------------------------------------------------------------------------

def tolerance(case):
    kind = case["kind"]
    if kind in ("density", "live"):
        # fp16 factors, fp32 sums: 3e-5 (many birds per cell) to 1.5e-4 (few)
        # off the 64-bit sum
        return {"rel": 6e-4, "max": 3e-3}
    if kind == "heatmap":
        # fp64 sums of fp32 values, in any order
        return {"rel": 4e-14, "max": 4e-13}
    return "exact"  # integers, and correctly rounded quotients of integers


def _exact_density(case, seed):
    xy, offsets, _ = _batch(case, seed)
    off = offsets.tolist()
    W, H, gw, gh = case["width"], case["height"], case["grid_w"], case["grid_h"]
    s = float(torch.tensor(case["sigma"], dtype=torch.float32))
    cx = (torch.arange(gw, device="cuda", dtype=torch.float64) + 0.5) * (W / gw)
    cy = (torch.arange(gh, device="cuda", dtype=torch.float64) + 0.5) * (H / gh)
    out = torch.zeros((case["frames"], gh, gw), dtype=torch.float64, device="cuda")
    for f in range(case["frames"]):
        p = xy[off[f]:off[f + 1]].double() / QUANTA
        if p.shape[0]:
            fx = torch.exp((cx[:, None] - p[None, :, 0]) ** 2 * (-0.5 / (s * s)))
            fy = torch.exp((cy[:, None] - p[None, :, 1]) ** 2 * (-0.5 / (s * s)))
            out[f] = torch.mm(fy, fx.t().contiguous()) / (2 * math.pi * s * s)
    return out


def _components(hot, connectivity):
    """Smallest flat index of every hot entry's component within its frame's
    grid (index over the whole batch), -1 elsewhere."""
    F, h, w = hot.shape
    n = F * h * w
    at = torch.arange(n, device=hot.device).reshape(F, h, w)
    lab = torch.where(hot, at, n)
    steps = [(0, 1), (1, 0)] + ([(1, 1), (1, -1)] if connectivity == 8 else [])
    while True:
        old = lab
        new = lab.clone()
        for dy, dx in steps:
            a = (slice(None), slice(0, h - dy), slice(max(0, -dx), w - max(0, dx)))
            b = (slice(None), slice(dy, h), slice(max(0, dx), w - max(0, -dx)))
            new[a] = torch.minimum(new[a], lab[b])
            new[b] = torch.minimum(new[b], lab[a])
        new = torch.where(hot, new, n)
        flat = torch.cat([new.reshape(-1), torch.tensor([n], device=hot.device)])
        for _ in range(4):
            flat = flat[flat]
        lab = torch.where(hot, flat[:n].reshape(F, h, w), n)
        if torch.equal(lab, old):
            return torch.where(hot, lab, -1)


def _exact_heatmap(case, seed):
    density = _heatmaps(case, seed)
    thr = torch.tensor(_threshold(case, density), dtype=torch.float32, device="cuda")
    d = density.double()
    hot = density >= thr
    total = d.sum(dim=(1, 2))
    p = d / total[:, None, None]
    entropy = -torch.where(d > 0, p * torch.log(p), torch.zeros_like(p)).sum(dim=(1, 2))
    degree = torch.where(hot, d, torch.zeros_like(d)).sum(dim=(1, 2)) / total
    lab = _components(hot, case["connectivity"])
    mass = torch.zeros(d.numel(), dtype=torch.float64, device="cuda")
    mass.scatter_add_(0, lab[hot], d[hot])
    return {"labels": None, "n_components": None, "entropy": entropy, "degree": degree, "comp_cells": None,
            "comp_mass": (mass * _area(case)).reshape(d.shape)}


def _exact_masks(case, seed):
    prob = _masks(case, seed)
    F, H, W = prob.shape
    hot = prob > 0.5
    lab = _components(hot, case["connectivity"])
    _, which = torch.unique(lab[hot], return_inverse=True)  # components in order of frame, then first pixel
    at = torch.nonzero(hot.reshape(-1)).reshape(-1) % (H * W)
    C = F * (2 * case["birds"] + 1024)
    zeros = lambda: torch.zeros(C, dtype=torch.float64, device="cuda")  # noqa: E731
    n = zeros().scatter_add_(0, which, torch.ones_like(which, dtype=torch.float64))
    x = zeros().scatter_add_(0, which, (at % W).double())
    y = zeros().scatter_add_(0, which, (at // W).double())
    score = zeros().scatter_reduce_(0, which, prob[hot].double(), "amax")
    one = torch.clamp(n, min=1.0)
    return {"labels": None, "n_components": None, "offsets": None, "label": None, "area": None, "box": None,
            "centroid": torch.stack([x / one, y / one], dim=1), "xy": None, "score": score}


def exact(case, seed):
    kind = case["kind"]
    if kind == "density":
        return _exact_density(case, seed)
    if kind == "live":
        return {"clusters": (None, None, None), "density": _exact_density(case, seed)}
    if kind == "heatmap":
        return _exact_heatmap(case, seed)
    if kind == "masks":
        return _exact_masks(case, seed)
    return None
