"""The work a user of this library has it do, as cases that can be timed and
compared: edge maps of one view and of whole scenes, the split of selected
Gaussians (plain and with the full record), the split mask, and one captured
densification step.

    listed()             the cases, from the smallest call to the largest
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs on the GPU, and the handle a program keeps
    run(state)           one pass through the public entry points
    work(case)           bytes a pass cannot do without
    exact(case, seed)    the outputs of run() in 64-bit torch arithmetic

Views are scene-like renderings made on the GPU (a colour gradient, random
filled polygons, half of them with a sinusoidal texture, and sensor noise of
5 grey levels), of the sizes of the benchmark's workloads; Gaussians,
gradients and pixel contributions follow the benchmark's distributions.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2603_08661_amd as igsp

ASPECT = (1.5, 16.0 / 9.0)
ALPHA, GAMMA, BETA = 0.5, 0.85, 0.6
GRAD_THRESHOLD = math.exp(-9.0 + 0.2533471)   # 40% of exp(N(-9, 1)) lie above it
# what a captured step of the largest listed scene covers
MOST_PIXELS = 586_000_000
MOST_GAUSSIANS = 3_000_000


# ----------------------------------------------------------------- the cases

def _edge(**kw):
    return dict(dict(kind="edge", precision="fp32", form="batched", views=1, w_lo=256, w_hi=256, height=0, halves=False,
                     polygons=60, texture=True, sizes=1), **kw)


def _las(**kw):
    return dict(dict(kind="las", gaussians=10_000, fraction=0.1, ls_mu=-4.0, ls_sd=0.5, record=False, features=0), **kw)


def _mask(**kw):
    return dict(dict(kind="mask", gaussians=100_000, views=8, w_lo=1297, w_hi=1297, height=840, halves=False, order="rows",
                     warmup=False, room=0.2, sizes=1), **kw)


def listed():
    return [
        # one thumbnail, plain FP32: a call that costs its launches
        dict(_edge(form="plain", height=192, polygons=12, texture=False), name="edge_fp32_256x192"),
        # one view of a 4x downsampled capture, plain FP32
        dict(_edge(form="plain", w_lo=1297, w_hi=1297, height=840), name="edge_fp32_1297x840"),
        # a mini-batch of ragged crops and pyramid levels, odd sizes, FP16 storage
        dict(_edge(precision="fp16", views=40, w_lo=33, w_hi=517, polygons=12, sizes=2), name="edge_fp16_40v_ragged"),
        # a small scene with the call's default options (FP32 storage, batched)
        dict(_edge(views=24, w_lo=1000, w_hi=2473, sizes=3), name="edge_fp32_24v"),
        # an indoor scene, 200 views of a 4x downsampled capture, FP16 storage
        dict(_edge(precision="fp16", views=200, w_lo=1000, w_hi=1560, sizes=4), name="edge_fp16_200v"),
        # an outdoor scene at two scales, BF16 storage
        dict(_edge(precision="bf16", views=150, w_lo=2473, w_hi=2473, height=1643, halves=True, sizes=5), name="edge_bf16_150v"),
        # one densification step of a training run, replayed as a HIP graph:
        # maps of 300 views, then the split of a fifth of 3M Gaussians
        dict(_edge(precision="bf16", views=300, w_lo=1000, w_hi=2473, sizes=6), **{k: v for k, v in _las(
            gaussians=3_000_000, fraction=0.2, ls_mu=-4.5, ls_sd=0.7).items() if k != "kind"}, name="step_bf16_300v_3m")
        | {"kind": "step"},
        # the split of a scene's first Gaussians
        dict(_las(), name="las_10k"),
        # the split of a grown scene, few rows selected
        dict(_las(gaussians=1_000_000, fraction=0.05), name="las_1m"),
        # the split a trainer calls: SH features and both Adam moments of every group
        dict(_las(gaussians=3_000_000, fraction=0.2, ls_mu=-4.5, ls_sd=0.7, record=True, features=48), name="las_record_3m_f48"),
        # the selection over a mini-batch of views early in training
        dict(_mask(), name="mask_100k_8v"),
        # the selection over a whole scene
        dict(_mask(gaussians=3_000_000, views=300, w_lo=1000, w_hi=2473, height=0, sizes=6), name="mask_3m_300v"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_views(rng, most_views, most_pixels=MOST_PIXELS):
    w_hi = round(_log(rng, 96, 2473))
    w_lo = max(24, round(w_hi * rng.uniform(0.4, 1.0)))
    room = most_pixels / (w_hi * w_hi / ASPECT[0])
    return dict(views=max(1, min(int(room), round(_log(rng, 1, most_views)))), w_lo=w_lo, w_hi=w_hi, height=0,
                sizes=rng.randrange(10, 1 << 30))


def draw(rng):
    kind = rng.choice(["edge", "edge", "edge", "las", "las", "mask", "step"])
    n = round(_log(rng, 2_000, MOST_GAUSSIANS))
    split = dict(gaussians=n, fraction=round(rng.uniform(0.02, 0.3), 3), ls_mu=-4.0, ls_sd=0.5)
    if kind == "las":
        record = rng.random() < 0.5
        # (the widest record is the listed one's)
        split["fraction"] = min(split["fraction"], 0.2) if record else split["fraction"]
        return _las(record=record, features=rng.choice([0, 3, 9, 27, 45, 48]) if record else 0, **split)
    if kind == "mask":
        order = rng.choice(["rows", "rows", "rows", "spread"])
        c = _mask(order=order, warmup=rng.random() < 0.25, room=round(rng.uniform(0.02, 0.5), 3), **_draw_views(rng, 300))
        c["gaussians"] = n if order == "rows" else min(n, 700_000)
        return c
    texture = rng.random() < 0.7
    if kind == "step":
        v = _draw_views(rng, 300)
        c = _edge(precision=rng.choice(["bf16", "fp16"]), texture=texture, **v)
        if c["precision"] == "fp16":
            c["views"] = min(c["views"], 150)
        split["fraction"] = min(split["fraction"], 0.2)
        return dict(c, **split) | {"kind": "step"}
    precision, form = rng.choice([("fp32", "plain"), ("fp32", "batched"), ("fp16", "batched"), ("bf16", "batched")])
    most = {"plain": 12, "batched": 300}[form]
    px = MOST_PIXELS if precision == "bf16" else 200_000_000
    return _edge(precision=precision, form=form, texture=texture, polygons=rng.choice([12, 60]),
                 halves=rng.random() < 0.2, **_draw_views(rng, most, px))


# ----------------------------------------------------------------- inputs

def _sizes(case):
    """Widths, heights, byte and float offsets of the case's views."""
    rng = random.Random(case["sizes"])
    W, H = [], []
    for v in range(case["views"]):
        w = rng.randint(case["w_lo"], case["w_hi"])
        h = case["height"] or max(3, round(w / rng.uniform(*ASPECT)))
        if case["halves"] and v % 2:
            w, h = w // 2, h // 2
        W.append(w)
        H.append(h)
    W, H = np.array(W, np.int32), np.array(H, np.int32)
    px = W.astype(np.int64) * H
    ino = np.concatenate([[0], np.cumsum(-(-3 * px // 256) * 256)[:-1]]).astype(np.int64)
    outo = np.concatenate([[0], np.cumsum(-(-px // 64) * 64)[:-1]]).astype(np.int64)
    return W, H, ino, outo


def _pixels(case):
    W, H, _, _ = _sizes(case)
    return int((W.astype(np.int64) * H).sum())


def _canvas(rng, W, H, polygons, texture, dev):
    """One noise-free scene, float32 (H, W, 3)."""
    x = torch.arange(W, device=dev, dtype=torch.float32) + 0.5
    y = (torch.arange(H, device=dev, dtype=torch.float32) + 0.5)[:, None]
    c0, c1 = ([rng.uniform(0, 255) for _ in range(3)] for _ in range(2))
    th = rng.uniform(0, 2 * math.pi)
    ct, st = math.cos(th), math.sin(th)
    t = (((x - W / 2) * ct + (y - H / 2) * st) / (W * abs(ct) + H * abs(st)) + 0.5).clamp_(0, 1)
    img = torch.stack([a + (b - a) * t for a, b in zip(c0, c1)], -1)
    for k in range(polygons):
        cx, cy, R = rng.uniform(0, W), rng.uniform(0, H), rng.uniform(0.03, 0.25) * min(W, H)
        ang = sorted(rng.uniform(0, 2 * math.pi) for _ in range(rng.randint(3, 8)))
        P = [(cx + R * s * math.cos(a), cy + R * s * math.sin(a)) for a in ang for s in [rng.uniform(0.5, 1.0)]]
        colour = [rng.uniform(0, 255) for _ in range(3)]
        f, a, phi = rng.uniform(1 / 64, 1 / 8), rng.uniform(0, 2 * math.pi), rng.uniform(0, 2 * math.pi)
        xa, xb = max(0, int(min(p[0] for p in P))), min(W, int(max(p[0] for p in P)) + 1)
        ya, yb = max(0, int(min(p[1] for p in P))), min(H, int(max(p[1] for p in P)) + 1)
        if xa >= xb or ya >= yb:
            continue
        px, py = x[xa:xb], y[ya:yb]
        inside = torch.zeros((yb - ya, xb - xa), dtype=torch.bool, device=dev)
        for (x0, y0), (x1, y1) in zip(P, P[1:] + P[:1]):     # even-odd rule
            if y0 != y1:
                inside ^= ((py >= y0) != (py >= y1)) & (px < x0 + (py - y0) * ((x1 - x0) / (y1 - y0)))
        wave = 0.0
        if texture and k % 2 == 0:
            wave = 20.0 * torch.sin(2 * math.pi * f * (px * math.cos(a) + py * math.sin(a)) + phi)
        for c in range(3):
            cell = img[ya:yb, xa:xb, c]
            cell.copy_(torch.where(inside, colour[c] + wave, cell))
    return img


def _images(case, seed, dev):
    """The packed views. A case of many views crops and flips a few scenes."""
    W, H, ino, _ = _sizes(case)
    rng = random.Random(seed)
    gen = torch.Generator(device=dev).manual_seed(seed)
    buf = torch.zeros(int(ino[-1]) + 3 * int(W[-1]) * int(H[-1]) + 16, dtype=torch.uint8, device=dev)
    own = len(W) <= 2
    scenes = [] if own else [_canvas(rng, int(W.max()), int(H.max()), case["polygons"], case["texture"], dev) for _ in range(4)]
    for w, h, o in zip(W.tolist(), H.tolist(), ino.tolist()):
        if own:
            s = _canvas(rng, w, h, case["polygons"], case["texture"], dev)
        else:
            s = scenes[rng.randrange(4)]
            y0, x0 = rng.randint(0, s.shape[0] - h), rng.randint(0, s.shape[1] - w)
            s = s[y0:y0 + h, x0:x0 + w].flip([d for d in (0, 1) if rng.random() < 0.5])
        noisy = torch.randn((h, w, 3), generator=gen, device=dev).mul_(5.0).add_(s)
        buf[o:o + 3 * w * h] = noisy.round_().clamp_(0, 255).to(torch.uint8).reshape(-1)
    return buf


def _gaussians(case, seed, dev):
    """Parameters (`capacity` rows, N live), the mask of K rows to split."""
    gen = torch.Generator(device=dev).manual_seed(seed + 1)
    N = case["gaussians"]
    K = round(case["fraction"] * N)
    cap = N + K
    g = {"means": torch.rand((N, 3), generator=gen, device=dev) * 2 - 1,
         "log_scales": torch.randn((N, 3), generator=gen, device=dev) * case["ls_sd"] + case["ls_mu"],
         "quats": torch.nn.functional.normalize(torch.randn((N, 4), generator=gen, device=dev), dim=1),
         "opacity_logits": torch.logit(torch.rand(N, generator=gen, device=dev), eps=1e-6)}
    g = {k: torch.cat([v, v.new_zeros((K,) + v.shape[1:])]) for k, v in g.items()}
    mask = torch.zeros(cap, dtype=torch.uint8, device=dev)
    mask[torch.randperm(N, generator=gen, device=dev)[:K]] = 1
    moments = {}
    if case.get("features"):
        g["features"] = torch.randn((cap, case["features"]), generator=gen, device=dev)
    if case.get("record"):
        for k, v in g.items():
            moments[k] = tuple(torch.randn(v.shape, generator=gen, device=dev) for _ in range(2))
    return g, mask, moments, N, K


def _contributions(case, seed, dev):
    """Each Gaussian covers a clipped disc of radius 1..5 in one view, with
    weight a exp(-d^2 / (r^2 / 2)). "rows": the entries of a view's rows one
    after another, as a rasteriser meets them; "spread": in no order."""
    W, H, _, _ = _sizes(case)
    gen = torch.Generator(device=dev).manual_seed(seed + 2)
    N = case["gaussians"]
    tw, th = torch.from_numpy(W).to(dev), torch.from_numpy(H).to(dev)
    v = torch.randint(0, len(W), (N,), generator=gen, device=dev)
    cx = (torch.rand(N, generator=gen, device=dev) * tw[v]).int().minimum(tw[v] - 1)
    cy = (torch.rand(N, generator=gen, device=dev) * th[v]).int().minimum(th[v] - 1)
    r = torch.randint(1, 6, (N,), generator=gen, device=dev)
    a = torch.rand(N, generator=gen, device=dev) * 0.95 + 0.05
    row0 = torch.cumsum(th, 0) - th
    parts = []
    for rad in range(1, 6):
        off = [(dx, dy) for dy in range(-rad, rad + 1) for dx in range(-rad, rad + 1) if dx * dx + dy * dy <= rad * rad]
        dx, dy = torch.tensor(off, dtype=torch.int32, device=dev).T
        g = (r == rad).nonzero()
        x, y = cx[g] + dx, cy[g] + dy
        ok = (x >= 0) & (y >= 0) & (x < tw[v[g]]) & (y < th[v[g]])
        w = a[g] * torch.exp((dx * dx + dy * dy) * (-2.0 / (rad * rad)))
        parts.append([t.expand_as(ok)[ok] for t in (g.int(), v[g].int(), y * tw[v[g]] + x, w, (row0[v[g]] + y).int())])
    g, view, pixel, weight, row = (torch.cat(t) for t in zip(*parts))
    del parts
    if case["order"] == "rows":
        # rows in order, inside a row by Gaussian, left to right
        at = torch.argsort(row.long() * N + g, stable=True)
    else:
        at = torch.randperm(g.numel(), generator=gen, device=dev)
    return [t[at].contiguous() for t in (g, view, pixel, weight)]


def _mask_inputs(case, seed, dev):
    W, H, _, outo = _sizes(case)
    gen = torch.Generator(device=dev).manual_seed(seed + 3)
    n = int(outo[-1]) + int(W[-1]) * int(H[-1])
    # maps as the edge pass leaves them: a third of the pixels survive, their
    # values spread around the median 1
    maps = torch.empty(n, device=dev)
    for i in range(0, n, 1 << 26):
        m = maps[i:i + (1 << 26)]
        m.normal_(generator=gen).mul_(0.8).exp_()
        m *= torch.rand(m.shape, generator=gen, device=dev) < 1 / 3
    N = case["gaussians"]
    grad = torch.randn(N, generator=gen, device=dev).sub_(9.0).exp_()
    return maps, grad, _contributions(case, seed, dev)


# ----------------------------------------------------------------- prepare, run

class _State:
    pass


def _counts(N, dev):
    return torch.tensor([N], dtype=torch.int64, device=dev)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    s = _State()
    s.kind, s.case = case["kind"], case
    if s.kind in ("edge", "step"):
        W, H, ino, outo = s.views = _sizes(case)
        s.images = _images(case, seed, dev)
        s.maps = torch.zeros(int(outo[-1]) + int(W[-1]) * int(H[-1]), device=dev)
    if s.kind in ("las", "step"):
        s.g, s.mask, s.moments, s.N, _ = _gaussians(case, seed, dev)
        cap = s.mask.numel()
        s.features = s.g.pop("features", None)
        s.count = _counts(s.N, dev)
        s.split_idx = torch.zeros(cap, dtype=torch.int32, device=dev)
        s.status = torch.zeros(1, dtype=torch.int32, device=dev)
    if s.kind == "step":
        s.step = igsp.Step(s.images, s.views, s.maps, dict(s.g, count=s.count), s.mask, s.split_idx, s.status,
                           precision=case["precision"])
    if s.kind == "mask":
        s.views = _sizes(case)
        s.maps, s.grad, s.contributions = _mask_inputs(case, seed, dev)
        N = case["gaussians"]
        s.count = _counts(N, dev)
        s.mask = torch.zeros(N, dtype=torch.uint8, device=dev)
        s.scores = torch.zeros(N, dtype=torch.int64, device=dev)
        s.selected = torch.zeros(1, dtype=torch.int64, device=dev)
        s.budget = N + round(case["room"] * N)
    return s


def run(s):
    if s.kind == "edge":
        igsp.edge_importance(s.images, s.views, s.maps, precision=s.case["precision"], batched=s.case["form"] != "plain")
        return {"maps": s.maps}
    if s.kind == "mask":
        igsp.split_mask(s.maps, s.views, *s.contributions, s.grad, s.count, s.mask, s.scores,
                        grad_threshold=GRAD_THRESHOLD, warmup=s.case["warmup"], budget=s.budget, n_selected=s.selected)
        return {"mask": s.mask, "scores": s.scores, "selected": s.selected}
    s.count.fill_(s.N)   # a trainer prunes between two splits: the live count falls again
    out = dict(s.g, count=s.count, split_idx=s.split_idx, status=s.status)
    if s.kind == "step":
        s.step.launch()
        return dict(out, maps=s.maps)
    args = (s.g["means"], s.g["log_scales"], s.g["quats"], s.g["opacity_logits"], s.count, s.mask, s.split_idx, s.status)
    if s.case["record"]:
        igsp.long_axis_split_full(*args, s.moments, features=s.features)
        out["moments"] = s.moments
    else:
        igsp.long_axis_split(*args, features=s.features)
    return out if s.features is None else dict(out, features=s.features)


def work(case):
    px = _pixels(case) if "views" in case else 0
    b = 0
    if case["kind"] in ("edge", "step"):
        b += 7 * px                                      # RGB in, float32 map out
    if case["kind"] in ("las", "step"):
        N, K, F = case["gaussians"], round(case["fraction"] * case["gaussians"]), case["features"] if "features" in case else 0
        b += N + K * (44 + 28 + 44 + 4 + 8 * F)          # mask; the row read, both children and the index written
        if case.get("record"):
            b += K * 2 * 2 * 4 * (11 + F)                # both moments of both children
    if case["kind"] == "mask":
        N = case["gaussians"]
        n = 35 * N                                       # mean entries of a disc, nearly none clipped
        b += 16 * n + 4 * min(px, n) + N * (4 + 8 + 1)
    return {"bytes": b, "flops": 0}


# ----------------------------------------------------------------- exact

def _reflect(n, k, dev):
    i = torch.arange(-k, n + k, device=dev).abs()
    return torch.where(i >= n, 2 * (n - 1) - i, i).abs()


def _taps(t, weights, dim):
    """Correlation along `dim` with reflect-101 borders."""
    k = len(weights) // 2
    n = t.shape[dim]
    p = t.index_select(dim, _reflect(n, k, t.device))
    return sum(w * p.narrow(dim, i, n) for i, w in enumerate(weights) if w)


def _exact_map(rgb):
    """float64 map of one view (H, W, 3): integers up to the squared
    magnitude, then float64."""
    rgb = rgb.to(torch.int64)
    g = 299 * rgb[..., 0] + 587 * rgb[..., 1] + 114 * rgb[..., 2]
    b = _taps(_taps(g, (1, 4, 6, 4, 1), 1), (1, 4, 6, 4, 1), 0)
    gx = _taps(_taps(b, (-1, 0, 1), 1), (1, 2, 1), 0)
    gy = _taps(_taps(b, (1, 2, 1), 1), (-1, 0, 1), 0)
    M = gx * gx + gy * gy
    H, W = M.shape
    P = M.index_select(0, _reflect(H, 1, M.device)).index_select(1, _reflect(W, 1, M.device))
    at = lambda dy, dx: P[1 + dy:1 + dy + H, 1 + dx:1 + dx + W]  # noqa: E731
    ax, ay = gx.abs().double(), gy.abs().double()
    tan = math.sqrt(2.0) - 1.0
    horizontal, vertical, same = ay < tan * ax, ax < tan * ay, (gx >= 0) == (gy >= 0)
    pick = lambda h, v, d, e: torch.where(horizontal, h, torch.where(vertical, v, torch.where(same, d, e)))  # noqa: E731
    A = pick(at(0, -1), at(-1, 0), at(-1, -1), at(1, -1))
    B = pick(at(0, 1), at(1, 0), at(1, 1), at(-1, 1))
    back = torch.where(vertical, gy, gx) < 0
    S, T = torch.where(back, B, A), torch.where(back, A, B)
    keep = (M > S) & (M >= T) & (M > 0)
    m = M.double().sqrt_()
    kept = m[keep]
    if not kept.numel():
        return torch.zeros_like(m)
    return torch.where(keep, m / kept.sort().values[(kept.numel() - 1) // 2], 0.0)


def _exact_edge(case, seed, dev):
    W, H, ino, outo = _sizes(case)
    images = _images(case, seed, dev)
    maps = torch.zeros(int(outo[-1]) + int(W[-1]) * int(H[-1]), dtype=torch.float64, device=dev)
    for w, h, i, o in zip(W.tolist(), H.tolist(), ino.tolist(), outo.tolist()):
        maps[o:o + w * h] = _exact_map(images[i:i + 3 * w * h].view(h, w, 3)).reshape(-1)
    return maps


def _exact_split(case, seed, dev):
    g, mask, moments, N, K = _gaussians(case, seed, dev)
    g = {k: v.double() for k, v in g.items()}
    i = mask.nonzero()[:, 0]
    s = g["log_scales"][i]
    axis = torch.argmax(s, 1, keepdim=True)
    w, x, y, z = torch.nn.functional.normalize(g["quats"][i], dim=1).unbind(1)
    R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)
    column = R.gather(2, axis[:, None, :].expand(-1, 3, 1))[..., 0]
    d = column * (ALPHA * s.gather(1, axis).exp())
    small = torch.full_like(s, math.log(GAMMA)).scatter_(1, axis, math.log(ALPHA)) + s
    o = torch.logit(BETA * torch.sigmoid(g["opacity_logits"][i]))
    mean = g["means"][i]
    for rows, m in ((i, mean + d), (slice(N, N + K), mean - d)):
        g["means"][rows], g["log_scales"][rows], g["opacity_logits"][rows] = m, small, o
    g["quats"][N:] = g["quats"][i]
    if "features" in g:
        g["features"][N:] = g["features"][i]
    for pair in moments.values():
        for t in pair:
            t[i] = 0.0
            t[N:] = 0.0
    out = dict(g, count=None, split_idx=None, status=None)
    if moments:
        out["moments"] = {k: tuple(t.double() for t in pair) for k, pair in moments.items()}
    return out


def exact(case, seed):
    dev = torch.device("cuda:0")
    if case["kind"] == "mask":
        return None                                      # whole numbers and bytes only
    out = {}
    if case["kind"] in ("las", "step"):
        out = _exact_split(case, seed, dev)
    if case["kind"] in ("edge", "step"):
        out["maps"] = _exact_edge(case, seed, dev)
    return out
