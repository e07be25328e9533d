"""The work that users of the 4D Gaussian renderer have it do, as cases that can be timed and checked.

Scenes follow the synthetic generators of this repository (uniform positions in [-1, 1]^3 and times in [0, 1],
log-normal scales, unit quaternions, normal opacity logits and 4DSH coefficients), seen by pinhole cameras on a ring
of radius 4 that look at the origin with a 60 degree field of view. `exact` renders the same inputs from the
definition in plain torch, in 64 bits.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2310_10642_amd import g4d

TILE = 16
T_CULL, NEAR = 0.05, 0.2
GROUPS = ("means4", "log_scales4", "q_left", "q_right", "opacity_logit", "coeffs")
# learning rates of the six groups, of the order that 3D Gaussian Splatting trains with
LRS = (1.6e-4, 5e-3, 1e-3, 1e-3, 5e-2, 2.5e-3)


def _case(name, kind, n, views, width, height, sh=3, fourier=2, **more):
    """kind: render | noalloc | step | fused | autograd | adam. log_t: mean log time-scale (how long primitives
    live); mixed: every other view is 800x800; loss: l1 | l2; densify: densification statistics are on."""
    c = dict(name=name, kind=kind, n=n, views=views, width=width, height=height, sh=sh, fourier=fourier,
             log_t=-3.0, mixed=False, depth=True, loss="l1", densify=False)
    c.update(more)
    return c


def listed():
    return [
        # a preview of a tiny scene: launches and latency are all there is
        _case("view_1k_64x64", "render", 1000, 1, 64, 64, sh=1, fourier=1),
        # one frame for an interactive viewer: image, depth and alpha of one (camera, time)
        _case("view_300k_1352x1014", "render", 300_000, 1, 1352, 1014),
        # a frame of a serving loop that may not allocate, at the monocular 800x800 setting
        _case("noalloc_150k_800x800", "noalloc", 150_000, 1, 800, 800, depth=False),
        # an evaluation batch: many test views of a large scene in one call, two image sizes
        _case("batch_1m_16views_mixed", "render", 1_000_000, 16, 1352, 1014, log_t=-4.0, mixed=True, depth=False),
        # a long video from four cameras in one call
        _case("sequence_3m_240views_1080p", "render", 3_000_000, 240, 1920, 1080, log_t=-5.0, depth=False),
        # a training step early in a run: few primitives, small odd images
        _case("step_5k_4views_203x151", "step", 5000, 4, 203, 151, sh=2, fourier=1, loss="l2"),
        # a training step on one view
        _case("step_300k_1view", "step", 300_000, 1, 1352, 1014),
        # the batched training step: eight (camera, time) samples
        _case("step_300k_8views", "step", 300_000, 8, 1352, 1014),
        # the same with the loss folded into the backward and the density-control statistics on
        _case("fused_500k_8views_densify", "fused", 500_000, 8, 1352, 1014, loss="l2", densify=True),
        # a step through torch autograd with depth and alpha losses, a batch of four samples
        _case("autograd_100k_4views_800x800", "autograd", 100_000, 4, 800, 800, loss="l2"),
        # the optimiser's share of a step
        _case("adam_300k", "adam", 300_000, 1, 16, 16),
        # the optimiser on an odd count of low-order primitives
        _case("adam_20001_sh1", "adam", 20_001, 1, 16, 16, sh=1, fourier=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("render", "render", "noalloc", "step", "step", "fused", "autograd", "adam"))
    sh, fourier = rng.choice(((3, 2), (3, 2), (3, 1), (2, 1), (1, 1), (0, 2), (3, 0)))
    width = _log_int(rng, 64, 1920)
    height = max(48, int(width * rng.uniform(0.55, 1.0)))
    loss, log_t = rng.choice(("l1", "l2")), rng.choice((-3.0, -4.0, -5.0))
    depth, densify = rng.random() < 0.5, rng.random() < 0.3
    c = _case("", kind, _log_int(rng, 1000, 1_000_000), _log_int(rng, 1, 24), width, height, sh, fourier,
              loss=loss, log_t=log_t, depth=depth, densify=densify)
    if kind == "noalloc":
        # within the limits of the no-allocation render: one view, and primitives x image area bounded
        c.update(n=min(c["n"], int(200_000 * min(1.0, (1352.0 / width) ** 2))), views=1)
    elif kind == "adam":
        c.update(views=1, width=16, height=16)
    elif kind != "render":
        c.update(n=min(c["n"], 500_000), views=min(c["views"], 8))
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------------ inputs ----
def _camera(theta, width, height, radius=4.0):
    """A ring camera looking at the origin, world up +y, OpenCV axes."""
    eye = np.array([radius * math.sin(theta), 0.0, radius * math.cos(theta)])
    fwd = -eye / np.linalg.norm(eye)
    right = np.cross(fwd, [0.0, 1.0, 0.0])
    right /= np.linalg.norm(right)
    rot = np.stack([right, np.cross(fwd, right), fwd])
    w2c = np.concatenate([rot, (-rot @ eye)[:, None]], 1).astype(np.float32)
    f = float(np.float32(0.5 * width / math.tan(math.radians(30.0))))
    return SimpleNamespace(width=width, height=height, fx=f, fy=f, cx=0.5 * width, cy=0.5 * height,
                           world_to_cam=w2c, center=eye.astype(np.float32))


def _coeffs(case):
    return (case["fourier"] + 1) * (case["sh"] + 1) ** 2


def _inputs(case, seed):
    """Primitives on the GPU, cameras and times on the host, all from the seed."""
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(1_000_003 * int(seed) + 17)
    n = case["n"]

    def normal(*shape, mean=0.0, std=1.0):
        return torch.randn(*shape, device=dev, generator=g).mul_(std).add_(mean)

    def uniform(*shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, device=dev, generator=g).mul_(hi - lo).add_(lo)

    means = torch.cat([uniform(n, 3, lo=-1.0), uniform(n, 1)], 1).contiguous()
    scales = torch.cat([normal(n, 3, mean=-3.0, std=0.5), normal(n, 1, mean=case["log_t"], std=0.5)], 1).contiguous()
    ql = torch.nn.functional.normalize(normal(n, 4), dim=1)
    qr = torch.nn.functional.normalize(normal(n, 4), dim=1)
    prims = [means, scales, ql, qr, normal(n), normal(n, _coeffs(case), 3, std=0.3)]
    rng = np.random.default_rng(int(seed) + 5)
    cams, times = [], []
    for v in range(case["views"]):
        small = case["mixed"] and v % 2 == 0
        w, h = (800, 800) if small else (case["width"], case["height"])
        if case["views"] > 32:  # a video: consecutive frames from four fixed cameras
            cams.append(_camera((v % 4) * math.pi / 2.0 + 0.01 * (int(seed) % 100), w, h))
            times.append(float(np.float32(0.4 + 0.2 * (v // 4) / (case["views"] / 4))))
        else:
            cams.append(_camera(rng.uniform(0.0, 2.0 * math.pi), w, h))
            times.append(float(np.float32(rng.uniform(0.05, 0.95))))
    pixels = sum(c.width * c.height for c in cams)
    target = None
    if case["kind"] in ("step", "fused", "autograd"):
        target = uniform(3 * pixels)
    return SimpleNamespace(dev=dev, prims=prims, cams=cams, times=times, pixels=pixels, target=target, normal=normal)


def _loss_scale(case, pixels):
    return 1.0 / (3 * pixels)


def prepare(case, seed):
    i = _inputs(case, seed)
    s = SimpleNamespace(case=dict(case), cams=i.cams, times=i.times, prims=i.prims, target=i.target)
    s.renderer = g4d.Renderer(case["sh"], case["fourier"], 1.0)
    kind = case["kind"]
    if kind == "adam":
        k = 17 + 3 * _coeffs(case)
        s.grads = [i.normal(*p.shape, std=1e-4) for p in i.prims]
        s.exp_avg = i.normal(case["n"] * k, std=1e-4)
        s.exp_avg_sq = i.normal(case["n"] * k, std=1e-4).square_()
        s.step = 100
        return s
    if kind == "autograd":
        s.prims = [p.requires_grad_() for p in i.prims]
        return s
    r = s.renderer
    r.set_primitives(*s.prims)
    # the buffers that a training or serving loop keeps
    s.rgb = torch.empty(3 * i.pixels, device=i.dev)
    s.planes = tuple(torch.empty(i.pixels, device=i.dev) if case["depth"] and kind in ("render", "noalloc") else None
                     for _ in range(2))
    if kind in ("step", "fused"):
        s.scale = _loss_scale(case, i.pixels)
        s.kind_code = g4d.G4D_LOSS_L2 if case["loss"] == "l2" else g4d.G4D_LOSS_L1
        s.loss = torch.zeros(1, device=i.dev)
        s.dl = torch.empty_like(s.rgb) if kind == "step" else None
        s.grads = r.grad_buffers(i.dev)
        if case["densify"]:
            n = case["n"]
            s.stats = (torch.zeros(n, device=i.dev), torch.zeros(n, device=i.dev),
                       torch.zeros(n, device=i.dev, dtype=torch.int32))
            r.set_densify_stats(*s.stats)
    return s


def run(s):
    case, r = s.case, s.renderer
    kind = case["kind"]
    if kind == "adam":
        r.adam_step(s.prims, s.grads, s.exp_avg, s.exp_avg_sq, s.step, LRS)
        s.step += 1
        return dict(zip(GROUPS, s.prims), exp_avg=s.exp_avg, exp_avg_sq=s.exp_avg_sq)
    if kind == "autograd":
        rgb, depth, alpha = g4d.render(r, s.cams, s.times, *s.prims)
        err = rgb - s.target
        err = err.square() if case["loss"] == "l2" else err.abs()
        loss = err.mean() + 0.1 * depth.mean() - 0.05 * alpha.square().mean()
        grads = torch.autograd.grad(loss, s.prims)
        return dict(zip(GROUPS, grads), rgb=rgb.detach(), depth=depth.detach(), alpha=alpha.detach(),
                    loss=loss.detach())
    if kind == "render":
        rgb, depth, alpha = r.render(s.cams, s.times, depth=case["depth"], alpha=case["depth"],
                                     out=(s.rgb, *s.planes))
        return dict(rgb=rgb, depth=depth, alpha=alpha)
    if kind == "noalloc":
        rgb, depth, alpha = r.render_noalloc(s.cams, s.times, out=(s.rgb, *s.planes))
        return dict(rgb=rgb, depth=depth, alpha=alpha)
    r.render(s.cams, s.times, depth=False, alpha=False, out=(s.rgb, None, None))
    s.loss.zero_()
    if kind == "step":
        r.image_loss(s.kind_code, s.rgb, s.target, s.scale, s.loss, s.dl)
        r.backward(s.dl, out=s.grads)
    else:
        r.backward_loss(s.kind_code, s.rgb, s.target, s.scale, s.loss, out=s.grads)
    out = dict(zip(GROUPS, s.grads), rgb=s.rgb, loss=s.loss)
    if case["densify"]:
        out.update(uv_grad=s.stats[0], t_grad=s.stats[1], blends=s.stats[2])
    return out


# -------------------------------------------------------------------------------------------------------- work ----
def work(case):
    """Bytes: parameters in, planes out, and for a step the target in and the gradients out. Operations: 16 lane
    operations for each list entry a pixel blends (27 more backward), two flops each. A pixel blends what covers it
    until it is opaque, at most about 80 entries in these scenes."""
    n, k = case["n"], 17 + 3 * _coeffs(case)
    if case["kind"] == "adam":
        return dict(bytes=7.0 * 4 * n * k, flops=14.0 * n * k)
    pixels = sum((800 * 800 if case["mixed"] and v % 2 == 0 else case["width"] * case["height"])
                 for v in range(case["views"]))
    planes = 3 + (2 if case["kind"] == "autograd" or (case["depth"] and case["kind"] in ("render", "noalloc")) else 0)
    # share of the primitives that pass the temporal filter, and entries over a pixel: sigma = exp(-3) at distance 4
    alive = min(1.0, 2.45 * 2.0 * math.exp(case["log_t"]) * 1.2)
    sigma = math.exp(-3.0) / 4.0 / (2.0 * math.tan(math.radians(30.0)))  # of the image's width
    aspect = case["width"] / case["height"]
    cover = n * alive * math.pi * (2.0 * sigma) ** 2 * aspect
    entries = pixels * min(80.0, cover)
    out = dict(bytes=4.0 * (n * k + planes * pixels), flops=2.0 * 16 * entries)
    if case["kind"] in ("step", "fused", "autograd"):
        out["bytes"] += 4.0 * (n * k + 3 * pixels)
        out["flops"] += 2.0 * 27 * entries
    return out


# ------------------------------------------------------------------------- the same from the definition, in FP64 ----
def _sh_basis(d, degree):
    """Orthonormal real spherical harmonics with the Condon-Shortley phase, index l*l + l + m, through
    K_l^m, the associated Legendre recurrence and (x + iy)^m."""
    x, y, z = d.unbind(-1)
    cols = [None] * (degree + 1) ** 2
    re, im = torch.ones_like(x), torch.zeros_like(x)
    for m in range(degree + 1):
        if m:
            re, im = re * x - im * y, re * y + im * x
        pmm = torch.full_like(z, float((-1) ** m * np.prod(np.arange(1, 2 * m, 2, dtype=np.float64))))
        prev, cur = torch.zeros_like(z), pmm
        for l in range(m, degree + 1):
            if l > m:
                prev, cur = cur, ((2 * l - 1) * z * cur - (l + m - 1) * prev) / (l - m)
            k = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - m) / math.factorial(l + m))
            if m == 0:
                cols[l * l + l] = k * cur
            else:
                cols[l * l + l + m] = math.sqrt(2.0) * k * cur * re
                cols[l * l + l - m] = math.sqrt(2.0) * k * cur * im
    return torch.stack(cols, -1)


def _left(q):
    a, b, c, d = q.unbind(-1)
    return torch.stack([torch.stack(r, -1) for r in ([a, -b, -c, -d], [b, a, -d, c], [c, d, a, -b], [d, -c, b, a])], -2)


def _right(q):
    p, q_, r, s = q.unbind(-1)
    return torch.stack([torch.stack(w, -1) for w in ([p, -q_, -r, -s], [q_, p, s, -r], [r, -s, p, q_], [s, r, -q_, p])], -2)


def _project(prims, cam, t, case):
    """One view's visible primitives: index, u, v, z, opacity * p(t), conic, colour, tile rectangle."""
    means, scales, ql, qr, logit, coeffs = prims
    m = (_left(torch.nn.functional.normalize(ql, dim=-1)) @ _right(torch.nn.functional.normalize(qr, dim=-1)))
    m = m * scales.exp().unsqueeze(-2)
    v3 = (m[:, :3] * m[:, 3:4]).sum(-1)
    s44 = m[:, 3].square().sum(-1)
    dt = t - means[:, 3]
    pt = torch.exp(-0.5 * dt * dt / s44)
    w2c = torch.from_numpy(cam.world_to_cam.astype(np.float64)).to(means.device)
    rot, trans = w2c[:, :3].contiguous(), w2c[:, 3]
    muc = means[:, :3] + v3 * (dt / s44).unsqueeze(-1)
    pc = muc @ rot.T.contiguous() + trans
    with torch.no_grad():
        idx = torch.nonzero((pt >= float(np.float32(T_CULL))) & (pc[:, 2] > float(np.float32(NEAR)))).reshape(-1)
    m, v3, s44, dt, pt, muc, pc = (x[idx] for x in (m, v3, s44, dt, pt, muc, pc))
    cov = torch.stack([(m[:, i] * m[:, j]).sum(-1) - v3[:, i] * v3[:, j] / s44 for i in range(3) for j in range(3)], -1)
    cov = cov.reshape(-1, 3, 3)
    fx, fy = float(np.float32(cam.fx)), float(np.float32(cam.fy))
    iz = 1.0 / pc[:, 2]
    u, v = fx * pc[:, 0] * iz + cam.cx, fy * pc[:, 1] * iz + cam.cy
    lx, ly = 1.3 * 0.5 * cam.width / fx, 1.3 * 0.5 * cam.height / fy
    xi, eta = (pc[:, 0] * iz).clamp(-lx, lx), (pc[:, 1] * iz).clamp(-ly, ly)
    j0 = fx * iz.unsqueeze(-1) * (rot[0] - xi.unsqueeze(-1) * rot[2])
    j1 = fy * iz.unsqueeze(-1) * (rot[1] - eta.unsqueeze(-1) * rot[2])
    c0, c1 = (cov * j0.unsqueeze(-2)).sum(-1), (cov * j1.unsqueeze(-2)).sum(-1)
    a2, b2, c2 = (c0 * j0).sum(-1) + 0.3, (c0 * j1).sum(-1), (c1 * j1).sum(-1) + 0.3
    det = a2 * c2 - b2 * b2
    op = torch.sigmoid(logit[idx]) * pt
    with torch.no_grad():
        mid = 0.5 * (a2 + c2)
        rad = torch.ceil(3.0 * torch.sqrt(mid + torch.sqrt((mid * mid - det).clamp_min(0.0))))
        # no pixel outside the box of the 1/255 ellipse can count, so the lists leave its tiles out
        reach = (2.0 * torch.log(255.0 * op).clamp_min(0.0))
        hx, hy = torch.sqrt(reach * a2) + 0.01, torch.sqrt(reach * c2) + 0.01
        tx, ty = (cam.width + TILE - 1) // TILE, (cam.height + TILE - 1) // TILE

        def span(c, h, n):
            lo = torch.maximum(torch.floor((c - rad) / TILE), torch.floor((c - h) / TILE)).clamp(0, n)
            hi = torch.minimum(torch.floor((c + rad) / TILE), torch.floor((c + h) / TILE)).add(1).clamp(0, n)
            return lo.long(), hi.long()

        x0, x1 = span(u, hx, tx)
        y0, y1 = span(v, hy, ty)
        keep = torch.nonzero((x1 > x0) & (y1 > y0) & (op >= 0.999 / 255.0) & (det > 0)).reshape(-1)
        # front to back by the camera-space z as the records hold it, ties by index
        keep = keep[torch.sort(pc[keep, 2].float(), stable=True).indices]
    rel = muc - torch.from_numpy(cam.center.astype(np.float64)).to(means.device)
    basis = _sh_basis(torch.nn.functional.normalize(rel[keep], dim=-1), case["sh"])
    ang = 2.0 * math.pi * dt[keep]
    z4 = torch.cat([torch.cos(n * ang).unsqueeze(-1) * basis for n in range(case["fourier"] + 1)], -1)
    colour = ((z4.unsqueeze(-1) * coeffs[idx[keep]]).sum(1) + 0.5).clamp_min(0.0)
    q = 1.0 / det
    rec = torch.stack([x[keep] for x in (u, v, pc[:, 2], op, c2 * q, -b2 * q, a2 * q)] + list(colour.unbind(-1)), -1)
    return idx[keep], rec, (x0[keep], x1[keep], y0[keep], y1[keep], tx, ty)


def _tile_lists(rect):
    """(record of each instance ordered by (tile, depth), first instance of each tile)."""
    x0, x1, y0, y1, tx, ty = rect
    w = x1 - x0
    count = w * (y1 - y0)
    rec = torch.repeat_interleave(torch.arange(len(count), device=count.device), count)
    k = torch.arange(len(rec), device=rec.device) - (torch.cumsum(count, 0) - count)[rec]
    tile = (y0[rec] + k // w[rec]) * tx + x0[rec] + k % w[rec]
    order = torch.sort(tile.int(), stable=True).indices
    start = torch.zeros(tx * ty + 1, dtype=torch.long, device=rec.device)
    start[1:] = torch.cumsum(torch.bincount(tile, minlength=tx * ty), 0)
    return rec[order], start


def _blend(rec, lists, start, length, tiles, tx, trans=None):
    """Blends entries [start, start + length) of `tiles` over their pixels: per pixel sums of w (r, g, b, z), the
    transmittance after them, the weights and the record of each entry."""
    at = start.unsqueeze(1) + torch.arange(int(length.max()), device=start.device).unsqueeze(0)
    live = torch.arange(at.shape[1], device=start.device).unsqueeze(0) < length.unsqueeze(1)
    ids = torch.where(live, lists[at.clamp_max(len(lists) - 1)], torch.zeros_like(at))
    e = rec[ids]  # [tiles, entries, 10]
    p = torch.arange(TILE * TILE, device=start.device)
    px = ((tiles % tx) * TILE).unsqueeze(1) + (p % TILE) + 0.5
    py = (torch.div(tiles, tx, rounding_mode="floor") * TILE).unsqueeze(1) + torch.div(p, TILE, rounding_mode="floor") + 0.5
    dx = px.unsqueeze(1) - e[..., 0:1]
    dy = py.unsqueeze(1) - e[..., 1:2]
    raw = e[..., 3:4] * torch.exp(-0.5 * (e[..., 4:5] * dx * dx + e[..., 6:7] * dy * dy) - e[..., 5:6] * dx * dy)
    a = torch.where((raw >= 1.0 / 255.0) & live.unsqueeze(-1), raw.clamp_max(0.99), torch.zeros_like(raw))
    after = torch.cumsum(torch.log1p(-a), 1)
    if trans is not None:
        after = after + torch.log(trans).unsqueeze(1)
    after = torch.exp(after)
    go = after.detach() >= 1e-4
    w = torch.where(go, a * after / (1.0 - a), torch.zeros_like(a))
    sums = torch.stack([(w * e[..., c:c + 1]).sum(1) for c in (7, 8, 9, 2)], 1)
    last = torch.where(go, after, torch.full_like(after, 2.0)).amin(1) if after.shape[1] else None
    first = trans if trans is not None else torch.ones_like(last)
    return sums, torch.where(go[:, 0], last, first), w, ids, go.all(1)


def _chunks(length, per=24_000_000):
    """Groups of tiles of like list length, bounded in (entries x pixels)."""
    order = torch.sort(length, descending=True).indices
    lens = length[order].tolist()
    i = 0
    while i < len(lens) and lens[i] > 0:
        k = max(1, per // (lens[i] * TILE * TILE))
        yield order[i:i + k][: sum(1 for x in lens[i:i + k] if x > 0)]
        i += k


def _forward_view(rec, rect, cam):
    """Planes [4, tiles, 256] (r, g, b, depth), final transmittance, and each tile's list length up to saturation."""
    lists, start = _tile_lists(rect)
    tx, ty = rect[4], rect[5]
    n_tiles = tx * ty
    planes = torch.zeros(n_tiles, 4, TILE * TILE, dtype=torch.float64, device=rec.device)
    trans = torch.ones(n_tiles, TILE * TILE, dtype=torch.float64, device=rec.device)
    stopped = torch.zeros(n_tiles, TILE * TILE, dtype=torch.bool, device=rec.device)
    used = torch.zeros(n_tiles, dtype=torch.long, device=rec.device)
    total = start[1:] - start[:-1]
    seg = 64
    while True:
        left = torch.where(stopped.all(1), torch.zeros_like(total), (total - used).clamp(0, seg))
        if not bool((left > 0).any()):
            break
        for tiles in _chunks(left, 64_000_000):
            sums, tr, _, _, go = _blend(rec, lists, start[tiles] + used[tiles], left[tiles], tiles, tx, trans[tiles])
            on = ~stopped[tiles]
            planes[tiles] += sums * on.unsqueeze(1)
            trans[tiles] = torch.where(on, tr, trans[tiles])
            stopped[tiles] |= ~go
        used += left
    return planes, trans, used, lists, start


def _to_image(tiled, cam, tx, ty):
    """[tiles, c, 256] -> flat [c * H * W]."""
    c = tiled.shape[1]
    im = tiled.reshape(ty, tx, c, TILE, TILE).permute(2, 0, 3, 1, 4).reshape(c, ty * TILE, tx * TILE)
    return im[:, :cam.height, :cam.width].reshape(-1)


def _to_tiles(flat, c, cam, tx, ty):
    im = torch.zeros(c, ty * TILE, tx * TILE, dtype=torch.float64, device=flat.device)
    im[:, :cam.height, :cam.width] = flat.reshape(c, cam.height, cam.width).double()
    return im.reshape(c, ty, TILE, tx, TILE).permute(1, 3, 0, 2, 4).reshape(ty * tx, c, TILE * TILE)


def exact(case, seed):
    i = _inputs(case, seed)
    if case["kind"] == "adam":
        k = 17 + 3 * _coeffs(case)
        grads = [i.normal(*p.shape, std=1e-4).double() for p in i.prims]
        m0 = i.normal(case["n"] * k, std=1e-4).double()
        v0 = i.normal(case["n"] * k, std=1e-4).square_().double()
        g = torch.cat([x.reshape(-1) for x in grads])
        b1, b2, eps = (float(np.float32(x)) for x in (0.9, 0.999, 1e-15))
        m1, v1 = b1 * m0 + (1 - b1) * g, b2 * v0 + (1 - b2) * g * g
        upd = (m1 / (1 - b1 ** 100)) / ((v1 / (1 - b2 ** 100)).sqrt() + eps)
        parts = torch.split(upd, [p.numel() for p in i.prims])
        new = [p.double() - float(np.float32(lr)) * u.view_as(p) for p, lr, u in zip(i.prims, LRS, parts)]
        return dict(zip(GROUPS, new), exp_avg=m1, exp_avg_sq=v1)
    step = case["kind"] in ("step", "fused", "autograd")
    # larger ones would take over about twenty seconds
    if i.pixels > (13_000_000 if step else 18_000_000) or case["n"] * case["views"] > 20_000_000:
        return None
    prims = [p.detach().double().requires_grad_(step) for p in i.prims]
    images, depths, alphas, loss = [], [], [], 0.0
    grads = [torch.zeros_like(p) for p in prims]
    uv, tg = torch.zeros(case["n"], dtype=torch.float64, device=i.dev), torch.zeros(case["n"], dtype=torch.float64, device=i.dev)
    scale, o3 = _loss_scale(case, i.pixels), 0
    for cam, t in zip(i.cams, i.times):
        hw = cam.width * cam.height
        ids, rec, rect = _project(prims, cam, t, case)
        tx, ty = rect[4], rect[5]
        with torch.no_grad():
            planes, trans, used, lists, start = _forward_view(rec.detach(), rect, cam)
            img = _to_image(planes[:, :3], cam, tx, ty)
            images.append(img)
            depths.append(_to_image(planes[:, 3:], cam, tx, ty))
            alphas.append(1.0 - _to_image(trans.unsqueeze(1), cam, tx, ty))
        if not step:
            continue
        err = img - i.target[o3:o3 + 3 * hw].double()
        o3 += 3 * hw
        loss += float((err.square() if case["loss"] == "l2" else err.abs()).sum()) * scale
        dl = scale * (2.0 * err if case["loss"] == "l2" else torch.sign(err))
        dl = _to_tiles(dl, 3, cam, tx, ty)
        dd = da = None
        if case["kind"] == "autograd":
            loss += (0.1 * float(depths[-1].sum()) - 0.05 * float(alphas[-1].square().sum())) / i.pixels
            dd = _to_tiles(torch.full((hw,), 0.1 / i.pixels, device=i.dev, dtype=torch.float64), 1, cam, tx, ty)
            da = _to_tiles(-0.1 / i.pixels * alphas[-1], 1, cam, tx, ty)
        grec = torch.zeros_like(rec)
        for tiles in _chunks(used):
            leaf = rec.detach().requires_grad_()
            sums, tr, _, _, _ = _blend(leaf, lists, start[tiles], used[tiles], tiles, tx)
            part = (sums[:, :3] * dl[tiles]).sum()
            if dd is not None:
                part = part + (sums[:, 3] * dd[tiles, 0]).sum() - (tr * da[tiles, 0]).sum()
            grec += torch.autograd.grad(part, leaf)[0]
        if case["densify"]:
            uv[ids] += grec[:, :2].norm(dim=1)
        for k, gk in enumerate(torch.autograd.grad(rec, prims, grec, allow_unused=True)):
            if gk is not None:
                grads[k] += gk
                if k == 0 and case["densify"]:
                    tg += gk[:, 3].abs()
        del grec, rec
    out = dict(rgb=torch.cat(images))
    if not step:
        return dict(out, depth=torch.cat(depths) if case["depth"] else None,
                    alpha=torch.cat(alphas) if case["depth"] else None)
    out.update(zip(GROUPS, grads))
    if case["kind"] == "autograd":
        return dict(out, depth=torch.cat(depths), alpha=torch.cat(alphas),
                    loss=torch.tensor(loss, dtype=torch.float64))
    out["loss"] = torch.tensor([loss], dtype=torch.float64)
    if case["densify"]:
        out.update(uv_grad=uv, t_grad=tg, blends=None)
    return out
