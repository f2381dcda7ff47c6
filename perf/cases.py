"""Performance cases: what a program that trains or renders ray-traced Gaussians has the library do.

A case names the calls ("do"), the scene and the options:

  map       gart_bounds and gart_build_tile_map (pre-processing of a view)
  render    map, then gart_forward (a view is shown)
  backward  gart_backward alone, on a frame whose forward has run
  step      map, forward, backward: one differentiable render, gradients of every parameter group
  train     Trainer.step: the same with an L1 loss and Adam, over four orbit views

Scenes have the distributions of paper_2608_17298_amd/scenes.py at any size and are drawn on the GPU from the
seed: "ball" (a foreground ball and a far shell: the 1m and 4m workloads; splats shrink as their number grows,
as in trained scenes), "clusters" (the small workload), "cube" (tiny), "large" (stress: large translucent
splats, hundreds of hits a ray).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_17298_amd import gart
from paper_2608_17298_amd.scenes import orbit_camera, pinhole_camera
from paper_2608_17298_amd.train import DEFAULT_LR, GROUPS, Trainer

ALPHA_MIN = float(np.float32(1.0 / 255.0))
T_MIN = float(np.float32(1e-4))
VIEWS = 4


def _case(name, do, scene, n, sh_degree, width, height, tile=8, mode="gather", precision="full"):
    return dict(name=name, do=do, scene=scene, n=n, sh_degree=sh_degree, width=width, height=height, tile=tile,
                mode=mode, precision=precision)


def listed():
    return [
        # a preview of a few splats: launches and latency count
        _case("render-preview", "render", "cube", 1500, 1, 77, 53),
        # the smallest training step: the tiny workload with its 16x16 tiles
        _case("step-tiny", "step", "cube", 4096, 0, 128, 128, tile=16),
        # an object-sized capture at VGA: the small workload
        _case("step-small", "step", "clusters", 100_000, 3, 640, 480),
        # the 1m workload: a view is shown, differentiated, and its backward alone
        _case("render-1m", "render", "ball", 1_000_000, 3, 1237, 822),
        _case("step-1m", "step", "ball", 1_000_000, 3, 1237, 822),
        _case("backward-1m", "backward", "ball", 1_000_000, 3, 1237, 822),
        # the 4m workload: pre-processing of a view, and the whole step
        _case("map-4m", "map", "ball", 4_000_000, 3, 1600, 1060),
        _case("step-4m", "step", "ball", 4_000_000, 3, 1600, 1060),
        # early training, large translucent splats: long tile lists, hundreds of hits a ray
        _case("step-large", "step", "large", 150_000, 3, 1024, 680),
        # the memory-saving variants: T-only buffer, and 8-byte entries on 16x16 tiles with lower SH degrees
        _case("step-hybrid", "step", "ball", 333_000, 2, 1001, 667, mode="hybrid"),
        _case("step-fixed16", "step", "ball", 250_000, 1, 979, 546, tile=16, precision="fixed16"),
        # a training iteration of a quarter-resolution capture
        _case("train-250k", "train", "ball", 250_000, 3, 979, 546),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["map", "render", "backward", "step", "step", "step", "train"])
    scene = rng.choice(["ball", "ball", "ball", "clusters", "cube", "large"])
    n = _log(rng, *dict(ball=(20_000, 4_000_000), clusters=(5_000, 400_000), cube=(1000, 20_000),
                        large=(10_000, 120_000))[scene])
    width = _log(rng, 64, 400) if scene == "cube" else _log(rng, 240, 1600)
    height = min(max(int(width * rng.uniform(0.5, 0.9)), 40), 1060)
    mode, precision = "gather", "full"
    if do in ("backward", "step"):
        mode = rng.choice(["gather", "gather", "gather", "hybrid"])
        precision = rng.choice(["full", "full", "half", "fixed16"])
    tile = rng.choice([8, 8, 8, 16])
    c = _case("", do, scene, n, rng.randint(0, 3), width, height, tile, mode, precision)
    del c["name"]
    return c


# ---- inputs ----------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(260817298 + int(seed))
    return g


def _sphere(gen, n):
    v = torch.randn((n, 3), device="cuda", generator=gen)
    return v / v.norm(dim=1, keepdim=True)


def _params(case, gen):
    n, k, scene = case["n"], (case["sh_degree"] + 1) ** 2, case["scene"]
    rand = lambda *s: torch.rand(s, device="cuda", generator=gen)  # noqa: E731
    randn = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    if scene == "ball":
        scale = math.log2(n / 1e6)
        fg = int(round((0.7 if n <= 2_000_000 else 0.6) * n))
        means = torch.cat([_sphere(gen, fg) * (2.0 * rand(fg, 1) ** (1 / 3)), _sphere(gen, n - fg) * 20.0])
        ls = (randn(n, 3) * 0.7 - (4.5 + 0.25 * scale)).clamp_max(-1.0)
        logit = (-0.5, 2.0)
    elif scene == "clusters":
        centre = _sphere(gen, 64) * (3.0 * rand(64, 1) ** (1 / 3))
        means = centre[torch.randint(0, 64, (n,), device="cuda", generator=gen)] + 0.3 * randn(n, 3)
        ls, logit = randn(n, 3) * 0.5 - 4.0, (0.0, 1.5)
    elif scene == "cube":
        means = rand(n, 3) * 2.0 - 1.0
        ls, logit = randn(n, 3) * 0.3 - 3.5, (0.0, 1.0)
    else:
        means = rand(n, 3) * 4.0 - 2.0
        ls, logit = randn(n, 3) * 0.3 - 2.0, (-3.0, 0.5)
    sh = 0.05 * randn(n, k, 3)
    sh[:, 0, :] = (rand(n, 3) - 0.5) * (2.0 * math.sqrt(math.pi))
    return dict(means=means, log_scales=ls, quats=randn(n, 4), opacity_logits=randn(n) * logit[1] + logit[0], sh=sh)


def _photo(case, gen):
    """A target image: smooth colours with some grain."""
    h, w = case["height"], case["width"]
    low = torch.rand((1, 3, 9, 12), device="cuda", generator=gen)
    img = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear", align_corners=True)[0].permute(1, 2, 0)
    return (img + 0.02 * torch.randn((h, w, 3), device="cuda", generator=gen)).clamp(0, 1).contiguous()


def _inputs(case, seed):
    gen = _gen(seed)
    p = _params(case, gen)
    dl = torch.where(torch.rand((case["height"], case["width"], 3), device="cuda", generator=gen) < 0.5, -1.0, 1.0)
    photos = [_photo(case, gen) for _ in range(VIEWS)] if case["do"] == "train" else None
    return p, dl, photos  # dl: the +-1 upstream gradient of an L1 loss


def _cameras(case):
    if case["do"] == "train":
        return [orbit_camera(case["width"], case["height"], 360.0 * k / VIEWS) for k in range(VIEWS)]
    return [pinhole_camera(case["width"], case["height"])]


class _HostScene:
    """What Trainer takes: the parameters as host arrays."""

    def __init__(self, case, p):
        self.sh_degree, self.tile = case["sh_degree"], case["tile"]
        for k, v in p.items():
            setattr(self, k, v.cpu().numpy())


def prepare(case, seed):
    p, dl, photos = _inputs(case, seed)
    cams = _cameras(case)
    if case["do"] == "train":
        tr = Trainer(_HostScene(case, p), cams, photos, tile=case["tile"])
        # a training program's frame has grown to its largest view
        for c in tr.cams:
            tr.frame = gart.prepare(tr.g, c, tr.settings, tr.frame, slack=1.25)
        return dict(do="train", trainer=tr)
    g = gart.Gaussians(p["means"], p["log_scales"], p["quats"], p["opacity_logits"], p["sh"], case["sh_degree"])
    cam = gart.make_camera(cams[0])
    st = gart.make_settings(case["tile"], case["mode"], lt_precision=case["precision"])
    frame = gart.prepare(g, cam, st)
    if case["do"] == "map":  # lists of a round length, zero past the view's pairs: scenes of other seeds fit too
        frame.grow(0, 1 << math.ceil(math.log2(1.05 * frame.pair_count + 64)))
        for t in (frame.pair_tile, frame.pair_prim, frame.pair_key):
            t.zero_()
    image = torch.empty((cam.height, cam.width, 3), dtype=torch.float32, device="cuda")
    s = dict(do=case["do"], g=g, cam=cam, st=st, frame=frame, image=image, dl=dl)
    if case["do"] in ("backward", "step"):
        s["grads"] = gart.empty_grads(g)
    if case["do"] == "backward":
        gart.gart_forward(g, cam, st, frame, image)
    return s


def run(s):
    if s["do"] == "train":
        tr = s["trainer"]
        loss = tr.step(tr.t % VIEWS)
        return dict(loss=loss, image=tr.image, grads=tr.grads, params={k: tr.param(k) for k in GROUPS})
    g, cam, st, f = s["g"], s["cam"], s["st"], s["frame"]
    if s["do"] != "backward":
        gart.prepare(g, cam, st, f)
    if s["do"] == "map":
        n = g.n
        return dict(rect=f.rect[:n], lt_offset=f.lt_offset[:n + 1], tile_count=f.tile_count[:n],
                    pair_offset=f.pair_offset[:n + 1], pair_tile=f.pair_tile, pair_prim=f.pair_prim,
                    pair_key=f.pair_key, tile_range=f.tile_range)
    if s["do"] != "backward":
        gart.gart_forward(g, cam, st, f, s["image"])
    if s["do"] == "render":
        return dict(image=s["image"])
    gart.gart_backward(g, cam, st, f, s["dl"], s["grads"])
    return dict(image=s["image"], grads=s["grads"])


# ---- what a pass cannot do without -------------------------------------------
# composited hits a pixel and (tile, splat) pairs a splat at the workloads' sizes
HITS_PER_PIXEL = dict(ball=39.0, clusters=42.0, cube=6.0, large=300.0)
PAIRS_PER_SPLAT = dict(ball=7.0, clusters=8.0, cube=5.0, large=250.0)


def work(case):
    n, pix, k = case["n"], case["width"] * case["height"], (case["sh_degree"] + 1) ** 2
    params = 4 * (11 + 3 * k) * n
    hits = HITS_PER_PIXEL[case["scene"]] * pix
    pairs = PAIRS_PER_SPLAT[case["scene"]] * n
    fwd, bwd = 6 * k + 60, 12 * k + 120  # flops a hit
    do = case["do"]
    if do == "map":  # parameters in; rectangles, offsets, counts and the pair lists out
        return dict(bytes=params + (16 + 8 + 4 + 8) * n + 12 * pairs, flops=300 * n + 60 * pairs)
    if do == "render":
        return dict(bytes=params + 12 * pix, flops=300 * n + fwd * hits)
    entry = {"full": 16, "half": 8, "fixed16": 8}[case["precision"]]
    entry = entry // 4 if case["mode"] == "hybrid" else entry
    if do == "backward":  # parameters, entries, upstream gradient in; gradients out
        return dict(bytes=2 * params + entry * hits + 12 * pix, flops=200 * n + bwd * hits)
    step = dict(bytes=2 * params + 24 * pix, flops=500 * n + (fwd + bwd) * hits)
    if do == "train":  # Adam: moments in and out, parameters out
        step = dict(bytes=step["bytes"] + 5 * params + 12 * pix, flops=step["flops"] + 15 * params / 4)
    return step


def tolerance(case):
    if case["do"] == "map":
        return "exact"
    if case["do"] == "render":
        return {"rel": 3e-7}  # against exact(): 4e-8 to 8e-8
    # Gradients are 32-bit sums of up to thousands of hits, 1e-7 to 3e-7 from exact(); a colour within rounding of
    # its clamp at zero may fall on either side of it, which moves the whole of its SH gradients (1.3e-4 seen).
    if case["precision"] == "full":
        return {"rel": 5e-4}
    # stored values on the edge of a code may round either way; from exact(): fp16 entries up to 1.5e-3, fixed up to 3e-4
    return {"rel": 4e-3 if case["precision"] == "half" else 1e-3}


# ---- the same in 64 bits ------------------------------------------------------
Y0 = 0.5 / math.sqrt(math.pi)


def _sh_basis(d, k):
    """Real spherical harmonics without Condon-Shortley phase at unit directions d, index l*l + l + m."""
    x, y, z = d.unbind(-1)
    b = [torch.full_like(x, Y0)]
    if k > 1:
        c = math.sqrt(3 / (4 * math.pi))
        b += [c * y, c * z, c * x]
    if k > 4:
        c = math.sqrt(15 / math.pi)
        b += [c / 2 * x * y, c / 2 * y * z, math.sqrt(5 / math.pi) / 4 * (3 * z * z - 1), c / 2 * x * z,
              c / 4 * (x * x - y * y)]
    if k > 9:
        a, c, e = math.sqrt(35 / (2 * math.pi)) / 4, math.sqrt(105 / math.pi), math.sqrt(21 / (2 * math.pi)) / 4
        b += [a * y * (3 * x * x - y * y), c / 2 * x * y * z, e * y * (5 * z * z - 1),
              math.sqrt(7 / math.pi) / 4 * z * (5 * z * z - 3), e * x * (5 * z * z - 1), c / 4 * z * (x * x - y * y),
              a * x * (x * x - 3 * y * y)]
    return torch.stack(b, -1)


def _whiten(p, o):
    """World to unit-ball map W = S^-1 R^T, o_g = W (o - mean), opacity, of parameters p."""
    w, x, y, z = (p["quats"] / p["quats"].norm(dim=1, keepdim=True)).unbind(-1)
    r = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).view(-1, 3, 3)
    wm = r.transpose(1, 2) * torch.exp(-p["log_scales"])[:, :, None]
    og = (wm @ (o - p["means"])[:, :, None])[:, :, 0]
    return wm, og, torch.sigmoid(p["opacity_logits"])


def _render64(p, cam, dl, block=64):
    """Image and, with an upstream gradient dl (or a function of the image), gradients, in float64: the image is
    taken block by block; in a block every ray meets every splat whose bounding ball can reach it."""
    W, H = cam.width, cam.height
    dev = p["means"].device
    Rm = torch.tensor(np.asarray(cam.R, np.float64), device=dev)
    t = torch.tensor(np.asarray(cam.t, np.float64), device=dev)
    o = -Rm.T @ t
    k = p["sh"].shape[1]
    with torch.no_grad():
        sig = torch.sigmoid(p["opacity_logits"])
        d2c = 2 * torch.log(sig / ALPHA_MIN)
        live = sig > ALPHA_MIN
        rad = torch.where(live, d2c.clamp_min(0).sqrt() * torch.exp(p["log_scales"]).amax(1), 0.0) * (1 + 1e-9)
        c = p["means"] @ Rm.T + t
        near = c[:, 2] - rad < 1e-3  # reaches the eye plane: kept for every block
        zn, zf = (c[:, 2] - rad).clamp_min(1e-3), c[:, 2] + rad
        lo, hi = [], []
        for ax, f, cc in ((0, cam.fx, cam.cx), (1, cam.fy, cam.cy)):
            a, b = c[:, ax] - rad, c[:, ax] + rad
            lo.append(torch.where(near, -1e30, f * torch.minimum(a / zn, a / zf) + cc - 1))
            hi.append(torch.where(near, 1e30, f * torch.maximum(b / zn, b / zf) + cc + 1))
        live &= zf > 0
    image = torch.zeros((H, W, 3), dtype=torch.float64, device=dev)
    grads = {q: torch.zeros_like(v) for q, v in p.items()} if dl is not None else None
    for by in range(0, H, block):
        for bx in range(0, W, block):
            ex, ey = min(W, bx + block), min(H, by + block)
            sel = (live & (lo[0] <= ex) & (hi[0] >= bx) & (lo[1] <= ey) & (hi[1] >= by)).nonzero()[:, 0]
            if sel.numel() == 0:
                continue
            yy, xx = torch.meshgrid(torch.arange(by, ey, device=dev, dtype=torch.float64),
                                    torch.arange(bx, ex, device=dev, dtype=torch.float64), indexing="ij")
            u = torch.stack([(xx + 0.5 - cam.cx) / cam.fx, (yy + 0.5 - cam.cy) / cam.fy, torch.ones_like(xx)], -1)
            d = u.view(-1, 3) @ Rm
            d = d / d.norm(dim=1, keepdim=True)
            q = {a: v[sel].detach().requires_grad_(dl is not None) for a, v in p.items()}
            wm, og, s = _whiten(q, o)
            pi, gi = [], []
            with torch.no_grad():
                rows = max(1, int(4e7) // sel.numel())
                dc = d2c[sel]
                for r0 in range(0, len(d), rows):
                    dd = d[r0:r0 + rows]
                    dg = (dd @ wm.reshape(-1, 3).T).view(len(dd), -1, 3)
                    tau = -(dg * og).sum(-1) / (dg * dg).sum(-1)
                    d2 = (og + tau[..., None] * dg).square_().sum(-1)
                    a, b = ((tau > 0) & (d2 <= dc)).nonzero(as_tuple=True)
                    pi.append(a + r0)
                    gi.append(b)
            pi, gi = torch.cat(pi), torch.cat(gi)
            if pi.numel() == 0:
                continue

            def hit(pi, gi):
                dg = (wm[gi] @ d[pi][:, :, None])[:, :, 0]
                tau = -(dg * og[gi]).sum(-1) / (dg * dg).sum(-1)
                return tau, (og[gi] + tau[:, None] * dg).square().sum(-1)

            with torch.no_grad():  # order along each ray, then the hits that are composited
                tau, d2 = hit(pi, gi)
                at = torch.argsort(tau, stable=True)
                at = at[torch.argsort(pi[at], stable=True)]
                pi, gi, d2 = pi[at], gi[at], d2[at]
                cnt = torch.bincount(pi, minlength=len(d))
                rank = torch.arange(len(pi), device=dev) - (cnt.cumsum(0) - cnt)[pi]
                lt = torch.zeros((len(d), int(cnt.max())), dtype=torch.float64, device=dev)
                lt[pi, rank] = torch.log1p(-s[gi] * torch.exp(-0.5 * d2))
                lt = lt.cumsum(1) - lt
                keep = lt[pi, rank] >= math.log(T_MIN)
                pi, gi, rank = pi[keep], gi[keep], rank[keep]
                width = int(rank.max()) + 1
            a = s[gi] * torch.exp(-0.5 * hit(pi, gi)[1])
            col = (0.5 + (_sh_basis(d, k)[pi][:, :, None] * q["sh"][gi]).sum(1)).clamp_min(0.0)
            at = pi * width + rank
            l1 = torch.zeros(len(d) * width, dtype=torch.float64, device=dev).index_put((at,), torch.log1p(-a)).view(-1, width)
            T = torch.exp(l1.cumsum(1) - l1).reshape(-1)[at]
            out = torch.zeros_like(d).index_add(0, pi, (T * a)[:, None] * col).view(ey - by, ex - bx, 3)
            image[by:ey, bx:ex] = out.detach()
            if dl is not None:
                up = dl[by:ey, bx:ex] if isinstance(dl, torch.Tensor) else dl(out.detach(), slice(by, ey), slice(bx, ex))
                names = list(q)
                for a_, v in zip(names, torch.autograd.grad(out, [q[z] for z in names], up)):
                    grads[a_][sel] += v
    return image, grads


def exact(case, seed):
    if case["do"] == "map":
        return None  # whole numbers and codes of depth bounds
    if case["scene"] == "large" and case["n"] * case["width"] * case["height"] > 3e10:
        return None  # some hundred million hits
    p, dl, photos = _inputs(case, seed)
    p = {k: v.double() for k, v in p.items()}
    cam = _cameras(case)[0]
    if case["do"] == "render":
        return dict(image=_render64(p, cam, None)[0])
    up = dl.double()
    if case["do"] == "train":
        photo = photos[0].double()
        up = lambda img, ys, xs: torch.sign(img - photo[ys, xs])  # noqa: E731
    image, g = _render64(p, cam, up)
    g["logits"], p["logits"] = g.pop("opacity_logits"), p.pop("opacity_logits")
    if case["do"] != "train":
        return dict(image=image, grads=g)
    # Adam's first step from zero moments: the update is lr g / (|g| + eps)
    f = lambda v: float(np.float32(v))  # noqa: E731
    params = {k: p[k] - f(DEFAULT_LR[k]) * g[k] / (g[k].abs() + f(1e-15)) for k in GROUPS}
    return dict(loss=(image - photo).abs().sum().reshape(1), image=image, grads=g, params=params)
