"""The work that users of this library have it do, as timed cases.

Every case calls the public Python entry points (``gsc.Context``, ``gsc.Plan``
and the autograd functions) on synthetic scenes of the kinds in
``paper_2604_17155_amd.synthetic``: isotropic Gaussians in a cube ("plain") or
anisotropic ones clustered in blobs ("blobs"), cameras on a circle or a
hemisphere looking at the origin.  A case names its call, the scene's size, the
views, the channels, the SH degree and the targets' type:

  colorize  Context.colorize: images to SH coefficients
  plan      Plan.run over one or several scenes (sizes fixed when the plan was made)
  refine    Context.colorize_refine
  mask      Context.colorize of one mask channel, then Context.mask_filter
  render    Context.render: coefficients to images
  adjoint   Context.colorize_backward and Context.render_backward
  step      an optimisation step on opacity logits: sigmoid, autograd colorize,
            render, mean squared error, backward

``prepare`` makes the inputs on the device from the seed; ``run`` is one pass;
``exact`` evaluates the same quantity densely (every Gaussian at every pixel) in
64 bits with plain torch where that is affordable.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2604_17155_amd import autograd as ag
from paper_2604_17155_amd import gsc
from paper_2604_17155_amd import synthetic as syn

# Accepted contributions per pixel behind the operation counts of work(): the
# scenes here reach 24 to 69.
CONTRIBUTIONS_PER_PIXEL = 32
# Gaussian-pixel pairs that exact() evaluates at most, and those it keeps for
# the adjoints.
EXACT_PAIRS = 2.0e10
EXACT_PAIRS_KEPT = 4.0e7


def _case(name, do, geometry, n, views, width, height, C, L, dtype="f32", **more):
    c = {"do": do, "geometry": geometry, "n": n, "views": views, "width": width, "height": height,
         "C": C, "L": L, "dtype": dtype}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # The smallest call in use: a 2,000-Gaussian scene, eight thumbnails.
        # Latency: launches, the read-backs, host work.
        _case("colorize_2k_8x64", "colorize", "plain", 2000, 8, 64, 64, 3, 0),
        # The same scene behind a plan, as a serving loop keeps it.
        _case("plan_2k_8x64", "plan", "plain", 2000, 8, 64, 64, 3, 0, scenes=1),
        # Relighting: photographs of one lighting to degree-3 coefficients.
        _case("relight_100k_50x512", "colorize", "blobs", 100_000, 50, 512, 512, 3, 3),
        # A small capture of odd sizes: image edges inside a tile, a channel
        # count that fills no chunk, degree 2.
        _case("ragged_20k_9x333x251_c6", "colorize", "blobs", 20_011, 9, 333, 251, 6, 2),
        # Neural feature maps, 64 channels of BF16: the largest call.
        _case("features_500k_100x960x540", "colorize", "plain", 500_000, 100, 960, 540, 64, 0, "bf16"),
        # Segmentation labels, 16 channels of BF16, several scenes of uneven
        # size in one plan.
        _case("segment_plan_3_scenes", "plan", "plain", 210_000, 24, 1280, 720, 16, 0, "bf16", scenes=3),
        # One mask channel and the segmentation filter on the result.
        _case("mask_120k_20x800x600", "mask", "plain", 120_000, 20, 800, 600, 1, 0),
        # A viewer: one image of a relit scene.
        _case("render_300k_1x800", "render", "blobs", 300_000, 1, 800, 800, 3, 3),
        # Test-set renders of the same scene.
        _case("render_300k_40x800", "render", "blobs", 300_000, 40, 800, 800, 3, 3),
        # Coefficients refined against the residual, degree 1.
        _case("refine_100k_20x512", "refine", "blobs", 100_000, 20, 512, 512, 3, 1, passes=3),
        # Both adjoints on a small scene of odd sizes with BF16 targets.
        _case("adjoint_1500_5x61x47_c7", "adjoint", "blobs", 1500, 5, 61, 47, 7, 1, "bf16"),
        # An optimisation step through colorize and render.
        _case("step_300k_40x800", "step", "blobs", 300_000, 40, 800, 800, 3, 3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["colorize", "colorize", "colorize", "plan", "plan", "mask", "render", "refine", "adjoint", "step"])
    n = _log_int(rng, 1500, 400_000)
    views = _log_int(rng, 1, 100)
    width = _log_int(rng, 48, 1280)
    height = max(32, min(960, int(width * rng.uniform(0.5, 1.1))))
    L = rng.choice([0, 0, 1, 2, 3, 3])
    C = rng.choice([1, 2, 3, 3, 3, 3, 4, 6, 8, 13, 16, 16, 24, 32, 64])
    dtype = "bf16" if C >= 13 or rng.random() < 0.2 else "f32"
    if do == "mask":
        C, L, dtype = 1, 0, "f32"
    if do in ("adjoint", "step", "refine", "render") and C > 8:
        C = rng.choice([3, 3, 7, 8])
    if do == "plan" and C >= 13:
        L = 0
    if L > 0 and C > 16:
        L = 0
    if do == "render":
        dtype = "f32"
    # no dearer than the largest listed case: its items, pixels and sums
    per_pass = {"refine": 6, "step": 6, "adjoint": 4}.get(do, 1)
    views = max(1, min(views, int(2.0e7 / n / per_pass), int(2.5e7 * min(1.0, 16.0 / C) / (width * height) / per_pass)))
    c = _case(None, do, rng.choice(["plain", "blobs"]), n, views, width, height, C, L, dtype)
    if do == "plan":
        c["scenes"] = rng.choice([1, 2, 3, 5])
    if do == "refine":
        c["passes"] = rng.choice([1, 2, 4])
    return c


# ---- inputs ----------------------------------------------------------------

def _scenes(case):
    """(Gaussians, views, width, height) of each scene of the case."""
    n, v, w, h = case["n"], case["views"], case["width"], case["height"]
    out = []
    for k in range(case.get("scenes", 1)):
        # uneven scenes: each later one has fewer Gaussians, more or fewer
        # views and smaller images
        f = (1.0, 0.29, 0.081, 0.45, 0.17)[k % 5]
        out.append((max(64, int(n * f)), max(1, int(v * (1.0, 1.4, 0.9, 0.6, 1.2)[k % 5])),
                    max(16, int(w * (1.0, 0.63, 0.5, 0.75, 0.6)[k % 5])),
                    max(16, int(h * (1.0, 0.83, 0.67, 0.75, 0.75)[k % 5]))))
    return out


def _geometry(case, seed):
    """Concatenated Gaussians of the case's scenes, the scenes' cameras and
    the plan's scene table."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    parts, cams, table = [], [], []
    g0 = 0
    for n, v, w, h in _scenes(case):
        parts.append(syn.blob_geometry(rng, n) if case["geometry"] == "blobs" else syn.isotropic_geometry(rng, n))
        table.append((g0, n, len(cams), v))
        cams += syn.circle_cams(v, 3.0, w, h) if v <= 8 else syn.hemisphere_cams(v, 3.0, w, h)
        g0 += n
    return [np.ascontiguousarray(np.concatenate(p)) for p in zip(*parts)], cams, table


def _smooth(gen, n_img, C, h, w, cell, mode):
    """n_img smooth random maps [n_img, h * w, C] in [0, 1] (or normal values)."""
    lo = torch.randn((n_img, C, max(2, h // cell), max(2, w // cell)), generator=gen, device="cuda")
    x = torch.nn.functional.interpolate(lo, size=(h, w), mode="bilinear")
    if mode == "image":
        x = (0.5 + 0.25 * x).clamp_(0.0, 1.0)
    return x.permute(0, 2, 3, 1).reshape(n_img, h * w, C)


def _targets(case, cams, seed):
    """Images (C <= 8), label maps (C = 1: a mask; 16: one-hot) or feature maps."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    C = case["C"]
    out = torch.empty((sum(c.width * c.height for c in cams), C),
                      dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32, device="cuda")
    r = 0
    for c in cams:
        p = c.width * c.height
        if case["do"] == "mask":
            y = (_smooth(gen, 1, 1, c.height, c.width, 64, "normal")[0] > 0.0).float()
        elif C == 16 and case["dtype"] == "bf16":
            y = torch.nn.functional.one_hot(_smooth(gen, 1, C, c.height, c.width, 64, "normal")[0].argmax(1), C).float()
        elif C > 8:
            y = _smooth(gen, 1, C, c.height, c.width, 14, "normal")[0]
        else:
            y = _smooth(gen, 1, C, c.height, c.width, 24, "image")[0]
            y = y + 0.01 * torch.randn(y.shape, generator=gen, device="cuda")
        out[r:r + p] = y
        r += p
    return out


def _coeffs(case, n, seed):
    """Coefficients as colorize returns them: a mean colour, smaller higher degrees."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 77)
    nb, C = (case["L"] + 1) ** 2, case["C"]
    c = 0.1 * torch.randn((n, nb, C), generator=gen, device="cuda")
    c[:, 0] = torch.rand((n, C), generator=gen, device="cuda") / syn.Y00
    return c


def _lam(case):
    return [1e-4] if case["L"] == 0 else [float(v) for v in syn.paper_lambda(case["L"])]


def prepare(case, seed):
    geo, cams, table = _geometry(case, seed)
    s = {"case": case, "cams": cams, "lam": _lam(case),
         "geo": [torch.from_numpy(a).cuda() for a in geo], "context": gsc.Context()}
    do, n = case["do"], int(geo[0].shape[0])
    if do != "render":
        s["targets"] = _targets(case, cams, seed)
    if do == "render":
        s["coeffs"] = _coeffs(case, n, seed)
    elif do == "plan":
        s["plan"] = gsc.Plan(s["context"], table, *s["geo"], cams, case["C"], case["L"])
        s["out"] = (torch.zeros((n, (case["L"] + 1) ** 2, case["C"]), device="cuda"),
                    torch.zeros((n,), dtype=torch.uint8, device="cuda"))
    elif do == "adjoint":
        gen = torch.Generator(device="cuda").manual_seed(int(seed) + 5)
        s["coeffs"] = s["context"].colorize(*s["geo"], cams, s["targets"], case["L"], s["lam"])[0]
        s["grad_coeffs"] = torch.randn(s["coeffs"].shape, generator=gen, device="cuda")
        s["grad_images"] = torch.randn(s["targets"].shape, generator=gen, device="cuda")
    elif do == "step":
        s["logits"] = torch.logit(s["geo"][3].double()).float().requires_grad_(True)
        s["targets"].requires_grad_(True)
    return s


def run(s):
    case, ctx, cams, lam = s["case"], s["context"], s["cams"], s["lam"]
    do, L = case["do"], case["L"]
    m, sc, q, o = s["geo"]
    if do == "colorize":
        return ctx.colorize(m, sc, q, o, cams, s["targets"], L, lam)
    if do == "plan":
        return s["plan"].run(s["targets"], lam, *s["out"])
    if do == "refine":
        return ctx.colorize_refine(m, sc, q, o, cams, s["targets"], L, lam, case["passes"])
    if do == "mask":
        coeffs, status = ctx.colorize(m, sc, q, o, cams, s["targets"], 0, lam)
        return coeffs, status, ctx.mask_filter(coeffs, status=status)[0]
    if do == "render":
        return ctx.render(m, sc, q, o, cams, s["coeffs"])
    if do == "adjoint":
        gt, go = ctx.colorize_backward(m, sc, q, o, cams, s["targets"], L, lam, s["coeffs"], s["grad_coeffs"])
        gc, go2 = ctx.render_backward(m, sc, q, o, cams, s["coeffs"], s["grad_images"])
        return gt, go, gc, go2
    # step: the opacities are new tensors in every pass (their logits are what
    # is optimised), so each pass bins once and its four calls share the lists
    y, logits = s["targets"], s["logits"]
    y.grad = logits.grad = None
    op = torch.sigmoid(logits)
    coeffs = ag.colorize(y, op, m, sc, q, cams, L, lam, context=ctx, reuse_binning=True)
    images = ag.render(coeffs, op, m, sc, q, cams, context=ctx, reuse_binning=True)
    loss = ((images - y.detach().float()) ** 2).mean()
    loss.backward()
    return loss.detach(), coeffs.detach(), y.grad, logits.grad


def work(case):
    """What a pass cannot do without: geometry, targets or images and
    coefficients once; the weights and sums of the contributions, the fold of
    every (view, Gaussian) and the solves."""
    C, L = case["C"], case["L"]
    nb = (L + 1) ** 2
    ts = 2 if case["dtype"] == "bf16" else 4
    n = px = items = 0
    for gn, v, w, h in _scenes(case):
        n, px, items = n + gn, px + v * w * h, items + gn * v
    geo, coef = 44 * n, 4 * n * nb * C
    weight = 14 * px * CONTRIBUTIONS_PER_PIXEL
    sums = 2 * (C + 1) * px * CONTRIBUTIONS_PER_PIXEL
    fold = items * (nb * (nb + 1) + 2 * nb * C) if L else 0
    solve = n * (nb ** 3 / 3 + 2 * nb * nb * C)
    do = case["do"]
    if do == "render":
        return {"bytes": geo + coef + 4 * px * C, "flops": weight + sums + 2 * items * nb * C}
    if do == "refine":
        return {"bytes": geo + coef + ts * px * C, "flops": (1 + case["passes"]) * (weight + 2 * sums + fold + solve)}
    if do == "adjoint":
        return {"bytes": geo + 4 * coef + (ts + 8) * px * C + 8 * n, "flops": 3 * (weight + 2 * sums) + fold + solve}
    if do == "step":
        return {"bytes": geo + coef + 2 * ts * px * C + 8 * n, "flops": 4 * weight + 6 * sums + 2 * (fold + solve)}
    return {"bytes": geo + coef + ts * px * C + n, "flops": weight + sums + fold + solve}


# ---- 64-bit reference ------------------------------------------------------

def _sh(d, L):
    """Real orthonormal spherical harmonics of unit directions [N, 3]."""
    x, y, z = d.unbind(1)
    r = lambda a, b: math.sqrt(a / (b * math.pi))
    out = [torch.full_like(x, r(1, 4))]
    if L >= 1:
        out += [r(3, 4) * y, r(3, 4) * z, r(3, 4) * x]
    if L >= 2:
        out += [r(15, 4) * x * y, r(15, 4) * y * z, r(5, 16) * (3 * z * z - 1), r(15, 4) * x * z,
                r(15, 16) * (x * x - y * y)]
    if L >= 3:
        out += [r(35, 32) * y * (3 * x * x - y * y), r(105, 4) * x * y * z, r(21, 32) * y * (5 * z * z - 1),
                r(7, 16) * z * (5 * z * z - 3), r(21, 32) * x * (5 * z * z - 1), r(105, 16) * z * (x * x - y * y),
                r(35, 32) * x * (x * x - 3 * y * y)]
    return torch.stack(out, 1)


class _Dense:
    """One scene of a case, evaluated densely in 64 bits."""

    def __init__(self, geo, cams, L, dev, opacities=None):
        f = lambda a: torch.from_numpy(a).to(dev).double()
        self.m, self.s, self.q = f(geo[0]), f(geo[1]), f(geo[2])
        self.o = f(geo[3]) if opacities is None else opacities
        self.cams, self.L, self.dev, self.N = cams, L, dev, int(geo[0].shape[0])
        w, x, y, z = (self.q / self.q.norm(dim=1, keepdim=True)).unbind(1)
        R = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                         2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                         2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
        self.cov = (R * (self.s ** 2)[:, None, :]) @ R.transpose(1, 2).contiguous()
        self.views = [self._project(c) for c in cams]

    def _project(self, c):
        Rn = np.asarray(c.R, np.float32).astype(np.float64).reshape(3, 3)
        R = torch.from_numpy(Rn).to(self.dev)
        t = torch.tensor([float(np.float32(v)) for v in c.t], dtype=torch.float64, device=self.dev)
        fx, fy, cx, cy = (float(np.float32(v)) for v in (c.fx, c.fy, c.cx, c.cy))
        # the depth key is defined in binary32, as a chain of fused multiply-adds
        k = t[2]
        for i in (2, 1, 0):
            k = (R[2, i] * self.m[:, i] + k).float().double()
        p = self.m @ R.T.contiguous() + t
        iz = 1.0 / p[:, 2]
        J = torch.zeros((self.N, 2, 3), dtype=torch.float64, device=self.dev)
        J[:, 0, 0], J[:, 0, 2] = fx * iz, -fx * p[:, 0] * iz * iz
        J[:, 1, 1], J[:, 1, 2] = fy * iz, -fy * p[:, 1] * iz * iz
        T = J @ R
        S = T @ self.cov @ T.transpose(1, 2).contiguous()
        a, b, d = S[:, 0, 0] + float(np.float32(0.3)), S[:, 0, 1], S[:, 1, 1] + float(np.float32(0.3))
        det = a * d - b * b
        order = torch.argsort(k, stable=True)
        order = order[k[order] > float(np.float32(0.01))]
        centre = -(R.T @ t)
        direction = self.m - centre
        return {"u": (fx * p[:, 0] * iz + cx)[order], "v": (fy * p[:, 1] * iz + cy)[order],
                "a": (d / det)[order], "b": (-b / det)[order], "c": (a / det)[order], "order": order,
                "phi": _sh(direction / direction.norm(dim=1, keepdim=True), self.L), "w": c.width, "h": c.height}

    def weights(self, j, p0, p1):
        """Weights [visible Gaussians in depth order, pixels p0..p1) of view j."""
        V = self.views[j]
        px = torch.arange(p0, p1, device=self.dev)
        dx = (px % V["w"]).double() + 0.5 - V["u"][:, None]
        dy = (px // V["w"]).double() + 0.5 - V["v"][:, None]
        q = V["a"][:, None] * dx * dx + 2.0 * V["b"][:, None] * dx * dy + V["c"][:, None] * dy * dy
        alpha = (self.o[V["order"]][:, None] * torch.exp(-0.5 * q)).clamp(max=float(np.float32(0.99)))
        alpha = torch.where((q <= 9.0) & (alpha >= float(np.float32(1.0 / 255.0))), alpha, torch.zeros_like(alpha))
        T = torch.cumprod(1.0 - alpha, 0)
        before = torch.cat([torch.ones_like(T[:1]), T[:-1]])
        return torch.where(T >= float(np.float32(1e-4)), alpha * before, torch.zeros_like(T))

    def spans(self, j):
        n_px = self.cams[j].width * self.cams[j].height
        step = max(64, int(3e7 // max(self.N, 1)))
        return [(p, min(p + step, n_px)) for p in range(0, n_px, step)]

    def sums(self, y):
        """Per view: visibilities [N] and weighted target sums [N, C]."""
        out, r = [], 0
        for j in range(len(self.cams)):
            o = self.views[j]["order"]
            V = torch.zeros(self.N, dtype=torch.float64, device=self.dev)
            S = torch.zeros((self.N, y.shape[1]), dtype=torch.float64, device=self.dev)
            for p0, p1 in self.spans(j):
                w = self.weights(j, p0, p1)
                V = V.index_add(0, o, w.sum(1))
                S = S.index_add(0, o, w @ y[r + p0:r + p1])
            r += self.cams[j].width * self.cams[j].height
            out.append((V, S))
        return out

    def normal(self, sums):
        nb = (self.L + 1) ** 2
        A = torch.zeros((self.N, nb, nb), dtype=torch.float64, device=self.dev)
        B = torch.zeros((self.N, nb, sums[0][1].shape[1]), dtype=torch.float64, device=self.dev)
        w = torch.zeros(self.N, dtype=torch.float64, device=self.dev)
        for j, (V, S) in enumerate(sums):
            phi = self.views[j]["phi"]
            A = A + (V[:, None] * phi)[:, :, None] * phi[:, None, :]
            B = B + phi[:, :, None] * S[:, None, :]
            w = w + V
        return A, B, w

    def system(self, A, w, lam):
        lam = [float(np.float32(v)) for v in lam]
        d = [lam[l] if len(lam) > 1 else lam[0] for l in range(self.L + 1) for _ in range(2 * l + 1)]
        d = torch.tensor(d, dtype=torch.float64, device=self.dev)
        seen = w > 0
        eye = torch.eye(len(d), dtype=torch.float64, device=self.dev)
        return torch.where(seen[:, None, None], A + w[:, None, None] * torch.diag(d), eye), d, seen

    def solve(self, A, B, w, lam):
        M, _, seen = self.system(A, w, lam)
        L = torch.linalg.cholesky(M)
        x = torch.linalg.solve_triangular(L.transpose(1, 2), torch.linalg.solve_triangular(L, B, upper=False), upper=True)
        return torch.where(seen[:, None, None], x, torch.zeros_like(x))

    def render(self, coeffs):
        out = []
        for j in range(len(self.cams)):
            col = (self.views[j]["phi"][:, :, None] * coeffs).sum(1)[self.views[j]["order"]]
            out += [self.weights(j, p0, p1).T.contiguous() @ col for p0, p1 in self.spans(j)]
        return torch.cat(out)


def exact(case, seed):
    pairs = sum(n * v * w * h for n, v, w, h in _scenes(case))
    do = case["do"]
    passes = {"refine": 1 + 2 * case.get("passes", 0)}.get(do, 1)
    if pairs * passes > EXACT_PAIRS or (do in ("adjoint", "step") and pairs > EXACT_PAIRS_KEPT):
        return None
    dev = "cuda"
    geo, cams, table = _geometry(case, seed)
    L, lam = case["L"], _lam(case)
    if do == "render":
        c = _coeffs(case, int(geo[0].shape[0]), seed).to(dev).double()
        return _Dense(geo, cams, L, dev).render(c)
    if do in ("adjoint", "step"):
        return _exact_adjoint(case, seed, geo, cams, lam, dev)
    y = _targets(case, cams, seed).to(dev).double()
    res, r = [], 0
    for g0, n, c0, v in table:
        cs = cams[c0:c0 + v]
        rows = sum(c.width * c.height for c in cs)
        d = _Dense([a[g0:g0 + n] for a in geo], cs, L, dev)
        yk = y[r:r + rows]
        r += rows
        A, B, w = d.normal(d.sums(yk))
        x = d.solve(A, B, w, lam)
        for _ in range(case.get("passes", 0) if do == "refine" else 0):
            _, B, _ = d.normal(d.sums(yk - d.render(x)))
            M, diag, _ = d.system(A, w, lam)
            x = x + d.solve(A, B - w[:, None, None] * diag[:, None] * x, w, lam)
        res.append(x)
    coeffs = torch.cat(res)
    return (coeffs, None, None) if do == "mask" else (coeffs, None)


def _exact_adjoint(case, seed, geo, cams, lam, dev):
    s = prepare(case, seed)
    y = s["targets"].detach().to(dev).double().requires_grad_(True)
    if case["do"] == "step":
        z = s["logits"].detach().to(dev).double().requires_grad_(True)
        d = _Dense(geo, cams, case["L"], dev, torch.sigmoid(z))
        coeffs = d.solve(*d.normal(d.sums(y)), lam)
        loss = ((d.render(coeffs) - y.detach()) ** 2).mean()
        loss.backward()
        return loss.detach(), coeffs.detach(), y.grad, z.grad
    o = torch.from_numpy(geo[3]).to(dev).double().requires_grad_(True)
    d = _Dense(geo, cams, case["L"], dev, o)
    gt, go = torch.autograd.grad(d.solve(*d.normal(d.sums(y)), lam), (y, o), s["grad_coeffs"].to(dev).double())
    c = s["coeffs"].to(dev).double().requires_grad_(True)
    gc, go2 = torch.autograd.grad(d.render(c), (c, o), s["grad_images"].to(dev).double())
    return gt, go, gc, go2
