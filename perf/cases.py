"""Performance cases of the shape-measurement library.

Each case is one call sequence that a program using the package makes, through
its public entry points: the whole pipeline (centroid, moments, profile fit)
over batches of postage stamps, star sizes, chi^2 and its gradient for fits
driven from outside, the work-queue fit on preallocated outputs, and the front
end on whole frames.  Inputs are synthetic, drawn on the GPU from the seed
alone, with the distributions of the repository's own workloads: Sersic
galaxies of n U(0.5, 4), Re log-U(1.5, 6) px, e_i N(0, 0.25) with |e| < 0.7,
flux log-U(1e3, 1e5), S/N log-U(20, 200), sky 10; Moffat stars of beta
U(2.5, 5), FWHM U(2, 5), S/N log-U(50, 500); mixed-side batches with 20% stars
of beta 3; frames with one bright galaxy each.
"""
import math

import numpy as np
import torch

import paper_1203_0571_amd as shape

DEV = "cuda:0"
SKY = 10.0
CHUNK_PIXELS = 1 << 26   # pixels rendered at a time

# LM sweeps and weighted-moment steps per stamp on these inputs (means of the
# library's own counters), for the work estimate only
SWEEPS, CENTROID_STEPS, MOMENT_STEPS, STAR_STEPS = 9.3, 8, 7, 12


def listed():
    return [
        # a survey tile's galaxies, cut to 64 x 64 and stored in FP16: the
        # package's benchmark, and the largest batch of one call
        dict(name="pipeline_64_f16", kind="pipeline", n=262144, side=64, f16=True, mask=0xFF,
             perr=False),
        # one exposure's galaxies in 48 x 48 FP32 cut-outs, with error bars
        dict(name="pipeline_48", kind="pipeline", n=100000, side=48, f16=False, mask=0xFF,
             perr=True),
        # cut-outs sized by the objects: sides 16 to 128, galaxies and stars
        dict(name="pipeline_uneven", kind="uneven", n=200000, f16=False, perr=False),
        # one small field: a few dozen objects, where launches and the slowest
        # stamp count
        dict(name="pipeline_few", kind="pipeline", n=64, side=48, f16=False, mask=0xFF, perr=True),
        # the paper's split fit (centre and shape held) on one catalogue page
        dict(name="pipeline_32_size", kind="pipeline", n=1000, side=32, f16=False, mask=0xF0,
             perr=False),
        # the stars of a survey tile, for the point-spread function
        dict(name="stars_32", kind="stars", n=1048576, side=32, profile=1, beta=0.0),
        # a gradient step on the parameters of a whole batch, through autograd
        dict(name="gradient_64", kind="chi2", n=65536, side=64, f16=False, want="autograd"),
        # normal equations for a fit driven from outside, FP16 stamps
        dict(name="normal_48_f16", kind="chi2", n=20000, side=48, f16=True, want="normal"),
        # the same for one small field of odd-sided stamps
        dict(name="gradient_few", kind="chi2", n=100, side=33, f16=False, want="autograd"),
        # detection and cut-outs on the paper's 512 x 512 simulation frames
        dict(name="frames_512", kind="frames", n=4096, height=512, width=512, f16=False),
        # a few large detector frames as they arrive
        dict(name="frames_large", kind="frames", n=4, height=2048, width=2048, f16=False),
        # a serving loop: the fit without allocation, mixed sides, small batch
        dict(name="serve_uneven", kind="queue", n=2000, f16=False, side=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pipeline", "pipeline", "uneven", "stars", "chi2", "chi2", "frames",
                       "frames", "queue"])
    f16 = rng.random() < 0.4
    if kind == "pipeline":
        side = rng.choice([16, 32, 48, 64, 96, 128]) if rng.random() < 0.4 else _log_int(rng, 12, 128)
        return dict(kind=kind, n=_log_int(rng, 16, 3e8 / side ** 2), side=side, f16=f16,
                    mask=0xFF if rng.random() < 0.75 else 0xF0, perr=rng.random() < 0.5)
    if kind == "uneven":
        return dict(kind=kind, n=_log_int(rng, 50, 100000), f16=f16, perr=rng.random() < 0.5)
    if kind == "stars":
        side = 32 if rng.random() < 0.5 else _log_int(rng, 16, 64)
        profile = rng.choice([0, 1, 2])   # Gaussian, Moffat, Moffat with beta fixed
        return dict(kind=kind, n=_log_int(rng, 16, 3e8 / side ** 2), side=side, profile=profile,
                    beta=round(rng.uniform(2.5, 5.0), 2) if profile == 2 else 0.0)
    if kind == "chi2":
        side = rng.choice([16, 32, 48, 64, 96, 128]) if rng.random() < 0.4 else _log_int(rng, 12, 128)
        return dict(kind=kind, n=_log_int(rng, 16, 2e8 / side ** 2), side=side, f16=f16,
                    want=rng.choice(["autograd", "autograd", "normal", "value"]))
    if kind == "frames":
        height, width = _log_int(rng, 128, 4096), _log_int(rng, 128, 4096)
        if rng.random() < 0.4:
            width = height = rng.choice([256, 512, 1024, 2048, 4096])
        return dict(kind=kind, n=_log_int(rng, 1, 8e8 / (height * width)), height=height,
                    width=width, f16=f16)
    return dict(kind=kind, n=_log_int(rng, 16, 20000), f16=f16,
                side=0 if rng.random() < 0.5 else _log_int(rng, 12, 128))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _uniform(g, lo, hi, n):
    return lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _log_uniform(g, lo, hi, n):
    return torch.exp(_uniform(g, math.log(lo), math.log(hi), n))


def _ellipticity(g, n):
    """N(0, 0.25) in each component; those of |e| >= 0.7 are scaled inside."""
    e = 0.25 * torch.randn(n, 2, generator=g, device=DEV, dtype=torch.float64)
    r = torch.hypot(e[:, 0], e[:, 1])
    return e * torch.where(r >= 0.7, 0.7 * torch.rand(n, generator=g, device=DEV,
                                                      dtype=torch.float64) / r.clamp(min=1e-9),
                           torch.ones_like(r))[:, None]


def _b(n):
    """Half-light constant b(n), its asymptotic series (1e-5 or better here)."""
    return 2 * n - 1 / 3 + 4 / (405 * n) + 46 / (25515 * n ** 2) + 131 / (1148175 * n ** 3)


def _sersic_norm(n, re, b):
    """Integral of exp(-b (R/re)^(1/n))."""
    return 2 * math.pi * n * re ** 2 * torch.exp(torch.lgamma(2 * n) - 2 * n * torch.log(b))


def _galaxies(g, n, sides):
    """Truth parameters [n, 8] (FP64) and pixel noise."""
    p = torch.zeros(n, 8, device=DEV, dtype=torch.float64)
    c = (sides.double() - 1) / 2
    shift = torch.clamp(sides.double() / 16, max=2.0)
    p[:, 0] = c + shift * _uniform(g, -1, 1, n)
    p[:, 1] = c + shift * _uniform(g, -1, 1, n)
    p[:, 2:4] = _ellipticity(g, n)
    p[:, 4] = _log_uniform(g, 1.5, 6.0, n) * torch.clamp(sides.double() / 48, max=1.0)
    p[:, 5] = _uniform(g, 0.5, 4.0, n)
    p[:, 7] = SKY
    b = _b(p[:, 5])
    p[:, 6] = _log_uniform(g, 1e3, 1e5, n) / _sersic_norm(p[:, 5], p[:, 4], b)
    sigma = p[:, 6] * torch.sqrt(_sersic_norm(p[:, 5], p[:, 4], 2 * b)) / _log_uniform(g, 20, 200, n)
    return p, sigma


def _stars(g, n, sides, beta, flux, snr):
    p = torch.zeros(n, 8, device=DEV, dtype=torch.float64)
    c = (sides.double() - 1) / 2
    p[:, 0] = c + _uniform(g, -2, 2, n)
    p[:, 1] = c + _uniform(g, -2, 2, n)
    r, phi = 0.1 * torch.sqrt(_uniform(g, 0, 1, n)), _uniform(g, 0, 2 * math.pi, n)
    p[:, 2], p[:, 3] = r * torch.cos(phi), r * torch.sin(phi)
    p[:, 4] = _uniform(g, 2, 5, n) / (2 * torch.sqrt(2 ** (1 / beta) - 1))
    p[:, 5] = beta
    p[:, 6] = _log_uniform(g, *flux, n) * (beta - 1) / (math.pi * p[:, 4] ** 2)
    p[:, 7] = SKY
    sigma = p[:, 6] * torch.sqrt(math.pi * p[:, 4] ** 2 / (2 * beta - 1)) / _log_uniform(g, *snr, n)
    return p, sigma


def _r2(x, y, p):
    """The model's elliptical R^2; p's columns broadcast against x, y."""
    ux, uy = x - p[0], y - p[1]
    vx, vy = (1 - p[2]) * ux - p[3] * uy, -p[3] * ux + (1 + p[2]) * uy
    return ((vx * vx + vy * vy) / (1 - p[2] ** 2 - p[3] ** 2)).clamp(min=1e-8)


def _render(x, y, p, star):
    """Noiseless pixels with sky, FP32; star: truth value or a bool tensor."""
    r2 = _r2(x, y, p)
    n = p[5]
    if star is True:
        return p[6] * (1 + r2 / p[4] ** 2) ** -n + p[7]
    gal = p[6] * torch.exp(-_b(n) * (r2 / p[4] ** 2) ** (0.5 / n)) + p[7]
    if star is False:
        return gal
    return torch.where(star, p[6] * (1 + r2 / p[4] ** 2) ** -n + p[7], gal)


def _pack(noisy, f16):
    """noisy [k, npix] -> stored pixels and scale (a power of two per stamp)."""
    if not f16:
        return noisy, None
    scale = torch.exp2(torch.ceil(torch.log2(noisy.abs().amax(1).clamp(min=1e-30) / 32768.0)))
    return (noisy / scale[:, None]).half(), scale


def _uniform_batch(g, n, side, f16, p, sigma, star=False):
    """Stamps of one side, rendered in chunks."""
    p32, s32 = p.float(), sigma.float()
    pix = torch.empty(n, side * side, device=DEV, dtype=torch.float16 if f16 else torch.float32)
    scale = torch.ones(n, device=DEV) if f16 else None
    c = torch.arange(side, device=DEV, dtype=torch.float32)
    x, y = c.repeat(side)[None], c.repeat_interleave(side)[None]
    step = max(1, CHUNK_PIXELS // (side * side))
    for a in range(0, n, step):
        q = p32[a:a + step].T[:, :, None]
        m = _render(x, y, q, star)
        m += s32[a:a + step, None] * torch.randn(m.shape, generator=g, device=DEV)
        pix[a:a + step], sc = _pack(m, f16)
        if f16:
            scale[a:a + step] = sc
    return shape.DeviceBatch(pixels=pix.reshape(-1), sigma=s32, side0=side, scale=scale)


def _uneven_batch(g, n, f16):
    """Sides round(exp U(ln 16, ln 128)), 80% galaxies (Re = side / 8), 20% stars."""
    sides = torch.round(_log_uniform(g, 16, 128, n)).int()
    p, sigma = _galaxies(g, n, sides)
    flux_scale = (sides.double() / 8) / p[:, 4]     # Re = side / 8 at the same flux
    p[:, 4] *= flux_scale
    p[:, 6] /= flux_scale ** 2
    sigma = sigma / flux_scale
    ps, ss = _stars(g, n, sides, torch.full_like(sigma, 3.0), (1e3, 1e5), (20, 200))
    star = _uniform(g, 0, 1, n) < 0.2
    p, sigma = torch.where(star[:, None], ps, p), torch.where(star, ss, sigma)
    area = sides.long() ** 2
    offsets = torch.zeros(n, device=DEV, dtype=torch.int64)
    offsets[1:] = torch.cumsum(area, 0)[:-1]
    total = int(area.sum())
    pix = torch.empty(total, device=DEV, dtype=torch.float16 if f16 else torch.float32)
    scale = torch.ones(n, device=DEV) if f16 else None
    p32, s32 = p.float(), sigma.float()
    if f16:   # the peak bounds every pixel of the stamp
        peak = p32[:, 6].abs() + SKY + 6 * s32
        scale = torch.exp2(torch.ceil(torch.log2(peak / 32768.0)))
    host = torch.cat([offsets, torch.tensor([total], device=DEV)]).cpu().numpy()
    a = 0
    while a < n:
        e = max(a + 1, int(np.searchsorted(host, host[a] + CHUNK_PIXELS)) - 1)
        e = min(e, n)
        lo, hi = int(host[a]), int(host[e])
        k = torch.repeat_interleave(torch.arange(a, e, device=DEV), area[a:e])
        local = (torch.arange(lo, hi, device=DEV) - offsets[k]).int()
        w = sides[k]
        y = torch.div(local, w, rounding_mode="floor")
        x = local - y * w
        m = _render(x.float(), y.float(), p32[k].T, star[k])
        m += s32[k] * torch.randn(m.shape, generator=g, device=DEV)
        pix[lo:hi] = (m / scale[k]).half() if f16 else m
        a = e
    return shape.DeviceBatch(pixels=pix, sigma=s32, offsets=offsets, sides=sides, scale=scale,
                             model=star.to(torch.uint8))


def _frames(g, case):
    """One galaxy per frame, S/N log-U(5e3, 5e4), somewhere in the inner half;
    noise over the whole frame."""
    n, h, w = case["n"], case["height"], case["width"]
    p, _ = _galaxies(g, n, torch.full((n,), 64, device=DEV))
    p[:, 0], p[:, 1] = w * _uniform(g, 0.25, 0.75, n), h * _uniform(g, 0.25, 0.75, n)
    b = _b(p[:, 5])
    p[:, 6] = _log_uniform(g, 1e4, 1e6, n) / _sersic_norm(p[:, 5], p[:, 4], b)
    # the sum over a frame carries the noise of all its pixels, so the S/N
    # grows with the frame's side to keep its total flux as certain
    snr = _log_uniform(g, 5e3, 5e4, n) * max(1.0, math.sqrt(h * w) / 512)
    sigma = (p[:, 6] * torch.sqrt(_sersic_norm(p[:, 5], p[:, 4], 2 * b)) / snr).float()
    p32 = p.float()
    pix = torch.empty(n, h, w, device=DEV, dtype=torch.float16 if case["f16"] else torch.float32)
    scale = torch.ones(n, device=DEV) if case["f16"] else None
    x = torch.arange(w, device=DEV, dtype=torch.float32)[None, None, :]
    y = torch.arange(h, device=DEV, dtype=torch.float32)[None, :, None]
    step = max(1, CHUNK_PIXELS // (h * w))
    for a in range(0, n, step):
        m = _render(x, y, p32[a:a + step].T[:, :, None, None], False)
        m += sigma[a:a + step, None, None] * torch.randn(m.shape, generator=g, device=DEV)
        k = m.shape[0]
        got, sc = _pack(m.reshape(k, -1), case["f16"])
        pix[a:a + step] = got.reshape(k, h, w)
        if case["f16"]:
            scale[a:a + step] = sc
    return shape.DeviceFrames(pixels=pix, scale=scale), sigma


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind, n = case["kind"], case["n"]
    if kind == "frames":
        frames, sigma = _frames(g, case)
        cut = torch.zeros(n * 128 * 128, device=DEV)
        return dict(case=case, frames=frames, sigma=sigma, cut=cut)
    if kind == "uneven" or (kind == "queue" and case["side"] == 0):
        batch, p = _uneven_batch(g, n, case["f16"]), None
    else:
        sides = torch.full((n,), case["side"], device=DEV)
        if kind == "stars":
            p, sigma = _stars(g, n, sides, _uniform(g, 2.5, 5.0, n), (1e4, 1e6), (50, 500))
        else:
            p, sigma = _galaxies(g, n, sides)
        batch = _uniform_batch(g, n, case["side"], case.get("f16", False), p, sigma,
                               kind == "stars")
    s = dict(case=case, batch=batch)
    if kind in ("pipeline", "uneven"):
        s["opts"] = shape.default_opts(free_mask=case.get("mask", 0xFF))
    if kind == "chi2":
        # where an optimiser stands some steps from the end: each parameter a
        # few per cent off
        p = p.clone()
        p[:, 0:2] += 0.1 * torch.randn(n, 2, generator=g, device=DEV, dtype=torch.float64)
        p[:, 2:4] *= 0.95
        p[:, 4:7] *= 1 + 0.03 * torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
        p[:, 5].clamp_(0.3, 8.0)
        s["params"] = p.float().contiguous().requires_grad_(case["want"] == "autograd")
        s["upstream"] = _uniform(g, 0.5, 1.5, n).float()
    if kind == "queue":
        f32 = dict(device=DEV, dtype=torch.float32)
        i32 = dict(device=DEV, dtype=torch.int32)
        s["opts"], s["cfg"] = shape.default_opts(), shape.queue_cfg()
        s["out"] = dict(p=torch.empty(n, 8, **f32), chi2=torch.empty(n, **f32),
                        iters=torch.empty(n, **i32), status=torch.empty(n, **i32),
                        sweeps=torch.empty(n, **i32))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("pipeline", "uneven"):
        return shape.pipeline(state["batch"], state["opts"], want_perr=case["perr"])
    if kind == "stars":
        batch = state["batch"]
        rec0, _, _ = shape.centroid(batch)
        rec, it, st = shape.moments(batch, rec0)
        if case["profile"] == 2:
            out, its, sts = shape.star_moments_beta(batch, rec, case["beta"])
        else:
            out, its, sts = shape.star_moments(batch, rec, case["profile"])
        return dict(centroid=rec0, moments=rec, iters=it, status=st, star=out, star_iters=its,
                    star_status=sts)
    if kind == "chi2":
        batch, p = state["batch"], state["params"]
        if case["want"] == "value":
            return dict(chi2=shape.chi2_fwd(batch, p))
        if case["want"] == "normal":
            return shape.chi2_bwd(batch, p, want_normal=True)
        chi2 = shape.sersic_chi2(p, batch)
        grad, = torch.autograd.grad(chi2, p, state["upstream"])
        return dict(chi2=chi2.detach(), grad=grad)
    if kind == "frames":
        frames = state["frames"]
        d = shape.frame_detect(frames)
        batch = shape.frame_cut(frames, d["box"], state["sigma"], out=state["cut"])
        return dict(d, stamps=batch.pixels, offsets=batch.offsets, sides=batch.sides)
    batch = state["batch"]
    rec0, _, _ = shape.centroid(batch, state["opts"])
    rec, _, _ = shape.moments(batch, rec0, state["opts"])
    fit = shape.fit_queue_static(batch, rec=rec, opts=state["opts"], cfg=state["cfg"],
                                 out=state["out"])
    return dict(fit, moments=rec)


def work(case):
    kind, n = case["kind"], case["n"]
    size = 2 if case.get("f16") else 4
    if kind == "frames":
        px = n * case["height"] * case["width"]
        # one read of each frame, the cut-outs (6 r50 a side, about 24) out
        return {"bytes": px * size + n * (24 * 24 * 8 + 48), "flops": 3 * px}
    side = case.get("side", 0)
    px = n * (side * side if side else 3873)   # mean side^2 of exp U(ln 16, ln 128)
    if kind == "chi2":
        flops = {"value": 20, "autograd": 39, "normal": 86}[case["want"]]
        out = {"value": 4, "autograd": 4 + 32 + 32 + 4, "normal": 4 + 32 + 32 + 144}[case["want"]]
        return {"bytes": px * size + n * out, "flops": flops * px}
    steps = 14 * CENTROID_STEPS + 35 * MOMENT_STEPS
    if kind == "stars":
        return {"bytes": px * size + n * 112, "flops": px * (steps + 11 * STAR_STEPS)}
    return {"bytes": px * size + n * 150, "flops": px * (steps + 82 * SWEEPS)}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
def _b_exact(n):
    """b(n) of P(2n, b) = 1/2 by Newton's method on the incomplete gamma function."""
    b = _b(n)
    for _ in range(6):
        f = torch.special.gammainc(2 * n, b) - 0.5
        b = b - f * torch.exp(b + torch.lgamma(2 * n) - (2 * n - 1) * torch.log(b))
    return b


def _chi2_exact(case, seed):
    s = prepare(case, seed)
    batch, n, side = s["batch"], case["n"], case["side"]
    p = s["params"].detach().double()
    b = _b_exact(p[:, 5])
    h = 2e-3   # db/dn by a five-point rule
    db = (8 * (_b_exact(p[:, 5] + h) - _b_exact(p[:, 5] - h))
          - (_b_exact(p[:, 5] + 2 * h) - _b_exact(p[:, 5] - 2 * h))) / (12 * h)
    c = torch.arange(side, device=DEV, dtype=torch.float64)
    x, y = c.repeat(side)[None], c.repeat_interleave(side)[None]
    chi2 = torch.empty(n, device=DEV, dtype=torch.float64)
    jtr = torch.empty(n, 8, device=DEV, dtype=torch.float64)
    jtj = torch.empty(n, 36, device=DEV, dtype=torch.float64)
    pix = batch.pixels.reshape(n, -1)
    step = max(1, (1 << 23) // (side * side))
    for a in range(0, n, step):
        q = p[a:a + step].T[:, :, None]
        d = pix[a:a + step].double()
        if batch.scale is not None:
            d = d * batch.scale[a:a + step, None].double()
        r2 = _r2(x, y, q)
        ba, dba = b[a:a + step, None], db[a:a + step, None]
        lr = 0.5 * torch.log(r2) - torch.log(q[4])          # ln(R / Re)
        t = torch.exp(lr / q[5])
        m0 = torch.exp(-ba * t)
        r = (d - (q[6] * m0 + q[7]))
        # dm/dR^2 times dR^2/d(x0, y0, e1, e2)
        k = -q[6] * m0 * ba * t / (2 * q[5] * r2)
        ux, uy = x - q[0], y - q[1]
        vx, vy = (1 - q[2]) * ux - q[3] * uy, -q[3] * ux + (1 + q[2]) * uy
        D = 1 - q[2] ** 2 - q[3] ** 2
        J = [k * 2 / D * (-(1 - q[2]) * vx + q[3] * vy),
             k * 2 / D * (q[3] * vx - (1 + q[2]) * vy),
             k * 2 / D * (-ux * vx + uy * vy + q[2] * r2),
             k * 2 / D * (-uy * vx - ux * vy + q[3] * r2),
             q[6] * m0 * ba * t / (q[5] * q[4]),
             q[6] * m0 * t * (ba * lr / q[5] ** 2 - dba),
             m0, torch.ones_like(m0)]
        i2 = 1 / batch.sigma[a:a + step].double() ** 2
        chi2[a:a + step] = (r * r).sum(1) * i2
        for u in range(8):
            jtr[a:a + step, u] = (J[u] * r).sum(1) * i2
        if case["want"] == "normal":
            e = 0
            for u in range(8):
                for v in range(u, 8):
                    jtj[a:a + step, e] = (J[u] * J[v]).sum(1) * i2
                    e += 1
    if case["want"] == "value":
        return dict(chi2=chi2)
    if case["want"] == "normal":
        return dict(grad=-2 * jtr, chi2=chi2, jtj=jtj, jtr=jtr)
    return dict(chi2=chi2, grad=-2 * jtr * s["upstream"].double()[:, None])


def _frames_exact(case, seed):
    """info = (sky, r50, F) and the peak; the box follows from them."""
    s = prepare(case, seed)
    fr, (n, h, w) = s["frames"], (case["n"], case["height"], case["width"])
    info = torch.empty(n, 3, device=DEV, dtype=torch.float64)
    y, x = torch.arange(h, device=DEV)[:, None], torch.arange(w, device=DEV)[None, :]
    for i in range(n):
        f = fr.pixels[i].double()
        if fr.scale is not None:
            f = f * fr.scale[i].double()
        edge = f[0].sum() + f[-1].sum() + f[1:-1, 0].sum() + f[1:-1, -1].sum()
        sky = edge / (2 * w + 2 * h - 4)
        k = int(torch.nonzero(f.reshape(-1) == f.max())[0])   # the first among equals
        f = f - sky
        total = f.sum()
        ring = torch.ceil(torch.sqrt(((y - k // w) ** 2 + (x - k % w) ** 2).double()))
        ring = ring.long().clamp(min=1)
        curve = torch.zeros(h + w, device=DEV, dtype=torch.float64)
        curve.index_add_(0, ring.reshape(-1), f.reshape(-1))
        curve = torch.cumsum(curve, 0)
        hit = (curve >= total / 2) & (torch.arange(h + w, device=DEV) > 0)
        r = int(torch.argmax(hit.int()))
        r50 = r - 1 + (total / 2 - curve[r - 1]) / (curve[r] - curve[r - 1])
        info[i] = torch.stack([sky, r50, total])
    return dict(info=info, peak=None, box=None, status=None, stamps=None, offsets=None, sides=None)


def exact(case, seed):
    if case["kind"] == "chi2":
        return _chi2_exact(case, seed)
    if case["kind"] == "frames" and case["n"] <= 4096:
        return _frames_exact(case, seed)
    # the other calls stop an iteration by a tolerance: where it stops is
    # theirs to say, not a value of its own
    return None
