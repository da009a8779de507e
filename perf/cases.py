"""Measured cases: the work a user of this framework has it do, through its public entry points.

Every case is one of six kinds of call, at sizes taken from the repository's own workloads and tests or between them:

  iterate   a resident job (device buffers, one `em.Context`) advanced by a few EM iterations from a given iterate
  tol       the same through the stopping rule (`iterate_tol`), with the FP64 log-likelihood traced
  job       a whole job from its exposures: set-up, iterations with the FP64 log-likelihood traced, final log-likelihood
  fine      the super-resolution run on up-sampled exposures: `em.upsample`, then a whole job on the fine grid
  noalloc   a whole job in one call that allocates nothing (`em.run_noalloc`)
  psf       the super-resolved PSFs of a job's frames (`em.psf_fit`)
  serve     a burst of jobs of uneven size through a running `em.Server`, host arrays in, host arrays out

The data are sky-subtracted exposures of point sources and extended galaxies with per-pixel variances and masked pixels, as
`paper_2302_05804_amd/synth.py` describes them, drawn on the GPU so that they are quick to make.
"""
import math
import random

import numpy as np
import torch

from paper_2302_05804_amd import em

PRECISIONS = {"fp32": em.FP32, "bf16": em.BF16_SPLIT, "fp16": em.FP16_SPLIT}


def _case(kind, n=0, h=0, w=0, k=43, sr=1, prec="fp32", nu=0.0, iters=4, **more):
    return dict(kind=kind, n=n, h=h, w=w, k=k, sr=sr, prec=prec, nu=nu, iters=iters, **more)


def listed():
    return [
        # the oracle-size job: a cut-out around one object, where launches and host work count
        dict(_case("job", 4, 128, 128, 15, prec="fp32", iters=30), name="cutout-job-fp32"),
        # a small odd cut-out from a caller that may not allocate
        dict(_case("noalloc", 5, 147, 211, 43, prec="fp16", iters=4), name="cutout-noalloc-fp16"),
        # the plain single-precision job on one detector tile
        dict(_case("iterate", 8, 1024, 1024, 43, prec="fp32", iters=4), name="tile-fp32"),
        # single precision on a deep stack of half-size exposures
        dict(_case("iterate", 33, 2048, 2048, 43, prec="fp32", iters=1), name="stack-fp32"),
        # the headline: a stack of full exposures in the fastest form
        dict(_case("iterate", 33, 4096, 4096, 43, prec="fp16", iters=4, tune=True), name="stack-full-fp16"),
        # the more exact split form, on an odd mosaic
        dict(_case("iterate", 33, 1999, 2111, 43, prec="bf16", iters=4, tune=True), name="stack-odd-bf16"),
        # super-resolution x2 with down-sampling in the model, all frames of a visit
        dict(_case("iterate", 16, 2048, 2048, 43, sr=2, prec="fp16", iters=4, tune=True), name="superres-fp16"),
        # super-resolution in single precision, an odd frame count and size
        dict(_case("iterate", 9, 701, 1022, 43, sr=2, prec="fp32", iters=2), name="superres-odd-fp32"),
        # exposures with unflagged satellite trails: Student-t noise, run to a tolerance
        dict(_case("tol", 12, 1500, 1777, 43, prec="fp16", nu=4.0, iters=4), name="trails-tol-fp16"),
        # super-resolution on up-sampled exposures, from raw exposures to the result
        dict(_case("fine", 16, 512, 512, 43, prec="fp16", iters=4), name="upsampled-job-fp16"),
        # the super-resolved PSFs of a visit's frames
        dict(_case("psf", 16, 43, 43, 43, iters=2000), name="psf-fit"),
        # serving: a burst of jobs of uneven size, depth and factor
        dict(_case("serve", 8, 256, 768, 43, prec="fp16", iters=6, mix=4), name="serve-burst-fp16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["iterate"] * 6 + ["job", "job", "tol", "fine", "noalloc", "psf", "serve"])
    prec = rng.choice(["fp32", "bf16", "fp16", "fp16"])
    if kind == "psf":
        side = rng.choice([25, 31, 43])
        return _case("psf", _log(rng, 4, 33), side, side, rng.choice([25, 43]), iters=_log(rng, 300, 2000))
    if kind == "serve":
        return _case("serve", _log(rng, 4, 12), 256, _log(rng, 300, 900), 43, prec=rng.choice(["fp16", "bf16"]),
                     iters=_log(rng, 4, 8), mix=rng.randrange(1 << 16))
    if kind == "noalloc":
        return _case("noalloc", rng.randint(2, 8), _log(rng, 48, 320), _log(rng, 48, 320), rng.choice([15, 31, 43, 43]),
                     prec=prec, iters=rng.randint(2, 5))
    if kind == "fine":
        return _case("fine", rng.randint(4, 20), _log(rng, 128, 700), _log(rng, 128, 700), 43, prec=prec,
                     iters=rng.randint(2, 4))
    if kind == "job" and rng.random() < 0.4:
        return _case("job", rng.randint(2, 8), _log(rng, 64, 256), _log(rng, 64, 256), 15, prec=prec,
                     iters=rng.randint(3, 6) if prec == "fp16" else rng.randint(8, 30))
    sr = rng.choice([1, 1, 2])
    nu = 4.0 if kind == "tol" and rng.random() < 0.7 else 0.0
    # frame pixels per pass: up to the full stack in the split forms, a quarter of its time in single precision
    most = 9e7 if prec == "fp32" else 3e8
    n = rng.randint(4, 33)
    side = min(2100.0, math.sqrt(most / (n * 4)))
    h, w = _log(rng, 200, side), _log(rng, 200, side)
    return _case(kind, n, h, w, rng.choice([31, 43, 43, 43]), sr=sr, prec=prec, nu=nu,
                 iters=rng.randint(2, 4) if prec != "fp32" else rng.randint(1, 3),
                 **({"tune": True} if kind == "iterate" and prec != "fp32" else {}))


# ---------------------------------------------------------------- data


def _psfs(n, k, sr, rnd, fwhm=(3.0, 7.0)):
    """Elliptical Moffat PSFs with unit sums, 64-bit values rounded once to 32 bits."""
    c = (k - 1) / 2.0
    yy, xx = np.mgrid[0:k, 0:k].astype(np.float64)
    out = np.empty((n, k, k), np.float32)
    for t in range(n):
        f = rnd.uniform(*fwhm) * sr * (0.5 if k < 25 else 1.0)
        beta, q, th = rnd.uniform(2.5, 4.5), 1.0 - rnd.uniform(0.0, 0.3), rnd.uniform(0.0, math.pi)
        dy, dx = (rnd.random(), rnd.random()) if sr == 2 else (0.0, 0.0)
        a = f / (2.0 * math.sqrt(2.0 ** (1.0 / beta) - 1.0))
        u = math.cos(th) * (xx - c - dx) + math.sin(th) * (yy - c - dy)
        v = -math.sin(th) * (xx - c - dx) + math.cos(th) * (yy - c - dy)
        p = (1.0 + (u * u / q + v * v * q) / (a * a)) ** -beta
        out[t] = p / p.sum()
    return torch.from_numpy(out).cuda()


def _sky(hl, wl, gen):
    """Point sources (flux log-uniform in 1e2..1e5) and galaxies (1e3..1e5) of the density of the repository's recipes."""
    dev = "cuda"
    x = torch.zeros(hl * wl, dtype=torch.float64, device=dev)
    pts, gal = max(4, hl * wl // 524), max(2, hl * wl // 5243)
    at = torch.randint(0, hl * wl, (pts,), generator=gen, device=dev)
    x.index_add_(0, at, torch.exp(torch.rand(pts, generator=gen, device=dev, dtype=torch.float64) * math.log(1e3) + math.log(1e2)))
    r = torch.arange(-16, 17, device=dev, dtype=torch.float64)
    d = torch.sqrt(r[:, None] ** 2 + r[None, :] ** 2).reshape(1, -1)
    re = torch.rand(gal, 1, generator=gen, device=dev, dtype=torch.float64) * 5 + 3
    prof = torch.exp(-1.68 * (d / re - 1.0))
    flux = torch.exp(torch.rand(gal, 1, generator=gen, device=dev, dtype=torch.float64) * math.log(1e2) + math.log(1e3))
    prof = flux * prof / prof.sum(1, keepdim=True)
    cy = torch.randint(0, hl, (gal, 1), generator=gen, device=dev)
    cx = torch.randint(0, wl, (gal, 1), generator=gen, device=dev)
    oy, ox = torch.meshgrid(r.long(), r.long(), indexing="ij")
    py = (cy + oy.reshape(1, -1)).clamp(0, hl - 1)
    px = (cx + ox.reshape(1, -1)).clamp(0, wl - 1)
    x.index_add_(0, (py * wl + px).reshape(-1), prof.reshape(-1))
    return x.view(hl, wl)


def _fast(n):
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1 and n % 2 == 0:
            return n
        n += 1


class _Conv:
    """'Same' zero-filled convolution and its adjoint by the FFT (data, and the 64-bit values of exact())."""

    def __init__(self, h, w, k, dtype):
        self.h, self.w, self.c, self.dtype = h, w, (k - 1) // 2, dtype
        self.s = (_fast(h + k - 1), _fast(w + k - 1))

    def hat(self, a):
        return torch.fft.rfft2(a.to(self.dtype), s=self.s)

    def fwd(self, xh, f):
        z = torch.fft.irfft2(xh * self.hat(f), s=self.s)
        return z[self.c:self.c + self.h, self.c:self.c + self.w]

    def adj(self, r, f):
        z = torch.fft.irfft2(self.hat(r) * self.hat(torch.flip(f, (0, 1))), s=self.s)
        return z[self.c:self.c + self.h, self.c:self.c + self.w]


def _box(z):
    return z.view(z.shape[0] // 2, 2, z.shape[1] // 2, 2).sum((1, 3))


def _exposures(n, h, w, k, sr, seed, nu=0.0):
    """y, v (masked pixels NaN / inf), PSFs, and a positive iterate as a job has after some iterations."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 7919 + 17)
    rnd = random.Random(seed * 31 + 5)
    hl, wl = h * sr, w * sr
    sky = _sky(hl, wl, gen)
    f = _psfs(n, k, sr, rnd)
    conv = _Conv(hl, wl, k, torch.float32)
    xh = conv.hat(sky)
    y = torch.empty((n, h, w), dtype=torch.float32, device="cuda")
    v = torch.empty_like(y)
    blurred = None
    for t in range(n):
        m = conv.fwd(xh, f[t])
        if t == 0:
            blurred = m.clamp_min(0.0)
        m = (_box(m) if sr == 2 else m).clamp_min(0.0)
        v[t] = m + rnd.uniform(50.0, 500.0)
        y[t] = m + torch.sqrt(v[t]) * torch.randn((h, w), generator=gen, device="cuda")
        if nu:  # an unflagged satellite trail
            rows = torch.arange(h, device="cuda")
            cols = ((rows * rnd.uniform(-1.0, 1.0)).long() + rnd.randrange(w)) % w
            y[t][rows, cols] += rnd.uniform(20.0, 200.0) * torch.sqrt(v[t][rows, cols])
        mask = torch.rand((h, w), generator=gen, device="cuda") < 0.008
        mask[:, rnd.randrange(w)] = True
        y[t][mask] = float("nan")
        v[t][mask] = float("inf")
    faint = torch.exp(torch.rand((hl, wl), generator=gen, device="cuda") * math.log(1e3) + math.log(1e-2))
    x0 = (0.4 * sky.float() + 0.6 * blurred + faint).contiguous()
    return y, v, f, x0


def _problem(c):
    return em.Problem.make(c["n"], c["h"], c["w"], c["k"], sr=c["sr"], precision=PRECISIONS[c["prec"]], nu=c["nu"])


def _burst(c):
    """Shapes of a burst: side log-uniform in [h, w] (a multiple of 32), 4..12 frames, factor 1 or 2."""
    rnd = random.Random(c["mix"])
    jobs = []
    for _ in range(c["n"]):
        side = max(64, 32 * (_log(rnd, c["h"], c["w"]) // 32))
        jobs.append(dict(n=rnd.randint(4, 12), h=side, w=side, k=c["k"], sr=rnd.choice([1, 2]), prec=c["prec"], nu=0.0,
                         iters=rnd.randint(c["iters"] // 2, c["iters"])))
    return jobs


def _frame_psfs(c, seed):
    return _psfs(c["n"], c["h"], 1, random.Random(seed * 13 + 3), (3.0, 6.0))


def prepare(case, seed):
    c = case
    s = {"case": c}
    if c["kind"] == "psf":
        s["f"] = _frame_psfs(c, seed)
        return s
    if c["kind"] == "serve":
        s["jobs"] = []
        for i, j in enumerate(_burst(c)):
            y, v, f, _ = _exposures(j["n"], j["h"], j["w"], j["k"], j["sr"], seed * 64 + i)
            s["jobs"].append((_problem(j), y.cpu().numpy(), v.cpu().numpy(), f.cpu().numpy(), j["iters"]))
        s["server"] = em.Server(2 << 30, max_slots=16)
        return s
    p = _problem(c)
    y, v, f, x0 = _exposures(c["n"], c["h"], c["w"], c["k"], c["sr"], seed, c["nu"])
    s.update(p=p, y=y, v=v, f=f, x0=x0)
    if c["kind"] == "fine":
        return s
    s["x"] = torch.empty(p.latent_shape, dtype=torch.float32, device="cuda")
    if c["kind"] in ("iterate", "tol"):
        s["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(s["stream"]):
            s["ctx"] = em.Context(p, y, v, f, s["x"], x0=x0, stream=s["stream"])
            if c.get("tune"):
                s["ctx"].autotune(3)
    return s


def _whole_job(p, y, v, f, x, x0, iters):
    ctx = em.Context(p, y, v, f, x, x0=x0)
    trace = ctx.iterate(iters, trace=True)
    ll = ctx.loglik()
    ctx.close()
    return {"x": x, "first": float(trace[0]), "last": ll}


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "psf":
        h, _ = em.psf_fit(state["f"], out_k=c["k"], factor=2, objective=False, steps=c["iters"])
        return h
    if kind == "serve":
        srv = state["server"]
        ids = [srv.submit(*j) for j in state["jobs"]]
        out = []
        for i in ids:
            x, ll = srv.wait(i)
            out.append({"x": x, "ll": ll})
            srv.release(i)
        return out
    if kind == "fine":
        y, v = em.upsample(state["y"], state["v"], 2)
        p = em.Problem.make(c["n"], 2 * c["h"], 2 * c["w"], c["k"], precision=PRECISIONS[c["prec"]])
        x = torch.empty(p.latent_shape, dtype=torch.float32, device="cuda")
        return _whole_job(p, y, v, state["f"], x, None, c["iters"])
    if kind == "job":
        return _whole_job(state["p"], state["y"], state["v"], state["f"], state["x"], state["x0"], c["iters"])
    if kind == "noalloc":
        em.run_noalloc(state["p"], state["y"], state["v"], state["f"], state["x"], c["iters"], x0=state["x0"])
        return state["x"]
    with torch.cuda.stream(state["stream"]):
        state["x"].copy_(state["x0"])
        if kind == "tol":
            done, change, trace = state["ctx"].iterate_tol(c["iters"], 1e-9, check_every=2, trace=True)
            return {"x": state["x"], "done": done, "change": [float(v) for v in change], "ll": [float(v) for v in trace]}
        state["ctx"].iterate(c["iters"])
    return state["x"]


# ---------------------------------------------------------------- work and 64-bit values


def _job_work(n, h, w, k, sr, nu, iters, whole):
    """Each iteration convolves every frame pixel with its PSF once in each direction (Student-t: two adjoints) and has to read the
    weights (and, Student-t, the exposures) and x and the numerator, and write x."""
    keff, px, lat = k + sr - 1, n * h * w, h * w * sr * sr
    convs = 3 if nu else 2
    flops = 2.0 * keff * keff * px * convs * iters
    byts = iters * ((8.0 if nu else 4.0) * px + 12.0 * lat)
    if whole:
        flops += 2.0 * keff * keff * px * 2
        byts += 8.0 * px + 4.0 * lat
    return flops, byts


def work(case):
    c = case
    if c["kind"] == "psf":
        kf, kh = c["h"], c["k"]
        return {"flops": 4.0 * kf * kh * (kf + kh) * c["n"] * c["iters"], "bytes": 4.0 * c["n"] * (kf * kf + kh * kh)}
    if c["kind"] == "serve":
        parts = [_job_work(j["n"], j["h"], j["w"], j["k"], j["sr"], 0.0, j["iters"], True) for j in _burst(c)]
        return {"flops": sum(p[0] for p in parts), "bytes": sum(p[1] for p in parts)}
    up = 2 if c["kind"] == "fine" else 1
    flops, byts = _job_work(c["n"], c["h"] * up, c["w"] * up, c["k"], c["sr"], c["nu"], c["iters"],
                            c["kind"] not in ("iterate", "tol"))
    return {"flops": flops, "bytes": byts}


def _em64(y, v, f, x0, sr, nu, iters):
    """The iteration in 64 bits: (x, the log-likelihood before each update and after the last, the relative changes)."""
    n, h, w = y.shape
    hl, wl = h * sr, w * sr
    conv = _Conv(hl, wl, f.shape[-1], torch.float64)
    f = f.double()

    def weights(t):
        vt = v[t].double()
        seen = torch.isfinite(vt)
        return seen, torch.where(seen, 1.0 / vt, 0.0), torch.where(seen, y[t].double(), 0.0), vt

    def spread(r):
        return r.repeat_interleave(2, 0).repeat_interleave(2, 1) if sr == 2 else r

    if x0 is None:
        su = sum(float(weights(t)[1].sum()) for t in range(n))
        suy = sum(float((weights(t)[1] * weights(t)[2]).sum()) for t in range(n))
        x = torch.full((hl, wl), max(suy / su, 1e-3) / sr ** 2, dtype=torch.float64, device="cuda")
    else:
        x = x0.double()
    num = None
    lls, change = [], []
    for it in range(iters + 1):
        xh = conv.hat(x)
        ll = torch.zeros((), dtype=torch.float64, device="cuda")
        den = torch.zeros_like(x)
        top = torch.zeros_like(x) if nu or num is None else None
        for t in range(n):
            seen, u, yt, vt = weights(t)
            m = conv.fwd(xh, f[t])
            m = _box(m) if sr == 2 else m
            z = u * (yt - m) ** 2
            if nu:
                cst = math.lgamma((nu + 1) / 2) - math.lgamma(nu / 2) - 0.5 * math.log(nu * math.pi)
                ll += torch.where(seen, cst - 0.5 * torch.log(vt) - 0.5 * (nu + 1) * torch.log1p(z / nu), 0.0).sum()
                u = u * (nu + 1) / (nu + z)
            else:
                ll += torch.where(seen, -0.5 * (z + torch.log(2 * math.pi * vt)), 0.0).sum()
            if it < iters:
                den += conv.adj(spread(u * m), f[t])
            if top is not None:
                top += conv.adj(spread(u * yt), f[t])
        lls.append(float(ll))
        if it == iters:
            break
        if top is not None:
            num = top
        new = torch.where(x > 0, x * num.clamp_min(0.0) / den, 0.0)
        change.append(float(torch.linalg.norm(new - x) / torch.linalg.norm(x)))
        x = new
    return x, lls, change


def _psf64(f, kh, factor, steps, sigma=2.0, lam=1e-2, lr=1e-2, decay=1e-2, b1=0.9, b2=0.999, eps=1e-7):
    """Projected Adam on |A h A' - f|^2 + lam |grad h|^2 in 64 bits, A the blurred block sum."""
    n, kf = f.shape[0], f.shape[1]
    f = f.double()
    anchor, ch, rad = factor * ((kf - 1) // 2), (kh - 1) // 2, math.ceil(4 * sigma)
    g = {d: math.exp(-0.5 * (d / sigma) ** 2) for d in range(-rad, rad + 1)}
    tot = sum(g.values())
    a = torch.zeros((kf, kh), dtype=torch.float64)
    for i in range(kf):
        for p in range(kh):
            a[i, p] = sum(g.get(factor * i + q - (anchor + p - ch), 0.0) for q in range(factor)) / tot
    a = a.cuda()
    at = a.t().contiguous()
    fine = torch.arange(kh) + anchor - ch
    ok = (fine >= 0) & (fine < factor * kf)
    idx = (fine.clamp(0, factor * kf - 1) // factor).cuda()
    okd = (ok[:, None] & ok[None, :]).cuda()
    h = torch.where(okd, f[:, idx][:, :, idx].clamp_min(0.0) / factor ** 2, 0.0)
    top = f.abs().amax((1, 2), keepdim=True)
    m, v = torch.zeros_like(h), torch.zeros_like(h)
    for k in range(1, steps + 1):
        rho = a @ h @ at - f
        pad = torch.nn.functional.pad(h, (1, 1, 1, 1))
        lap = 4 * h - pad[:, 2:, 1:-1] - pad[:, :-2, 1:-1] - pad[:, 1:-1, 2:] - pad[:, 1:-1, :-2]
        grad = 2 * (at @ rho @ a) + 2 * lam * lap
        m = b1 * m + (1 - b1) * grad
        v = b2 * v + (1 - b2) * grad * grad
        step = lr * top * decay ** ((k - 1) / (steps - 1) if steps > 1 else 0.0)
        h = (h - step * (m / (1 - b1 ** k)) / (torch.sqrt(v / (1 - b2 ** k)) + eps)).clamp_min(0.0)
    return h


def exact(case, seed):
    c = case
    if c["kind"] == "psf":
        return _psf64(_frame_psfs(c, seed), c["k"], 2, c["iters"])
    if c["kind"] == "serve":
        out = []
        for i, j in enumerate(_burst(c)):
            y, v, f, _ = _exposures(j["n"], j["h"], j["w"], j["k"], j["sr"], seed * 64 + i)
            x, ll, _ = _em64(y, v, f, None, j["sr"], 0.0, j["iters"])
            out.append({"x": x.cpu().numpy(), "ll": ll[-1]})
        return out
    y, v, f, x0 = _exposures(c["n"], c["h"], c["w"], c["k"], c["sr"], seed, c["nu"])
    if c["kind"] == "fine":
        y = (y / 4).repeat_interleave(2, 1).repeat_interleave(2, 2)
        v = (v / 16).repeat_interleave(2, 1).repeat_interleave(2, 2)
        x0 = None
    x, ll, change = _em64(y, v, f, x0, c["sr"], c["nu"], c["iters"])
    if c["kind"] in ("iterate", "noalloc"):
        return x
    if c["kind"] == "tol":
        return {"x": x, "done": None, "change": change, "ll": ll[:-1]}
    return {"x": x, "first": ll[0], "last": ll[-1]}
