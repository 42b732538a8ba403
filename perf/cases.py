"""Timed cases: the calls a program makes of the deconvolution library.

A case is one call (or the few calls that belong together) of the Python
binding on inputs made on the GPU from a seed: sparse specimens of Gaussian
blobs over a background, seen through rotated anisotropic Gaussian PSFs, with
Poisson counts.  The sizes are those of the benchmark's workloads, of the
tests, and others of the same ranges; the forms are the ones a program
chooses between:

  plain      a handle on one volume: set the start, n iterations, read back
  batch      one handle on several blocks (time points of one crop)
  blocked    the block-wise form on a volume of any extents
  linear     the padded boundary
  combined   the all-views updates (ML-EM or the geometric mean)
  loss       PSF refinement: loss and gradients in the PSFs and the start
  layer      the autograd layer: recorded forward, then its backward
  noalloc    the one-call run without allocations, set-up included

Volumes are (nz, ny, nx) float32.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1308_0730_amd import autograd, mvd

DEV = "cuda"

def _case(name, form, dims, views, psf, variant, n, weights=False, lam=0.0, mean="", blocks=1):
    return dict(name=name, form=form, nx=dims[0], ny=dims[1], nz=dims[2], views=views, kx=psf[0], ky=psf[1],
                kz=psf[2], variant=variant, n=n, weights=weights, lam=lam, mean=mean, blocks=blocks)


def listed():
    return [
        # a preview-sized crop, two opposite views: launches and latency count
        _case("tiny64_eff", "plain", (64, 64, 64), 2, (17, 17, 17), "eff", 5),
        # one region of interest, four views, plain Richardson-Lucy steps
        _case("cube128_rl", "plain", (128, 128, 128), 4, (25, 25, 25), "rl", 10),
        # a cropped acquisition with uneven extents, partial overlap and noise control
        _case("ragged_150x108x90", "plain", (150, 108, 90), 3, (15, 17, 21), "opt2", 6, True, 0.0006),
        # a whole embryo, six views, weights and regularisation
        _case("embryo_512x512x256", "plain", (512, 512, 256), 6, (31, 31, 41), "opt1", 2, True, 0.0006),
        # the time points of one crop processed together
        _case("batch8_144x120x96_eff", "batch", (144, 120, 96), 4, (17, 17, 17), "eff", 5, blocks=8),
        # a volume that fits no transform, processed in blocks
        _case("blocked_820x535x172", "blocked", (820, 535, 172), 4, (21, 21, 31), "opt2", 2),
        # views that end at the volume's border: the padded boundary
        _case("linear_216x200x100", "linear", (216, 200, 100), 4, (21, 21, 31), "opt1", 3, True, 0.0006),
        # the classic all-views updates
        _case("mlem_128", "combined", (128, 128, 128), 4, (25, 25, 25), "rl", 8, mean="arithmetic"),
        # one step of a PSF refinement
        _case("refine_128_rl", "loss", (128, 128, 128), 4, (25, 25, 25), "rl", 4),
        # the deconvolution as a layer of a larger program, uneven extents
        _case("layer_96x80x72_eff", "layer", (96, 80, 72), 3, (13, 13, 17), "eff", 3),
        # a serving loop that may not allocate: set-up and run in one call
        _case("noalloc_96x80x64_opt1", "noalloc", (96, 80, 64), 3, (11, 11, 15), "opt1", 10),
    ]


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


def _pick(rng, lo, hi, even=False):
    """A 5-smooth extent of [lo, hi], spread over its logarithm."""
    t = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    ok = [n for n in range(lo, hi + 1) if _smooth(n // 2 if even else n) and not (even and n % 2)]
    return min(ok, key=lambda n: abs(n - t))


def _psf(rng, dims, cap):
    return [2 * rng.randint(2, (min(cap, d) - 1) // 2) + 1 for d in dims]


def draw(rng):
    form = rng.choice(["plain", "plain", "plain", "batch", "blocked", "linear", "combined", "loss", "layer", "noalloc"])
    variant = rng.choice(["rl", "eff", "opt1", "opt2"])
    views = rng.randint(1, 6)
    weights = rng.random() < 0.5
    lam = rng.choice([0.0, 0.0006])
    mean, blocks = "", 1
    if form == "plain":
        dims = [_pick(rng, 24, 512, True), _pick(rng, 24, 400), _pick(rng, 16, 256)]
        n = rng.randint(1, 8)
    elif form == "batch":
        dims = [_pick(rng, 48, 256, True), _pick(rng, 48, 256), _pick(rng, 48, 160)]
        blocks, n = rng.randint(2, 8), rng.randint(2, 5)
        weights = False
    elif form == "blocked":
        dims = [rng.randint(90, 700), rng.randint(90, 500), rng.randint(40, 150)]
        views, n = rng.randint(2, 4), rng.randint(1, 2)
    elif form == "linear":
        dims = [_pick(rng, 60, 256, True), _pick(rng, 50, 216), _pick(rng, 30, 108)]
        n = rng.randint(1, 4)
    elif form == "combined":
        dims = [_pick(rng, 32, 256, True), _pick(rng, 32, 256), _pick(rng, 32, 128)]
        weights, mean, n = False, rng.choice(["arithmetic", "geometric"]), rng.randint(2, 8)
    elif form in ("loss", "layer"):
        dims = [_pick(rng, 32, 160, True), _pick(rng, 32, 160), _pick(rng, 24, 128)]
        views, n = rng.randint(1, 4), rng.randint(1, 4)
    else:
        dims = [_pick(rng, 32, 96, True), _pick(rng, 32, 96), _pick(rng, 24, 72)]
        views, n = rng.randint(1, 3), rng.randint(2, 10)
    cap = {"loss": 25, "layer": 17, "noalloc": 15}.get(form, 31)
    psf = _psf(rng, dims, min(cap, 17) if variant == "eff" else cap)
    c = _case("", form, dims, views, psf, variant, n, weights, lam, mean, blocks)
    del c["name"]
    while work(c)["flops"] > 2.2e11 and c["n"] > 1:
        c["n"] -= 1
    while work(c)["flops"] > 2.2e11 and c["views"] > 1:
        c["views"] -= 1
    return c


def _dims(case):
    """Extents of the case's blocks (one for most forms)."""
    return [(case["nx"], case["ny"], case["nz"])] * case["blocks"]


def _angles(n):
    return [360.0 * v / n if n > 4 else (90.0 if n == 2 else 45.0) * v for v in range(n)]


def _cov(theta, sxy, sz):
    t = math.radians(theta)
    R = np.array([[math.cos(t), 0, math.sin(t)], [0, 1, 0], [-math.sin(t), 0, math.cos(t)]])
    return R @ np.diag([sxy ** 2, sxy ** 2, sz ** 2]) @ R.T


def _gauss(psf, theta, sxy, sz):
    kx, ky, kz = psf
    z, y, x = np.meshgrid(np.arange(kz) - (kz - 1) / 2, np.arange(ky) - (ky - 1) / 2, np.arange(kx) - (kx - 1) / 2,
                          indexing="ij")
    d = np.stack([x, y, z], -1)
    g = np.exp(-0.5 * np.einsum("...i,ij,...j->...", d, np.linalg.inv(_cov(theta, sxy, sz)), d))
    return (g / g.sum()).astype(np.float32)


def _volumes(case, dims, seed):
    """Views (Poisson counts), PSFs and weights of one volume."""
    nx, ny, nz = dims
    rng = np.random.default_rng([seed, nx, ny, nz])
    n = max(1, min(20000, round(40 * nx * ny * nz / 64 ** 3)))
    at = np.unique(rng.integers(0, nx * ny * nz, n))
    mass = rng.uniform(200.0, 1000.0, at.size) * 180.0
    pts = torch.zeros(nx * ny * nz, device=DEV)
    pts[torch.from_numpy(at).to(DEV)] = torch.from_numpy(mass.astype(np.float32)).to(DEV)
    S = torch.fft.rfftn(pts.view(nz, ny, nx))
    f = [2 * math.pi * torch.fft.fftfreq(m, device=DEV) for m in (nz, ny)]
    fz, fy, fx = f[0].view(-1, 1, 1), f[1].view(1, -1, 1), 2 * math.pi * torch.fft.rfftfreq(nx, device=DEV).view(1, 1, -1)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    sxy, sz = 1.0 + 0.2 * rng.uniform(), 3.5 + 0.5 * rng.uniform()
    views, psfs, ws = [], [], []
    for th in _angles(case["views"]):
        C = _cov(th, sxy, sz) + 4.0 * np.eye(3)
        q = C[0, 0] * fx * fx + C[1, 1] * fy * fy + C[2, 2] * fz * fz + 2 * C[0, 2] * fx * fz
        v = torch.fft.irfftn(S * torch.exp(-0.5 * q), s=(nz, ny, nx)).clamp_(min=0).add_(5.0)
        views.append(torch.poisson(v, generator=gen))
        psfs.append(torch.from_numpy(_gauss((case["kx"], case["ky"], case["kz"]), th, sxy, sz)))
    if case["weights"]:
        # each view sees the half-space on its detection side and a band
        # beyond it, falling off over a cosine ramp; summed weights limited
        # to the minimal overlap
        z = torch.arange(nz, device=DEV).view(-1, 1) - (nz - 1) / 2
        x = torch.arange(nx, device=DEV).view(1, -1) - (nx - 1) / 2
        band, ramp = 0.12 * (nx + nz) / 2, 0.06 * (nx + nz) / 2
        for th in _angles(case["views"]):
            t = math.radians(th)
            u = ((x * math.sin(t) + z * math.cos(t) + band + ramp) / ramp).clamp(0, 1)
            ws.append(0.5 - 0.5 * torch.cos(math.pi * u))
        tot = torch.stack(ws).sum(0)
        m = torch.where(tot > 0, tot, tot.max()).min()
        k = torch.clamp(m / tot.clamp(min=1e-12), max=1.0)
        ws = [(w * k).clamp(0, 1).view(nz, 1, nx).expand(nz, ny, nx).contiguous() for w in ws]
    return views, psfs, ws or None


def _inputs(case, seed):
    out = []
    for b, dims in enumerate(_dims(case)):
        views, psfs, ws = _volumes(case, dims, 1000 * int(seed) + b)
        s = sum(float(v.double().mean()) for v in views) / len(views)
        # the start: an earlier, smoother estimate of the same specimen
        start = torch.nn.functional.avg_pool3d(sum(views)[None, None] / len(views), 5, 1, 2)[0, 0].contiguous()
        out.append((views, psfs, ws, start.clamp_(min=0.1 * s)))
    return out


class _State(dict):
    pass


def prepare(case, seed):
    form = case["form"]
    ins = _inputs(case, seed)
    st = _State(case=case, start=[i[3] for i in ins])
    if form == "noalloc":
        v, p, w, start = ins[0]
        st.update(views=v, psfs=[q.to(DEV) for q in p], weights=w, out=torch.empty_like(start))
    elif form == "batch":
        st["d"] = mvd.Deconvolver.batch([(v, [q.to(DEV) for q in p], w) for v, p, w, _ in ins], lam=case["lam"])
    elif form == "blocked":
        v, p, w, _ = ins[0]
        st["d"] = mvd.Deconvolver.blocked(v, [q.to(DEV) for q in p], w, lam=case["lam"])
    else:
        v, p, w, start = ins[0]
        st["d"] = mvd.Deconvolver(v, [q.to(DEV) for q in p], w, lam=case["lam"],
                                  boundary="linear" if form == "linear" else "circular")
        if form in ("loss", "layer"):
            st["psfs"] = [q.clone().requires_grad_(True) for q in p]
            st["psi0"] = start.clone().requires_grad_(True)
            st["seed"] = v[0] / v[0].mean()
    return st


def run(state):
    case = state["case"]
    form, n, var = case["form"], case["n"], case["variant"]
    if form == "noalloc":
        return mvd.iterate_noalloc(state["views"], state["psfs"], n, var, weights=state["weights"], lam=case["lam"],
                                   psi0=state["start"][0], out=state["out"])
    d = state["d"]
    if form in ("loss", "layer"):
        args = [state["psi0"]] + state["psfs"]
        if form == "loss":
            loss = autograd.MVDLoss.apply(d, (n, var), *args)
            return [loss.detach().to(torch.float32), torch.autograd.grad(loss, args)]
        psi = autograd.MVDDeconvolve.apply(d, (n, var), *args)
        return [psi.detach(), torch.autograd.grad(psi, args, state["seed"])]
    for b, start in enumerate(state["start"]):
        d.set_estimate(start, b)
    if form == "combined":
        d.iterate_combined(n, var, case["mean"])
    else:
        d.iterate(n, var)
    return [d.estimate(b) for b in range(len(state["start"]))]


def work(case):
    """Inputs read once and outputs written once; the operations of the 5 N
    log2 N count of each convolution's two real transforms (half of a complex
    one's) and the pointwise steps, per voxel and view-update."""
    V = sum(a * b * c for a, b, c in _dims(case))
    N, n = case["views"], case["n"]
    grad = case["form"] in ("loss", "layer")
    vols = 2 + N * (2 if case["weights"] else 1) + (1 if grad else 0)
    lg = math.log2(max(2.0, V / len(_dims(case))))
    per = 2 * (2 * 2.5 * lg + 6) + 12
    return {"bytes": 4.0 * V * vols + 4.0 * N * case["kx"] * case["ky"] * case["kz"],
            "flops": per * V * N * n * (3 if grad else 1)}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the method's equations.

def _odd(p):
    return torch.nn.functional.pad(p, [q for s in reversed(p.shape) for q in (0, 1 - s % 2)])


def _flip(p):
    return torch.flip(p, (0, 1, 2))


def _full(a, b):
    """Linear convolution of two small kernels."""
    s = [m + n - 1 for m, n in zip(a.shape, b.shape)]
    return torch.fft.irfftn(torch.fft.rfftn(a, s=s) * torch.fft.rfftn(b, s=s), s=s)


def _crop(a, shape):
    o = [(m - n) // 2 for m, n in zip(a.shape, shape)]
    pad = [q for m, n in zip(reversed(a.shape), reversed(shape)) for q in (max(0, (n - m) // 2),) * 2]
    if any(pad):
        return _crop(torch.nn.functional.pad(a, pad), shape)
    return a[tuple(slice(i, i + n) for i, n in zip(o, shape))]


def _back(P, v, variant):
    """Back-projection kernel of view v."""
    K = _flip(P[v])
    if variant == "opt2":
        K = K ** len(P)
    elif variant != "rl":
        for w in range(len(P)):
            if w != v:
                a = _full(_flip(P[v]), P[w])
                if variant == "eff":
                    a = _full(a, _flip(P[w]))
                K = K * _crop(a, P[v].shape)
    return K / K.sum()


def _spectrum(K, shape):
    """Transform of a centred kernel wrapped around the grid."""
    full = torch.nn.functional.pad(K, [q for n, k in zip(reversed(shape), reversed(K.shape)) for q in (0, n - k)])
    return torch.fft.rfftn(torch.roll(full, [-(k // 2) for k in K.shape], (0, 1, 2)))


def _conv(x, H):
    return torch.fft.irfftn(torch.fft.rfftn(x) * H, s=x.shape)


def _tik(u, lam):
    return 2 * u / (1 + torch.sqrt(1 + 4 * lam * u)) if lam else u


def _deconvolve(psi, views, psfs, ws, s, case, nodata=None):
    lam, eps, var = case["lam"] / s, 1e-6 * s, case["variant"]
    P = [_odd(p) for p in psfs]
    P = [p / p.sum() for p in P]
    N = len(P)
    H = [_spectrum(p, psi.shape) for p in P]
    B = [_spectrum(_back(P, v, var), psi.shape) for v in range(N)]
    for _ in range(case["n"]):
        acc = None
        for v in range(N):
            q = views[v].double() / _conv(psi, H[v]).clamp(min=eps)
            if nodata is not None:
                q = torch.where(nodata, torch.ones_like(q), q)
            c = _conv(q, B[v]).clamp(min=0)
            if case["mean"]:
                acc = c if acc is None else (acc * c if case["mean"] == "geometric" else acc + c)
                continue
            t = _tik(psi * c, lam)
            psi = t if ws is None else psi + ws[v].double() * (t - psi)
        if case["mean"]:
            psi = _tik(psi * (acc ** (1.0 / N) if case["mean"] == "geometric" else acc / N), lam)
    return psi, H


def exact(case, seed):
    form = case["form"]
    outs = []
    for views, psfs, ws, start in _inputs(case, seed):
        psfs = [p.to(DEV).double() for p in psfs]
        s = sum(float(v.double().mean()) for v in views) / len(views)
        psi = start.double()
        if form == "linear":
            # the volume plus one PSF radius, rounded up to a grid
            u = psi.shape
            r = [max(k // 2 for k in ks) for ks in zip(*[tuple(m | 1 for m in p.shape) for p in psfs])]
            g = []
            for m, k, even in zip(u, r, (False, False, True)):
                t = m + 2 * k
                while not _smooth(t) or (even and t % 2):
                    t += 1
                g.append(t)
            box = tuple(slice(k, k + m) for k, m in zip(r, u))

            def put(x, fill):
                out = torch.full(g, float(fill), dtype=torch.float64, device=DEV)
                out[box] = x
                return out

            none = put(torch.zeros_like(psi), 1.0) > 0
            wv = None if ws is None else [put(w.double(), 1.0) for w in ws]
            got, _ = _deconvolve(put(psi, s), [put(v.double(), 0.0) for v in views], psfs, wv, s, case, none)
            outs.append(got[box].contiguous())
        elif form in ("loss", "layer"):
            psi.requires_grad_(True)
            for p in psfs:
                p.requires_grad_(True)
            got, H = _deconvolve(psi, views, psfs, ws, s, case)
            if form == "loss":
                loss = sum(((_conv(got, h) - v.double()) ** 2).sum() for h, v in zip(H, views))
                return [loss.detach(), torch.autograd.grad(loss, [psi] + psfs)]
            return [got.detach(), torch.autograd.grad(got, [psi] + psfs, (views[0] / views[0].mean()).double())]
        else:
            outs.append(_deconvolve(psi, views, psfs, ws, s, case)[0])
    return outs[0] if form == "noalloc" else outs
