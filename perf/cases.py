"""The work that users of this package have it do, as measurable cases.

A case names one operator of ``paper_2101_08072_amd.Plan`` (dirty image, model
visibilities, Hessian, PSF, PSF convolution, a preconditioned forward-backward
step, the wavelet backward step, exact-gradient iterations) and the shape of one
imaging job: image sides, bands, rows, channels, field of view, precision.

``prepare`` makes what an imaging program holds before the call: earth-rotation
uvw tracks, channel frequencies, weights, 10 % flags, a sky of point sources and
blobs, visibilities, the plan and (where the operator needs it) its resident PSF
spectrum.  ``run`` is one call of the operator.  ``exact`` gives the same result in
64 bits from the definitions: the direct Fourier sum, evaluated as matrix products
(the w phase by Chebyshev interpolation in w, to rounding), FFT convolutions, CG,
and the primal-dual iteration.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2101_08072_amd import Options, Plan

C0 = 299792458.0
N_ANT = 64
MIN_SIDE, MAX_SIDE = 64, 4096
EXACT_FLOPS = 2.5e14       # matrix-product work up to which exact() stays within seconds


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _case(op, nx, ny, n_band, n_row, n_chan, **kw):
    c = dict(op=op, nx=nx, ny=ny, n_band=n_band, n_row=n_row, n_chan=n_chan, fov_deg=1.0, uv_frac=0.4,
             precision="fp32", cg_iters=0, pd_iters=0, n_major=0, levels=3, graph=False)
    c.update(kw)
    return c


def listed():
    return [
        # a quick look at a small patch: one short call, launches and latency count
        dict(name="dirty_128_quicklook", **_case("dirty", 128, 128, 1, 4096, 2)),
        # prediction for a small job of a serving mix
        dict(name="degrid_512_serving", **_case("degrid", 512, 512, 1, 20160, 16)),
        # the exact gradient on one band at the usual size (1 degree, 6.4e7 visibilities)
        dict(name="hessian_2048_oneband", **_case("hessian", 2048, 2048, 1, 1_000_000, 64)),
        # a rectangular image whose sides are no powers of two (the padded grids), two bands
        dict(name="dirty_1728x1200_ragged", **_case("dirty", 1728, 1200, 2, 30001, 16)),
        # prediction of a large multi-band job, the short-baseline uv density of 4096^2 images
        dict(name="degrid_4x4096_large", **_case("degrid", 4096, 4096, 4, 500_000, 128, uv_frac=0.2)),
        # a double precision gradient for the accuracy checks and deep-field work
        dict(name="hessian_1024_double", **_case("hessian", 1024, 1024, 1, 25200, 16, precision="fp64")),
        # the PSF and its spectrum, formed once for each job
        dict(name="psf_1024_setup", **_case("psf", 1024, 1024, 1, 125_000, 16)),
        # one application of the approximate Hessian to a small image
        dict(name="conv_512_single", **_case("conv", 512, 512, 1, 20160, 8)),
        # one served iteration of a small job, replayed from its captured graph
        dict(name="fb_512_graph", **_case("fb", 512, 512, 1, 20160, 8, cg_iters=20, graph=True)),
        # one iteration of a large multi-band job: 21 convolutions of 4 x 4096^2 pixels
        dict(name="fb_4x4096_large", **_case("fb", 4096, 4096, 4, 16128, 16, uv_frac=0.2, cg_iters=20)),
        # the backward step with the wavelet prior at the usual size
        dict(name="prox_2048_wavelets", **_case("prox", 2048, 2048, 1, 60480, 16, pd_iters=10)),
        # whole exact-gradient iterations (gradient, CG, backward step) of a small two-band job
        dict(name="clean_512_twoband", **_case("clean", 512, 512, 2, 20160, 16, cg_iters=10, pd_iters=5, n_major=2)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another job of the same ranges: any operator, sides 64 .. 4096 (even, powers of
    two or not, square or not), 1 .. 8 bands, 1e3 .. 2e7 visibilities."""
    op = rng.choice(["dirty", "dirty", "degrid", "degrid", "hessian", "hessian", "psf", "conv", "fb", "prox", "clean"])
    double = rng.random() < 0.15
    most_px = {"psf": 2 ** 22, "prox": 2 ** 22, "clean": 2 ** 20}.get(op, 2 ** 25)   # padded pixels over all bands
    most_side = {"psf": 2048, "prox": 2048, "clean": 1024}.get(op, MAX_SIDE)
    most_vis = {"conv": 2 ** 19, "fb": 2 ** 19, "prox": 2 ** 19, "clean": 2 ** 20, "psf": 2 ** 21}.get(op, 2 * 10 ** 7)
    if double:
        most_px, most_side, most_vis = min(most_px, 2 ** 20), min(most_side, 1024), min(most_vis, 4 * 10 ** 5)
    wavelet = op in ("prox", "clean")
    step = 8 if wavelet else 2                    # sides are even; a multiple of 2^levels under the wavelet prior
    nx = _log_int(rng, MIN_SIDE, most_side)
    nx = 1 << (nx.bit_length() - 1) if rng.random() < 0.4 else max(MIN_SIDE, nx // step * step)
    ny = nx
    if rng.random() < 0.4:
        ny = max(MIN_SIDE, int(nx * rng.uniform(0.5, 1.0)) // step * step)
    pad = (1 << (nx - 1).bit_length()) * (1 << (ny - 1).bit_length())
    n_band = max(1, min(rng.choice([1, 1, 1, 2, 3, 4, 8]), most_px // pad))
    n_chan = n_band * rng.choice([1, 2, 5, 8, 16])
    n_row = max(64, _log_int(rng, 1000, most_vis) // n_chan)
    iters = rng.choice([5, 10, 20])
    return _case(op, nx, ny, n_band, n_row, n_chan, fov_deg=round(rng.uniform(0.3, 2.0), 3),
                 uv_frac=round(rng.uniform(0.2, 0.45), 3), precision="fp64" if double else "fp32",
                 cg_iters=iters if op in ("fb", "clean") else 0, pd_iters=5 if wavelet else 0,
                 n_major=2 if op == "clean" else 0, graph=op == "fb" and rng.random() < 0.5)


# ---------------------------------------------------------------------------
# inputs (from the seed alone)
# ---------------------------------------------------------------------------

def _tracks(rng, case, f_hi):
    """Earth-rotation uvw (metres) of a random 64-antenna array whose longest
    baselines reach uv_frac / cell wavelengths at the highest frequency."""
    cell = math.radians(case["fov_deg"]) / max(case["nx"], case["ny"])
    radius = 0.5 * case["uv_frac"] / cell * C0 / f_hi
    r, th = radius * np.sqrt(rng.uniform(size=N_ANT)), rng.uniform(0, 2 * math.pi, N_ANT)
    east, north = r * np.cos(th), r * np.sin(th)
    a, b = np.triu_indices(N_ANT, 1)
    e, n = east[b] - east[a], north[b] - north[a]
    lat, dec = math.radians(34.0), math.radians(40.0)
    x, z = -n * math.sin(lat), n * math.cos(lat)
    n_t = -(-case["n_row"] // e.size)
    hour = (np.linspace(-4.0, 4.0, n_t) * math.pi / 12.0)[:, None]
    sh, ch = np.sin(hour), np.cos(hour)
    along = ch * x - sh * e
    uvw = np.stack([sh * x + ch * e, math.cos(dec) * z - math.sin(dec) * along, math.sin(dec) * z + math.cos(dec) * along], -1)
    return np.ascontiguousarray(uvw.reshape(-1, 3)[: case["n_row"]]), cell


def _sky(rng, case, dev):
    """Point sources and Gaussian blobs with power-law fluxes, the same in every band."""
    nx, ny = case["nx"], case["ny"]
    img = torch.zeros(nx, ny, dtype=torch.float64, device=dev)
    n_pts = min(500, max(8, nx * ny // 512))
    flux = 1e-3 / (1.0 - rng.uniform(size=n_pts) * 0.999)
    at = (torch.as_tensor(rng.integers(0, nx, n_pts), device=dev), torch.as_tensor(rng.integers(0, ny, n_pts), device=dev))
    img.index_put_(at, torch.as_tensor(flux, device=dev), accumulate=True)
    i, j = torch.arange(nx, device=dev, dtype=torch.float64), torch.arange(ny, device=dev, dtype=torch.float64)
    for _ in range(20):
        ci, cj, s = rng.uniform(0, nx), rng.uniform(0, ny), rng.uniform(2.0, max(3.0, min(20.0, nx / 16)))
        gi, gj = torch.exp(-0.5 * ((i - ci) / s) ** 2), torch.exp(-0.5 * ((j - cj) / s) ** 2)
        img += rng.uniform(0.05, 1.0) / (2 * math.pi * s * s) * gi[:, None] * gj[None, :]
    img = torch.where(img > 1e-9, img, torch.zeros_like(img))
    return img.to(torch.float32).expand(case["n_band"], nx, ny).contiguous()


def _inputs(case, seed):
    """Everything drawn from the seed, as both prepare and exact take it."""
    dev = "cuda"
    real, cplx = (torch.float64, torch.complex128) if case["precision"] == "fp64" else (torch.float32, torch.complex64)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    n_row, n_chan = case["n_row"], case["n_chan"]
    freq = np.linspace(0.9e9, 1.7e9, n_chan)
    uvw, cell = _tracks(rng, case, float(freq[-1]))
    per = n_chan // case["n_band"]
    d = dict(freq=freq, cell=cell, chan_band=(np.arange(n_chan) // per).astype(np.int32), per=per,
             uvw=torch.as_tensor(uvw, device=dev),
             weight=(torch.rand(n_row, n_chan, generator=gen, device=dev) + 0.5).to(real),
             flag=(torch.rand(n_row, n_chan, generator=gen, device=dev) < 0.1).to(torch.uint8),
             sky=_sky(rng, case, dev).to(real))
    if case["op"] in ("dirty", "clean"):
        # a bright source at the phase centre plus receiver noise
        d["vis"] = torch.view_as_complex(torch.randn(n_row, n_chan, 2, generator=gen, device=dev)).to(cplx) + 1.0
    if case["op"] in ("fb", "prox"):
        # the sky with the errors of an iteration: fluxes 10 % low, a little noise
        d["rough"] = 0.9 * d["sky"] + 0.005 * torch.randn(d["sky"].shape, generator=gen, device=dev).to(real)
    return d


def _threshold(case):
    # lambda of the wavelet prior: a thousandth of the PSF peak (1 mJy under the metric)
    return 1e-3 * 0.9 * case["n_row"] * (case["n_chan"] // case["n_band"])


def _norm_bound(psf):
    """An upper bound of the PSF convolution's norm, rounded up to two digits."""
    top = max(float(torch.fft.rfft2(p.to(torch.float64)).abs().max()) for p in psf)
    unit = 10.0 ** (math.floor(math.log10(top)) - 1)
    return math.ceil(1.05 * top / unit) * unit


def prepare(case, seed):
    d = _inputs(case, seed)
    plan = Plan(d["uvw"], d["freq"], d["weight"], d["flag"], d["chan_band"], case["n_band"], case["nx"], case["ny"],
                d["cell"], d["cell"], Options(precision=case["precision"]))
    s = dict(case=case, plan=plan, sky=d["sky"], vis=d.get("vis"))
    op = case["op"]
    if op == "conv":
        plan.make_psf(want_image=False)
    if op in ("fb", "prox", "clean"):
        s["unorm"] = _norm_bound(plan.make_psf())
        s["sigma"] = 1e-3 * s["unorm"]
    if op == "fb":
        s["dirty"] = plan.psf_conv(d["sky"])
        s["x0"] = d["rough"].clamp_min(0)
    if op == "prox":
        s["z"] = d["rough"]
    if op == "clean":
        s["dirty"] = plan.grid(s["vis"])
        s["x0"] = d["sky"]
    if op in ("prox", "clean"):
        s["ws"] = plan.prox_workspace(7)
    if op in ("fb", "clean"):
        s["x"] = torch.empty_like(s["sky"])
    if case["graph"]:
        s["x"].copy_(s["x0"])
        s["graph"] = plan.fb_graph(s["dirty"], s["x"], s["sigma"], 1.0, 1e-3, case["cg_iters"])
    return s


# ---------------------------------------------------------------------------
# one call
# ---------------------------------------------------------------------------

def run(state):
    case, plan, op = state["case"], state["plan"], state["case"]["op"]
    if op == "dirty":
        return plan.grid(state["vis"])
    if op == "degrid":
        return plan.degrid(state["sky"])
    if op == "hessian":
        return plan.hessian(state["sky"])
    if op == "psf":
        return plan.make_psf()
    if op == "conv":
        return plan.psf_conv(state["sky"])
    if op == "prox":
        return plan.prox(state["z"], plan.image(), state["ws"], _threshold(case), 1.0, state["sigma"], state["unorm"],
                         case["pd_iters"], 7, case["levels"])
    x = state["x"]
    x.copy_(state["x0"])           # iterations start from the current model
    if case["graph"]:
        state["graph"].launch()
        return x
    if op == "fb":
        return plan.fb_step(state["dirty"], x, state["sigma"], 1.0, 1e-3, case["cg_iters"])
    return plan.clean(state["dirty"], x, state["ws"], state["sigma"], 1.0, _threshold(case), state["unorm"], case["cg_iters"],
                      case["pd_iters"], case["n_major"], 7, case["levels"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    """Inputs read once, outputs written once; the arithmetic of the fast algorithms
    (W^3 complex x real multiply-adds per visibility, FFTs on the oversampled grid, a
    zero-padded FFT pair per convolution, the wavelet taps)."""
    dbl = case["precision"] == "fp64"
    r, W = (8, 13) if dbl else (4, 7)
    nx, ny, nb, op = case["nx"], case["ny"], case["n_band"], case["op"]
    n, px = case["n_row"] * case["n_chan"], nb * nx * ny
    m = 0.9 * n
    fft = 5.0 * 4 * px * math.log2(4.0 * nx * ny)                 # one complex FFT of the doubled grid
    planes = 1 + (0 if op == "psf" else W)                        # at least W + 1 w-planes hold the data
    nufft = m * (4.0 * W ** 3 + 60.0 * W) + planes * fft
    conv_b, conv_f = (3 + 4) * r * px, fft                        # x, y, the real PSF spectrum; two real FFTs
    taps = 16.0 * sum(2 * k for k in range(1, 7)) * px * 4.0 / 3.0  # six bases, both axes, analysis + synthesis
    if op == "dirty":
        return {"bytes": n * (3 * r + 1) + px * r, "flops": nufft}
    if op == "degrid":
        return {"bytes": n * (2 * r + r + 1) + px * r, "flops": nufft}
    if op == "hessian":
        return {"bytes": n * (r + 1) + 2 * px * r, "flops": 2 * nufft}
    if op == "psf":
        return {"bytes": n * (r + 1) + 4 * px * r, "flops": m * (2.0 * W ** 2 + 40.0 * W) + 4 * fft}
    if op == "conv":
        return {"bytes": conv_b, "flops": conv_f}
    cg = case["cg_iters"]
    fb_b, fb_f = (1 + cg) * conv_b + cg * 5 * r * px, (1 + cg) * conv_f + cg * 10.0 * px
    if op == "fb":
        return {"bytes": fb_b, "flops": fb_f}
    pd_b, pd_f = conv_b + 14 * r * px, conv_f + taps
    if op == "prox":
        return {"bytes": case["pd_iters"] * pd_b, "flops": case["pd_iters"] * pd_f}
    one_b = n * (r + 1) + 2 * px * r + fb_b + case["pd_iters"] * pd_b
    return {"bytes": case["n_major"] * one_b, "flops": case["n_major"] * (2 * nufft + fb_f + case["pd_iters"] * pd_f)}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------

class _Band:
    """One band's entries: coordinates in wavelengths, weights (0 where flagged)."""

    def __init__(self, case, d, b):
        self.sel = slice(b * d["per"], (b + 1) * d["per"])
        scale = torch.as_tensor(d["freq"][self.sel] / C0, device="cuda")
        coord = d["uvw"][:, None, :] * scale[None, :, None]
        live = d["flag"][:, self.sel] == 0
        self.live, (self.u, self.v, self.w) = live, coord[live].unbind(-1)
        self.wt = d["weight"][:, self.sel].to(torch.float64)[live]
        nx, ny = case["nx"], case["ny"]
        self.l = (torch.arange(nx, device="cuda", dtype=torch.float64) - nx // 2) * d["cell"]
        self.m = (torch.arange(ny, device="cuda", dtype=torch.float64) - ny // 2) * d["cell"]
        r2 = self.l[:, None] ** 2 + self.m[None, :] ** 2
        self.n = torch.sqrt(1.0 - r2)
        self.s = -r2 / (1.0 + self.n)                            # n - 1
        # Chebyshev nodes in w: enough for the phase range, to rounding
        lo, hi = float(self.w.min()), float(self.w.max())
        half = max(0.5 * (hi - lo), 1e-9)
        phase = 2 * math.pi * half * 0.5 * float(-self.s.min())
        k = int(math.ceil(1.2 * phase)) + 22
        t = np.cos((np.arange(k) + 0.5) * math.pi / k)
        self.t = torch.as_tensor(t, device="cuda")
        self.bary = torch.as_tensor(((-1.0) ** np.arange(k)) * np.sin((np.arange(k) + 0.5) * math.pi / k), device="cuda")
        self.wk = 0.5 * (lo + hi) + half * t
        self.tw = (self.w - 0.5 * (lo + hi)) / half
        self.sc = 0.5 * float(self.s.min())                      # the phase is split there, which halves its range
        self.flops = 8.0 * self.u.numel() * nx * ny * k
        self.chunk = max(1024, 2 ** 25 // max(nx, ny, k))

    def parts(self, sign):
        for a in range(0, self.u.numel(), self.chunk):
            c = slice(a, a + self.chunk)
            turn = lambda x, y: torch.polar(torch.ones((), device="cuda", dtype=torch.float64).expand(x.numel(), y.numel()).contiguous(),
                                            sign * 2 * math.pi * torch.remainder(x[:, None] * y[None, :], 1.0))  # noqa: E731
            gap = self.tw[c][:, None] - self.t[None, :]
            hit = gap == 0
            q = self.bary / torch.where(hit, torch.ones_like(gap), gap)
            lag = torch.where(hit.any(1, keepdim=True), hit.to(q.dtype), q / q.sum(1, keepdim=True))
            yield c, turn(self.u[c], self.l), turn(self.v[c], self.m), lag, torch.polar(torch.ones_like(self.w[c]), sign * 2 * math.pi * self.w[c] * self.sc)

    def screen(self, k, sign):
        return torch.polar(1.0 / self.n, sign * 2 * math.pi * float(self.wk[k]) * (self.s - self.sc))

    def forward(self, x):
        out = torch.zeros(self.u.numel(), dtype=torch.complex128, device="cuda")
        maps = [x * self.screen(k, -1) for k in range(len(self.wk))]
        for c, a, b, lag, split in self.parts(-1):
            for k, y in enumerate(maps):
                out[c] += lag[:, k] * ((a @ y) * b).sum(1)
            out[c] *= split
        return out

    def adjoint(self, z):
        acc = [torch.zeros_like(self.n, dtype=torch.complex128) for _ in self.wk]
        for c, a, b, lag, split in self.parts(1):
            zc = z[c] * self.wt[c] * split
            at = a.transpose(0, 1).contiguous()
            for k in range(len(acc)):
                acc[k] += at @ ((lag[:, k] * zc)[:, None] * b)
        return sum((acc[k] * self.screen(k, 1)).real for k in range(len(acc)))

    def psf(self, nx, ny, cell):
        l = (torch.arange(2 * nx, device="cuda", dtype=torch.float64) - nx) * cell
        m = (torch.arange(2 * ny, device="cuda", dtype=torch.float64) - ny) * cell
        out = torch.zeros(2 * nx, 2 * ny, dtype=torch.float64, device="cuda")
        for a in range(0, self.u.numel(), self.chunk):
            c = slice(a, a + self.chunk)
            p, q = 2 * math.pi * self.u[c][:, None] * l, 2 * math.pi * self.v[c][:, None] * m
            wt = self.wt[c][:, None]
            out += torch.cos(p).transpose(0, 1).contiguous() @ (wt * torch.cos(q)) - torch.sin(p).transpose(0, 1).contiguous() @ (wt * torch.sin(q))
        out[0] = 0
        out[:, 0] = 0
        return out


def _daubechies(n):
    """Orthonormal minimum-phase low-pass filter with n vanishing moments."""
    roots = np.roots([math.comb(n - 1 + k, k) for k in range(n)][::-1]) if n > 1 else []
    inside = []
    for y in roots:
        b = 1.0 - 2.0 * y
        z = b + np.sqrt(b * b - 1.0 + 0j)
        inside.append(z if abs(z) < 1 else 1.0 / z)
    h = np.real(np.poly(np.array([-1.0] * n + inside, dtype=complex)))
    return h * (math.sqrt(2.0) / h.sum())


def _wave(x, h, axis):
    n = x.shape[axis]
    even = torch.arange(0, n, 2, device=x.device)
    lo = sum(float(h[j]) * x.index_select(axis, (even + j) % n) for j in range(len(h)))
    hi = sum((-1.0) ** j * float(h[-1 - j]) * x.index_select(axis, (even + j) % n) for j in range(len(h)))
    return torch.cat([lo, hi], axis)


def _unwave(c, h, axis):
    n = c.shape[axis]
    even = torch.arange(0, n, 2, device=c.device)
    lo, hi = c.narrow(axis, 0, n // 2), c.narrow(axis, n // 2, n // 2)
    x = torch.zeros_like(c)
    for j in range(len(h)):
        x.index_add_(axis, (even + j) % n, float(h[j]) * lo + (-1.0) ** j * float(h[-1 - j]) * hi)
    return x


def _analysis(x, filters, levels):
    out = [x]
    for h in filters:
        c, nx, ny = x.clone(), x.shape[-2], x.shape[-1]
        for k in range(levels):
            blk = c[:, : nx >> k, : ny >> k]
            c[:, : nx >> k, : ny >> k] = _wave(_wave(blk, h, 2), h, 1)
        out.append(c)
    return torch.stack(out) / math.sqrt(len(out))


def _synthesis(v, filters, levels):
    acc = v[0].clone()
    for h, c in zip(filters, v[1:]):
        c, nx, ny = c.clone(), c.shape[-2], c.shape[-1]
        for k in reversed(range(levels)):
            blk = c[:, : nx >> k, : ny >> k]
            c[:, : nx >> k, : ny >> k] = _unwave(_unwave(blk, h, 1), h, 2)
        acc += c
    return acc / math.sqrt(len(v))


def _prox(conv, z, x, v, sigma, lam, unorm, iters, levels):
    filters = [_daubechies(k) for k in range(1, 7)]
    beta = unorm + sigma
    tau = 0.99 / (0.5 * beta + beta)
    v = torch.zeros((7, *z.shape), dtype=torch.float64, device="cuda") if v is None else v
    for _ in range(iters):
        dx = x - z
        new = (x - tau * (conv(dx) + sigma * dx + _synthesis(v, filters, levels))).clamp_min(0)
        v = v + beta * _analysis(2 * new - x, filters, levels)
        size = v.square().sum(1, keepdim=True).sqrt()
        v = v * (lam / torch.where(size > 0, size, torch.ones_like(size))).clamp_max(1.0)
        x = new
    return x, v


def _cg(conv, g, sigma, iters):
    dot = lambda a, b: (a * b).sum((1, 2), keepdim=True)  # noqa: E731
    y, r = torch.zeros_like(g), g.clone()
    p, rr = r.clone(), dot(g, g)
    for _ in range(iters):
        ap = conv(p) + sigma * p
        alpha = rr / dot(p, ap)
        y += alpha * p
        r -= alpha * ap
        new = dot(r, r)
        p = r + (new / rr) * p
        rr = new
    return y


def exact(case, seed):
    op, nx, ny, nb = case["op"], case["nx"], case["ny"], case["n_band"]
    flat = 4.0 * 0.9 * case["n_row"] * case["n_chan"] / nb * 4.0 * nx * ny * nb
    if op in ("psf", "conv", "fb", "prox", "clean") and flat > EXACT_FLOPS:
        return None
    if op in ("dirty", "degrid", "hessian") and 8.0 * 22 * 0.9 * case["n_row"] * case["n_chan"] / nb * nx * ny * nb > EXACT_FLOPS:
        return None
    d = _inputs(case, seed)
    bands = [_Band(case, d, b) for b in range(nb)]
    times = {"hessian": 2, "clean": 1 + 2 * case["n_major"]}.get(op, 1)
    if op in ("dirty", "degrid", "hessian", "clean") and times * sum(b.flops for b in bands) > EXACT_FLOPS:
        return None
    sky = d["sky"].to(torch.float64)

    def hessian(x):
        return torch.stack([b.adjoint(b.forward(x[k])) for k, b in enumerate(bands)])

    def dirty():
        return torch.stack([b.adjoint(d["vis"][:, b.sel].to(torch.complex128)[b.live]) for b in bands])

    if op == "dirty":
        return dirty()
    if op == "degrid":
        out = torch.zeros(case["n_row"], case["n_chan"], dtype=torch.complex128, device="cuda")
        for k, b in enumerate(bands):
            part = torch.zeros(case["n_row"], d["per"], dtype=torch.complex128, device="cuda")
            part[b.live] = b.forward(sky[k])
            out[:, b.sel] = part
        return out
    if op == "hessian":
        return hessian(sky)
    psf = torch.stack([b.psf(nx, ny, d["cell"]) for b in bands])
    if op == "psf":
        return psf
    spec = [torch.fft.rfft2(torch.roll(p, (-nx, -ny), (0, 1))) for p in psf]

    def conv(x):
        return torch.stack([torch.fft.irfft2(torch.fft.rfft2(x[k], s=(2 * nx, 2 * ny)) * spec[k], s=(2 * nx, 2 * ny))[:nx, :ny]
                            for k in range(nb)])

    if op == "conv":
        return conv(sky)
    unorm = _norm_bound(psf)
    sigma = 1e-3 * unorm
    if op == "fb":
        x = d["rough"].clamp_min(0).to(torch.float64)
        return (x - _cg(conv, conv(x) - conv(sky), sigma, case["cg_iters"]) - 1e-3).clamp_min(0)
    if op == "prox":
        z = d["rough"].to(torch.float64)
        return _prox(conv, z, z.clamp_min(0), None, sigma, _threshold(case), unorm, case["pd_iters"], case["levels"])[0]
    x, v, image = sky, None, dirty()
    for k in range(case["n_major"]):
        z = x - _cg(conv, hessian(x) - image, sigma, case["cg_iters"])
        x, v = _prox(conv, z, z.clamp_min(0) if k == 0 else x, v, sigma, _threshold(case), unorm, case["pd_iters"], case["levels"])
    return x
