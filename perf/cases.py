"""What the framework is timed on: the evaluations that a user's program runs, through the public entry points.

The path is the differentiable PSF model: a pupil (Zernike terms, optionally a bicubic map and a phase
screen), one two-sided matrix Fourier transform per star, wavelength and frame, binning to detector
pixels, the likelihood, and the gradient to every parameter. A program holds a plan, the telescope's static
arrays and the data, and calls the model (simulation), the model and its gradient (fits, calibration) or
one of the parts, again and again with new parameters.

Sizes follow the repository's workloads (``synth/configs.py``, ``bench.py``); ``draw`` spreads over the same
ranges. Inputs are what such a program meets in the middle of a fit: photon noise on the images of a "true"
telescope (formed here with plain torch products), and parameters a little off the truth.

Gradients are returned in the type of the parameters they belong to (FP32), as an optimiser's step takes
them and as the torch autograd entry point hands them over: their FP64 arrays hold FP64 sums of FP32 fields.
The likelihood call alone, which has no FP32 transform in it, returns its FP64 results as they are.
"""
import math
import random

import numpy as np
import torch

from paper_2406_08703_amd import BatchPlan, CapturedEval, Geometry, PsfPlan, evaluate, psf_loss

DIAMETER = 0.5
MU, SIGMA = 1.0, 0.05
TWO_PI = 2.0 * math.pi

# One problem: pupil samples, detector pixels and focal samples per pixel (Q); the band and its wavelengths;
# stars, frames, Zernike terms, bicubic nodes. `pixel`: the detector pixel in units of (band centre)/D, 0.5 is
# Nyquist. `dithers`: "none", "subpixel" (every frame has its own star positions) or "integer" (whole pixels,
# one enlarged plane). `kernel`: the intra-pixel response, "none", "shared" or "pixel" (one for each).
BASE = dict(entry="eval", precision="fp32", kind="poisson", n_pupil=64, n_det=32, oversample=2, n_wl=1,
            band_lo=600e-9, band_hi=600e-9, n_sources=1, n_frames=1, n_zernike=10, n_map=0, pixel=0.5, log_flux=6.0,
            obstruction=0.3, dithers="none", margin=0, kernel="none", kernel_grad=False, screen=False,
            store_fields=False, n_problems=1, sizes_seed=0)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    poly = dict(n_pupil=256, n_det=128, oversample=4, n_wl=20, band_lo=500e-9, band_hi=700e-9, n_zernike=64,
                log_flux=8.0)
    joint = dict(n_pupil=512, n_det=256, oversample=3, n_wl=32, band_lo=500e-9, band_hi=700e-9, n_sources=2,
                 n_zernike=128, log_flux=8.0, dithers="subpixel", kernel="shared")
    return [
        # the smallest fit: one star, one wavelength, an unobstructed pupil; launches and host work count
        _case("small eval", obstruction=0.0),
        # one polychromatic image, replayed from a captured graph as a fit loop does
        _case("polychromatic graph", entry="graph", **poly),
        # the same through torch autograd, split precision, fields kept between forward and backward
        _case("polychromatic autograd bf16x3", entry="autograd", precision="bf16x3", store_fields=True, **poly),
        # odd and ragged sizes, chi-squared data term, the three separate calls
        _case("ragged three calls", entry="calls", kind="chi2", n_pupil=251, n_det=85, oversample=3, n_wl=7,
              band_lo=500e-9, band_hi=700e-9, n_sources=2, n_frames=3, n_zernike=37, log_flux=7.0,
              dithers="subpixel", kernel="shared"),
        # joint flat-field and phase retrieval over dithered frames of a binary: the largest job
        _case("joint 64 frames", entry="graph", n_frames=64, **joint),
        # the same in split precision, as many frames as a night of a smaller programme
        _case("joint 12 frames bf16x3", precision="bf16x3", n_frames=12, **joint),
        # the paper's run: 20 stars, 3 wavelengths, 5 frames dithered by whole pixels, a phase plate
        _case("integer dithers graph", entry="graph", n_pupil=512, n_det=1024, oversample=1, n_wl=3,
              band_lo=545e-9, band_hi=645e-9, n_sources=20, n_frames=5, n_zernike=7, pixel=0.0489, log_flux=7.5,
              obstruction=0.2, dithers="integer", margin=20, screen=True),
        # millions of flat-field pixels, Zernike terms and a bicubic phase map
        _case("megapixel calibration", n_pupil=1024, n_det=1024, oversample=2, n_wl=16, band_lo=500e-9,
              band_hi=700e-9, n_frames=4, n_zernike=256, n_map=64, log_flux=8.0, dithers="subpixel"),
        # many uneven fits in one plan, one launch per stage
        _case("batch of uneven fits", entry="batch", n_problems=24, sizes_seed=3, band_lo=450e-9, band_hi=800e-9),
        # simulating images: the forward model alone
        _case("simulate images", entry="forward", n_pupil=384, n_det=192, oversample=2, n_wl=12, band_lo=500e-9,
              band_hi=700e-9, n_sources=3, n_frames=4, n_zernike=48, log_flux=7.0, dithers="subpixel"),
        # calibrating the response inside every pixel: one kernel per pixel and its gradient
        _case("intra-pixel calibration", n_pupil=128, n_det=100, oversample=2, n_wl=8, band_lo=500e-9,
              band_hi=700e-9, n_frames=6, n_zernike=20, log_flux=7.5, dithers="subpixel", kernel="pixel",
              kernel_grad=True),
        # the likelihood, residual and flat-field gradient of given model images
        _case("likelihood only", entry="loss", n_pupil=128, n_det=512, oversample=1, n_frames=16, log_flux=8.0,
              dithers="subpixel", pixel=0.1),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        entry = rng.choice(["eval", "eval", "graph", "graph", "calls", "autograd", "forward", "batch", "loss"])
        c = dict(BASE, entry=entry, precision=rng.choice(["fp32", "fp32", "bf16x3"]),
                 kind=rng.choice(["poisson", "poisson", "chi2"]), n_pupil=_spread(rng, 32, 800),
                 n_det=_spread(rng, 16, 640), oversample=rng.choice([1, 2, 3, 4]), n_wl=_spread(rng, 1, 40),
                 band_lo=rng.choice([450e-9, 500e-9, 545e-9]), n_sources=_spread(rng, 1, 12),
                 n_frames=_spread(rng, 1, 40), n_zernike=_spread(rng, 4, 130), log_flux=rng.uniform(0.0, 1.0),
                 pixel=rng.choice([0.5, 0.5, 0.5, rng.uniform(0.06, 0.5)]), obstruction=rng.choice([0.0, 0.2, 0.3]),
                 kernel=rng.choice(["none", "shared"]), screen=rng.random() < 0.2)
        # exposures are as deep as the detector's far pixels ask for
        c["log_flux"] += 6.0 + 2.0 * math.log10(max(1.0, c["n_det"] / 64))
        c["band_hi"] = c["band_lo"] * rng.uniform(1.05, 1.6) if c["n_wl"] > 1 else c["band_lo"]
        if rng.random() < 0.5:   # sizes are as often round as not
            c["n_pupil"] = max(32, c["n_pupil"] // 32 * 32)
            c["n_det"] = max(16, c["n_det"] // 16 * 16)
        if c["precision"] == "bf16x3" and c["n_det"] > 128:
            c["kind"] = "chi2"   # split precision does not resolve the faintest far pixels, where 1/m weighs most
        if c["pixel"] < 0.25:    # such fine pixels need no samples inside them
            c["oversample"] = 1
        if entry == "batch":
            c.update(n_problems=rng.randint(4, 24), sizes_seed=rng.randrange(1 << 20), kernel="none", screen=False,
                     n_frames=1, band_lo=450e-9, band_hi=800e-9, pixel=0.5)
        elif c["n_frames"] > 1:
            c["dithers"] = "subpixel"
            if rng.random() < 0.3 and entry != "loss":
                c.update(dithers="integer", margin=rng.randint(2, 20))
        if entry in ("eval", "graph", "calls") and rng.random() < 0.2:
            c["n_map"] = rng.randint(6, 64)
        if entry == "autograd":
            c["store_fields"] = rng.random() < 0.5
        if entry in ("eval", "calls") and c["dithers"] != "integer" and rng.random() < 0.2:
            c.update(kernel="pixel", kernel_grad=True)
        if sum(_dense_flops(p) for p in _problems(c)) < 5e12 and _focal(c) <= 2048:
            return c


# ------------------------------------------------------------------------------------------------ shapes
def _n_plane(c):
    """Detector pixels per side of the plane that is propagated."""
    return c["n_det"] + (2 * c["margin"] if c["dithers"] == "integer" else 0)


def _focal(c):
    return c["oversample"] * _n_plane(c)


def _n_psf(c):
    return c["n_wl"] * c["n_sources"] * (1 if c["dithers"] == "integer" else c["n_frames"])


def _dense_flops(c):
    ni, no = c["n_pupil"], _focal(c)
    return 8.0 * no * ni * (ni + no) * _n_psf(c)


def _problems(c):
    """The problems of a case: itself, or the uneven ones of a batch."""
    if c["entry"] != "batch":
        return [c]
    rng = random.Random(c["sizes_seed"])
    out = []
    for _ in range(c["n_problems"]):
        q = rng.choice([2, 3, 4])
        out.append(dict(c, n_pupil=rng.choice([128, 192, 256, 384, 512]), n_det=rng.choice([64, 128, 256]) // q,
                        oversample=q, n_wl=rng.randint(8, 64), n_zernike=rng.randint(16, 128),
                        n_sources=rng.randint(1, 3), log_flux=rng.uniform(6.0, 8.0), obstruction=0.3))
    return out


def _wavelengths(c):
    n = c["n_wl"]
    return np.linspace(c["band_lo"], c["band_hi"], n) if n > 1 else np.array([0.5 * (c["band_lo"] + c["band_hi"])])


def _det_pixel(c):
    return c["pixel"] * 0.5 * (c["band_lo"] + c["band_hi"]) / DIAMETER


def _dither_list(c):
    """Whole-pixel offsets of the frames, within the margin."""
    rng, m = random.Random(c["n_frames"] * 1000 + c["margin"]), c["margin"]
    return [(0, 0)] + [(rng.choice([-m, m, rng.randint(-m, m)]), rng.choice([-m, m, rng.randint(-m, m)]))
                       for _ in range(c["n_frames"] - 1)]


def _geometry(c):
    lam = _wavelengths(c)
    integer = c["dithers"] == "integer"
    return Geometry(n_pupil=c["n_pupil"], n_focal=c["oversample"] * c["n_det"], oversample=c["oversample"],
                    wavelengths=tuple(lam), weights=tuple([1.0 / len(lam)] * len(lam)), n_sources=c["n_sources"],
                    n_frames=c["n_frames"], n_zernike=c["n_zernike"], n_map=c["n_map"], diameter=DIAMETER,
                    focal_pixel=_det_pixel(c) / c["oversample"],
                    dithers=tuple(_dither_list(c)) if integer else (), margin=c["margin"] if integer else 0)


# ------------------------------------------------------------------------------------------------ inputs
def _centred(n, pitch, dtype=torch.float64):
    return (torch.arange(n, device="cuda", dtype=dtype) - (n - 1) / 2.0) * pitch


def _aperture(n, obstruction):
    """Grey circular aperture with a central obstruction and, then, four vanes two pixels wide."""
    s = _centred(3 * n, DIAMETER / n / 3)
    r = torch.hypot(s[:, None], s[None, :])
    t = r <= DIAMETER / 2
    if obstruction > 0:
        t &= r >= obstruction * DIAMETER / 2
        half = DIAMETER / n
        t &= ~((s.abs() < half)[:, None] | (s.abs() < half)[None, :])
    return t.double().reshape(n, 3, n, 3).mean(dim=(1, 3)).float()


def _zernikes(count, n):
    """Zernike terms in the order of rising degree (tilts first), unit RMS over the disk, zero outside."""
    x = _centred(n, 2.0 / n)
    rho, theta = torch.hypot(x[:, None], x[None, :]), torch.atan2(x[:, None], x[None, :])
    inside = rho <= 1.0
    out = torch.empty((count, n, n), device="cuda", dtype=torch.float32)
    i, deg = 0, 1
    while i < count:
        powers = {}
        for m in range(deg % 2, deg + 1, 2):
            r = torch.zeros_like(rho)
            for k in range((deg - m) // 2 + 1):
                e = deg - 2 * k
                if e not in powers:
                    powers[e] = rho ** e
                r += ((-1) ** k * math.factorial(deg - k) / (math.factorial(k) * math.factorial((deg + m) // 2 - k)
                                                             * math.factorial((deg - m) // 2 - k))) * powers[e]
            for f in ((None,) if m == 0 else (torch.cos, torch.sin)):
                if i < count:
                    z = math.sqrt(deg + 1) * r if f is None else math.sqrt(2 * (deg + 1)) * r * f(m * theta)
                    out[i] = torch.where(inside, z, torch.zeros_like(z)).float()
                    i += 1
        deg += 1
    return out


def _cubic_matrix(n, nodes):
    """Cubic convolution (a = -1/2) from `nodes` across the pupil to its samples, edges repeated."""
    xn0, h = -0.5 * DIAMETER + 0.5 * DIAMETER / nodes, DIAMETER / nodes
    t0 = ((np.arange(n) - (n - 1) / 2.0) * DIAMETER / n - xn0) / h
    j0, out = np.floor(t0).astype(int), np.zeros((n, nodes))
    for off in (-1, 0, 1, 2):
        t = np.abs(t0 - (j0 + off))
        w = np.where(t <= 1, 1.5 * t ** 3 - 2.5 * t ** 2 + 1, np.where(t < 2, -0.5 * t ** 3 + 2.5 * t ** 2 - 4 * t + 2, 0.0))
        np.add.at(out, (np.arange(n), np.clip(j0 + off, 0, nodes - 1)), w)
    return torch.from_numpy(out).float().cuda()


def _inputs(c, seed, with_data=True):
    """Static arrays, data and the parameters of one problem, on the GPU."""
    rng = np.random.default_rng([seed & 0x7fffffff, c["n_pupil"], c["n_det"], c["n_wl"]])
    n, nd, q, f, s = c["n_pupil"], c["n_det"], c["oversample"], c["n_frames"], c["n_sources"]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()  # noqa: E731
    x = dict(transmission=_aperture(n, c["obstruction"]), zbasis=_zernikes(c["n_zernike"], n),
             map_basis=_cubic_matrix(n, c["n_map"]) if c["n_map"] else None, intrapixel=None, screen=None)
    if c["kernel"] == "shared":
        x["intrapixel"] = dev(np.tile(1.0 + 0.005 * (np.arange(q) - (q - 1) / 2) / max(q - 1, 1), (q, 1)))
    elif c["kernel"] == "pixel":
        x["intrapixel"] = dev(1.0 + 0.01 * rng.normal(size=(nd, nd, q, q)))
    if c["screen"]:   # a half-wave plate: 0 or pi on regions bounded by the zeros of a few plane waves
        t = (np.arange(n) - (n - 1) / 2.0) / n
        wave = sum(np.cos(TWO_PI * (kx * t[None, :] + ky * t[:, None]) + ph)
                   for kx, ky, ph in zip(rng.uniform(-6, 6, 6), rng.uniform(-6, 6, 6), rng.uniform(0, TWO_PI, 6)))
        x["screen"] = dev(np.where(wave > 0, np.pi, 0.0))
    pix = _det_pixel(c)
    if s == 2:      # a binary, ten resolution elements apart or a third of a small detector
        sep, pa = min(10 * c["band_lo"] / DIAMETER, nd * pix / 3), rng.uniform(0, TWO_PI)
        pos = 0.5 * sep * np.array([[np.cos(pa), np.sin(pa)], [-np.cos(pa), -np.sin(pa)]])
        flux = 10.0 ** c["log_flux"] * np.array([1.0, 0.3]) / 1.3
    else:
        lim = 0.0 if s == 1 else 0.45 * nd if c["dithers"] == "integer" else 0.25 * nd
        pos = rng.uniform(-lim, lim, size=(s, 2)) * pix
        flux = 10.0 ** (c["log_flux"] + rng.uniform(-0.5, 0.5, size=s))
    src = np.concatenate([pos, flux[:, None]], axis=1)
    truth_src = np.tile(src, (1 if c["dithers"] == "integer" else f, 1, 1))
    if c["dithers"] == "subpixel":
        truth_src[:, :, :2] += rng.uniform(-min(4, nd / 8), min(4, nd / 8), size=(f, 1, 2)) * pix
    scale = 20e-9 * min(1.0, math.sqrt(64.0 / max(1, c["n_zernike"])))
    truth = dict(coeffs=scale * rng.normal(size=c["n_zernike"]), sources=truth_src,
                 phase_map=5e-9 * rng.normal(size=(c["n_map"],) * 2) if c["n_map"] else None,
                 flat=1.0 + SIGMA * rng.normal(size=(nd, nd)))
    # where the fit stands: aberrations and positions nearly found, the pixel response not yet
    now_src = truth_src.copy()
    now_src[:, :, :2] += 0.05 * pix * rng.normal(size=(s, 2))
    now_src[:, :, 2] *= 1.0 + 0.02 * rng.normal(size=s)
    now = dict(coeffs=truth["coeffs"] + 0.1 * scale * rng.normal(size=c["n_zernike"]), sources=now_src,
               phase_map=None if truth["phase_map"] is None else 0.9 * truth["phase_map"],
               flat=1.0 + 0.5 * (truth["flat"] - 1.0))
    shape = lambda a: a[0] if c["dithers"] == "integer" else a  # noqa: E731
    truth = {k: None if v is None else dev(v) for k, v in truth.items()}
    x.update({k: None if v is None else dev(shape(v) if k == "sources" else v) for k, v in now.items()})
    if with_data:
        gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 40)))
        model = _plain_model(c, x, truth["coeffs"], truth["phase_map"], shape(truth["sources"]), truth["flat"],
                             torch.complex64)[1]
        x["data"] = torch.poisson(model.float().clamp_min(0.0), generator=gen)
    return x


# ------------------------------------------------------------------------------------------------ plain torch
class _Plain:
    """The model's pieces in plain torch products (direct transforms), in the given complex type."""

    def __init__(self, c, x, coeffs, phase_map, ctype):
        f64 = torch.float64
        self.c, self.ctype, self.lam = c, ctype, _wavelengths(c)
        n, no = c["n_pupil"], _focal(c)
        self.dx, self.du = DIAMETER / n, _det_pixel(c) / c["oversample"]
        self.xs, self.us = _centred(n, self.dx), _centred(no, self.du)
        self.opd = torch.zeros((n, n), device="cuda", dtype=f64)
        for j in range(c["n_zernike"]):
            self.opd += coeffs[j].double() * x["zbasis"][j].double()
        if c["n_map"]:
            b = x["map_basis"].double()
            self.opd += b @ phase_map.double() @ b.T
        a = x["transmission"].double()
        self.amp = a / a.square().sum().sqrt()
        self.screen = 0.0 if x["screen"] is None else x["screen"].double()

    def pupil(self, lam, pos):
        """[S, n, n] pupil fields of the stars at pos [S, 2]."""
        a, b = pos[:, 0].double()[:, None, None], pos[:, 1].double()[:, None, None]
        ph = (TWO_PI / lam) * (self.opd + self.xs[None, None, :] * a + self.xs[None, :, None] * b) + self.screen
        return torch.polar(self.amp.expand_as(ph).contiguous(), ph).to(self.ctype)

    def matrix(self, lam):
        t = self.us[:, None] * self.xs[None, :] / lam
        t = -TWO_PI * (t - t.round())
        return torch.polar(torch.ones_like(t), t).to(self.ctype).contiguous()

    def field(self, lam, m, p):
        s, n, no = p.shape[0], p.shape[1], m.shape[0]
        t = (p.reshape(s * n, n) @ m.T.contiguous()).reshape(s, n, no)
        return (self.dx * self.du / lam) * torch.stack([m @ t[i] for i in range(s)])

    def adjoint(self, lam, m, y):
        s, no, n = y.shape[0], y.shape[1], m.shape[1]
        t = (y.reshape(s * no, no) @ m.conj().resolve_conj().contiguous()).reshape(s, no, n)
        mh = m.conj().resolve_conj().T.contiguous()
        return (self.dx * self.du / lam) * torch.stack([mh @ t[i] for i in range(s)])

    def on_focal(self, k):
        """The intra-pixel kernel on the focal grid."""
        q, nd = self.c["oversample"], _n_plane(self.c)
        k = k.double()
        return k.repeat(nd, nd) if k.dim() == 2 else k.permute(0, 2, 1, 3).reshape(nd * q, nd * q)


def _star_list(c, sources):
    """Positions and fluxes as [frames propagated, S, 3]."""
    return sources[None] if c["dithers"] == "integer" else sources


def _windows(c):
    m = c["margin"]
    return [(m - dy, m - dx) for dx, dy in _dither_list(c)]


def _plain_model(c, x, coeffs, phase_map, sources, flat, ctype):
    """Binned and model images [F, n_det, n_det] and the pieces used."""
    p = _Plain(c, x, coeffs, phase_map, ctype)
    src, nd, q = _star_list(c, sources), _n_plane(c), c["oversample"]
    out = torch.zeros((src.shape[0], nd, nd), device="cuda", dtype=torch.float64)
    k = None if x["intrapixel"] is None else p.on_focal(x["intrapixel"])
    step = max(1, int(2e8 // (c["n_sources"] * _focal(c) ** 2)))   # a few GB of fields at a time
    for lam in p.lam:
        m = p.matrix(lam)
        for f0 in range(0, src.shape[0], step):
            part = src[f0:f0 + step]
            e = p.field(lam, m, p.pupil(lam, part.reshape(-1, 3)[:, :2]))
            i = (torch.view_as_real(e).double().square().sum(-1) * part.reshape(-1, 3)[:, 2].double()[:, None, None])
            i = i.reshape(part.shape[0], c["n_sources"], *i.shape[1:]).sum(1) / len(p.lam)
            if k is not None:
                i = i * k
            out[f0:f0 + step] += i.reshape(-1, nd, q, nd, q).sum(dim=(2, 4))
    if c["dithers"] == "integer":
        n = c["n_det"]
        out = torch.stack([out[0, r:r + n, s:s + n] for r, s in _windows(c)])
    return out, flat.double() * out, p


def _plain_loss(c, binned, model, data, flat):
    m, d, fl = model.clamp_min(1e-30), data.double(), flat.double()
    if c["kind"] == "poisson":
        ell, r = m - torch.where(d != 0, d * m.log(), torch.zeros_like(d)), 1.0 - d / m
    else:
        w = d.clamp_min(1.0)
        ell, r = 0.5 * (m - d).square() / w, (m - d) / w
    loss = ell.sum() + ((fl - MU).square().sum()) / (2 * SIGMA ** 2)
    return loss, r, (r * binned).sum(0) + (fl - MU) / SIGMA ** 2


def _plain_gradient(c, x, p, sources, flat, r):
    src, nd, q, ns = _star_list(c, sources), _n_plane(c), c["oversample"], c["n_sources"]
    h = flat.double() * r
    if c["dithers"] == "integer":
        n, wide = c["n_det"], torch.zeros((1, nd, nd), device="cuda", dtype=torch.float64)
        for f, (a, b) in enumerate(_windows(c)):
            wide[0, a:a + n, b:b + n] += h[f]
        h = wide
    k = None if x["intrapixel"] is None else p.on_focal(x["intrapixel"])
    g_opd, g_src = torch.zeros_like(p.opd), torch.zeros(src.shape, device="cuda", dtype=torch.float64)
    g_k = torch.zeros((nd, q, nd, q), device="cuda", dtype=torch.float64)
    step = max(1, int(1e8 // (ns * _focal(c) ** 2)))
    for lam in p.lam:
        m = p.matrix(lam)
        for f0 in range(0, src.shape[0], step):
            part = src[f0:f0 + step]
            nf, phi = part.shape[0], part.reshape(-1, 3)[:, 2].double()[:, None, None]
            pup = p.pupil(lam, part.reshape(-1, 3)[:, :2])
            e = p.field(lam, m, pup)
            hf = h[f0:f0 + step].repeat_interleave(q, 1).repeat_interleave(q, 2)
            g = hf if k is None else hf * k
            i = torch.view_as_real(e).square().sum(-1)
            g = g[:, None].expand(nf, ns, *g.shape[1:]).reshape(nf * ns, *g.shape[1:])
            g_src[f0:f0 + step, :, 2] += (g * i).sum(dim=(1, 2)).reshape(nf, ns) / len(p.lam)
            if c["kernel_grad"]:
                v = (phi * i).reshape(nf, ns, *i.shape[1:]).sum(1) * hf / len(p.lam)
                g_k += v.reshape(nf, nd, q, nd, q).sum(0)
            w = p.adjoint(lam, m, (phi / len(p.lam)) * g * e)
            gp = 2.0 * (pup.conj() * w).imag * (TWO_PI / lam)
            g_opd += gp.sum(0)
            g_src[f0:f0 + step, :, 0] += (gp * p.xs[None, None, :]).sum(dim=(1, 2)).reshape(nf, ns)
            g_src[f0:f0 + step, :, 1] += (gp * p.xs[None, :, None]).sum(dim=(1, 2)).reshape(nf, ns)
    out = dict(grad_coeffs=torch.stack([(z.double() * g_opd).sum() for z in x["zbasis"]]),
               grad_sources=g_src[0] if c["dithers"] == "integer" else g_src)
    if c["n_map"]:
        b = x["map_basis"].double()
        out["grad_map"] = b.T @ g_opd @ b
    if c["kernel_grad"]:
        out["grad_kernel"] = g_k.permute(0, 2, 1, 3).contiguous()
    return out


def exact(case, seed):
    """What run() returns, by direct transforms in 64 bits."""
    outs = []
    for p in _problems(case):
        x = _inputs(p, seed)
        if case["entry"] == "loss":
            binned, model = (v.double() for v in _given_images(p, x))
        else:
            binned, model, plain = _plain_model(p, x, x["coeffs"], x["phase_map"], x["sources"], x["flat"],
                                                torch.complex128)
        o = dict(binned=binned, model=model)
        if case["entry"] != "forward":
            o["loss"], o["r"], o["grad_flat"] = _plain_loss(p, binned, model, x["data"], x["flat"])
            if case["entry"] != "loss":
                o.update(_plain_gradient(p, x, plain, x["sources"], x["flat"], o["r"]))
            o["loss"] = o["loss"].reshape(1)
        outs.append(o)
    if case["entry"] == "batch":
        return {k: torch.cat([o[k].reshape(-1) for o in outs]) for k in _RETURNED if k in outs[0]}
    o = outs[0]
    if case["entry"] == "loss":
        return {k: o[k] for k in ("loss", "r", "grad_flat")}
    if case["entry"] == "autograd":
        return {k: v for k, v in o.items() if k not in ("binned", "model", "r")}
    return {k: o[k] for k in _RETURNED if k in o}


_RETURNED = ("binned", "model", "r", "loss", "grad_flat", "grad_coeffs", "grad_map", "grad_sources", "grad_kernel")


# ------------------------------------------------------------------------------------------------ the calls
def _given_images(c, x):
    """Model images in hand for the likelihood call: smooth stars of the given fluxes on a faint sky."""
    u = _centred(c["n_det"], _det_pixel(c))
    wide = 0.45 * c["band_lo"] / DIAMETER
    img = torch.full((c["n_frames"], c["n_det"], c["n_det"]), 3.0, device="cuda", dtype=torch.float64)
    for f in range(c["n_frames"]):
        for a, b, phi in x["sources"][f].double():
            g = torch.exp(-0.5 * ((u[None, :] - a).square() + (u[:, None] - b).square()) / wide ** 2)
            img[f] += phi * g / g.sum()
    binned = img.float()
    return binned, x["flat"] * binned


def prepare(case, seed):
    if case["entry"] == "batch":
        return _prepare_batch(case, seed)
    x = _inputs(case, seed)
    st = dict(x, case=case)
    st["plan"] = PsfPlan(_geometry(case), x["transmission"], x["zbasis"], x["map_basis"], x["intrapixel"],
                         precision=case["precision"], store_fields=case["store_fields"],
                         pixel_kernel=case["kernel"] == "pixel")
    if x["screen"] is not None:
        st["plan"].set_phase_screen(x["screen"])
    if case["entry"] == "graph":
        st["graph"] = CapturedEval(st["plan"], x["coeffs"], x["phase_map"], x["sources"], x["flat"], x["data"],
                                   case["kind"], MU, SIGMA)
    elif case["entry"] == "autograd":
        for k in ("coeffs", "sources", "flat"):
            st[k] = x[k].requires_grad_()
    elif case["entry"] == "loss":
        st["binned"], st["model"] = _given_images(case, x)
    return st


def _prepare_batch(case, seed):
    ps = _problems(case)
    xs = [_inputs(p, seed) for p in ps]
    plan = BatchPlan([_geometry(p) for p in ps], [x["transmission"] for x in xs], [x["zbasis"] for x in xs],
                     precision=case["precision"], grouped=True)
    st = dict(case=case, plan=plan, out=plan.buffers())
    for key, field in (("coeffs", "zernike_coeffs"), ("sources", "sources"), ("flat", "flat"), ("data", "images")):
        st[key] = plan.pack(field, [x[key] for x in xs])
    st["args"] = plan.eval_args(st["coeffs"], None, st["sources"], st["flat"], st["data"], st["out"], case["kind"],
                                MU, SIGMA)
    plan.capture(st["args"])
    return st


def _handed_over(c, o):
    """The results of an evaluation, gradients in the type of their parameters."""
    out = dict(binned=o.binned, model=o.model, r=o.r, loss=o.loss.float(), grad_flat=o.grad_flat.float(),
               grad_coeffs=o.grad_zernike[:c["n_zernike"]].float(), grad_sources=o.grad_sources.float())
    if c["n_map"]:
        out["grad_map"] = o.grad_map.float()
    if c["kernel_grad"]:
        out["grad_kernel"] = o.grad_intrapixel.float()
    return out


def run(st):
    c, plan = st["case"], st["plan"]
    if c["entry"] == "eval":
        return _handed_over(c, evaluate(plan, st["coeffs"], st["phase_map"], st["sources"], st["flat"], st["data"],
                                        c["kind"], MU, SIGMA, intrapixel_grad=c["kernel_grad"]))
    if c["entry"] == "graph":
        return _handed_over(c, st["graph"].replay())
    if c["entry"] == "batch":
        plan.replay()
        o = st["out"]
        return dict(binned=o["binned"], model=o["model"], r=o["r"], loss=o["loss"].float(),
                    grad_flat=o["grad_flat"].float(), grad_coeffs=o["grad_zernike"].float(),
                    grad_sources=o["grad_sources"].float())
    if c["entry"] == "loss":
        loss, r, gf = plan.loss_grad(st["model"], st["binned"], st["data"], st["flat"], c["kind"], MU, SIGMA)
        return dict(loss=loss, r=r, grad_flat=gf)
    if c["entry"] == "autograd":
        loss = psf_loss(plan, st["data"], st["coeffs"], None, st["sources"], st["flat"], c["kind"], MU, SIGMA)
        g = torch.autograd.grad(loss, (st["coeffs"], st["sources"], st["flat"]))
        return dict(loss=loss.detach().float().reshape(1), grad_coeffs=g[0], grad_sources=g[1], grad_flat=g[2])
    binned, model = plan.forward(st["coeffs"], st["phase_map"], st["sources"], st["flat"])
    if c["entry"] == "forward":
        return dict(binned=binned, model=model)
    loss, r, gf = plan.loss_grad(model, binned, st["data"], st["flat"], c["kind"], MU, SIGMA)
    gk = None
    if c["kernel_grad"]:
        gk = torch.empty(plan.k_shape, dtype=torch.float64, device="cuda")
    gz, gm, gs = plan.backward(st["coeffs"], st["phase_map"], st["sources"], st["flat"], r, grad_intrapixel=gk)
    out = dict(binned=binned, model=model, r=r, loss=loss.float(), grad_flat=gf.float(), grad_coeffs=gz.float(),
               grad_sources=gs.float())
    if gm is not None:
        out["grad_map"] = gm.float()
    if gk is not None:
        out["grad_kernel"] = gk.float()
    return out


def work(case):
    """Every input read once and every result written once; the operations of fast transforms between the two
    grids (both are regular, so lines of n = N_pupil + N_focal samples take 5 n log2 n operations each way),
    of the pupil's basis, and a few for each focal sample."""
    nbytes = flops = 0.0
    both = case["entry"] not in ("forward", "loss")
    for p in _problems(case):
        n, no, nd, f = p["n_pupil"], _focal(p), p["n_det"], p["n_frames"]
        images = f * nd * nd
        if case["entry"] == "loss":
            nbytes += 4.0 * (3 * images + nd * nd) + 4.0 * images + 8.0 * nd * nd
            flops += 30.0 * images
            continue
        stars = 12.0 * p["n_sources"] * (1 if p["dithers"] == "integer" else f)
        kernel = 4.0 * p["oversample"] ** 2 * {"none": 0, "shared": 1, "pixel": nd * nd}[p["kernel"]]
        nbytes += (4.0 * n * n * (p["n_zernike"] + 1 + (1 if p["screen"] else 0)) + 4.0 * p["n_map"] * (n + p["n_map"])
                   + stars + 4.0 * nd * nd + kernel + 4.0 * 2 * images)
        line = n + no
        each = 5.0 * line * line * math.log2(line) + 10.0 * no * no
        flops += _n_psf(p) * each + 2.0 * n * n * p["n_zernike"]
        if both:
            nbytes += 4.0 * 2 * images + 8.0 * nd * nd + 2 * stars + 8.0 * (p["n_zernike"] + p["n_map"] ** 2)
            nbytes += 2 * kernel if p["kernel_grad"] else 0.0
            flops += _n_psf(p) * each + 2.0 * n * n * p["n_zernike"]
    return {"bytes": nbytes, "flops": flops}
