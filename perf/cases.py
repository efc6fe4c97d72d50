"""The work a user of svconv has it do, as measurable cases.

A case names one call (``kind``) with its image size, kernel, basis, form and
precision:

  difference  D = (R (x) K) - I through ``Plan.difference``
  gradient    D and its gradients in R and a through autograd
  equations   the normal equations of the kernel fit (``normal_equations``)
  fit         the least-squares fit of a delta-basis kernel (``least_squares_fit``)
  stamps      isolated-star stamp selection (``stamp_mask``)
  mosaic      host-resident tiles streamed through ``Pipeline``

Images are synthetic star fields: Poisson sky of 1000 ADU, stars of flux
10^U(3, 5) with a Gaussian PSF of FWHM 2.5 pixels at the star density of a
2048 x 4096 chip with 20000 stars.  Sizes, bases and forms are those of the
repository's workloads: 15 x 15, 21 x 21 and 31 x 31 Gaussian kernels, the
7 x 7 delta basis, frames from 64 x 64 to one 4846 x 4868 camera tile.
"""

import math

import torch

from paper_1209_5823_amd import fit as svfit
from paper_1209_5823_amd import svconv

SKY = 1000.0
SIGMAS = (0.7, 1.5, 2.0)
DEGREES = {"22": (4, 2, 0), "49": (6, 4, 2)}   # bases of the 15 x 15 and the larger kernels
STARS_PER_PIXEL = 20000.0 / (2048 * 4096)
DEV = "cuda"


def _gauss(kind, h, w, half, bases, degree, form, precision, **more):
    return dict(kind=kind, height=h, width=w, half_width=half, bases=bases, spatial_degree=degree,
                form=form, precision=precision, **more)


def _delta(kind, h, w, half, degree, form, precision, **more):
    return _gauss(kind, h, w, half, "delta", degree, form, precision, **more)


def listed():
    cases = {
        # the smallest frame of the size study: a cut-out, latency counts
        "small_256": _gauss("difference", 256, 256, 7, "22", 2, "separable_regrouped", "fp16x3"),
        # one CCD chip in the fastest form: a survey's everyday call
        "chip": _gauss("difference", 2048, 4096, 10, "49", 2, "separable_regrouped", "fp16x3"),
        # the same chip at the accuracy of the FP32 path (float64 passes)
        "chip_f64": _gauss("difference", 2048, 4096, 10, "49", 2, "separable", "fp32"),
        # a plan with its default form and precision, on a ragged crop of a chip
        "default_crop": _gauss("difference", 1021, 1533, 10, "49", 2, "basis", "fp32",
                               frame_x=512, frame_y=300, frame_width=4096, frame_height=2048),
        # the 7 x 7 delta basis on one camera tile, the largest frame
        "tile_delta": _delta("difference", 4846, 4868, 3, 2, "regrouped", "fp32"),
        # wide kernels with cubic variation
        "k31": _gauss("difference", 4096, 4096, 15, "49", 3, "separable", "fp16x3"),
        # training a kernel model: forward and both adjoints on the matrix cores
        "grad_k31": _gauss("gradient", 2048, 2048, 15, "49", 3, "separable", "fp16x3"),
        # the same through the float64 passes, on a small ragged crop of a chip
        "grad_crop_f64": _gauss("gradient", 517, 771, 10, "49", 2, "separable", "fp32",
                                frame_x=1000, frame_y=700, frame_width=4096, frame_height=2048),
        # set-up of a Gaussian-basis fit
        "equations": _gauss("equations", 2048, 2048, 10, "49", 2, "separable", "fp32"),
        # a whole delta-basis fit of a cut-out: normal equations, factor, two steps
        "fit_delta": _delta("fit", 1024, 1024, 3, 2, "basis", "fp32"),
        # stamp selection on a chip
        "stamps": _gauss("stamps", 2048, 4096, 10, "49", 2, "separable", "fp32"),
        # tiles that live in host memory, as a mosaic camera writes them
        "mosaic": _gauss("mosaic", 1024, 2048, 10, "49", 2, "separable_regrouped", "fp16x3", tiles=4),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def draw(rng):
    def sides(lo, most_pixels, longest=4868):
        while True:
            s = [int(round(math.exp(rng.uniform(math.log(lo), math.log(longest))))) for _ in range(2)]
            if rng.random() < 0.5:
                s = [max(16, (v + 8) // 16 * 16) for v in s]
            if s[0] * s[1] <= most_pixels:
                return s

    kind = rng.choice(("difference", "difference", "difference", "delta", "gradient", "gradient",
                       "equations", "fit", "stamps", "mosaic"))
    half, bases = rng.choice(((7, "22"), (10, "49"), (15, "49")))
    if kind == "difference":
        form, precision = rng.choice((("separable_regrouped", "fp16x3"), ("separable_regrouped", "bf16x3"),
                                      ("separable", "fp32"), ("separable", "fp16x3"),
                                      ("separable", "bf16x3"), ("basis", "fp32"), ("basis", "fp16x3"),
                                      ("regrouped", "fp16x3"), ("regrouped", "fp32")))
        regrouped = form == "separable_regrouped"
        if regrouped:
            half = min(half, 10)
        degree = rng.choice((1, 2) if regrouped else (1, 2, 3))
        most = 1024 * 1024 if form == "basis" else 2048 * 2048 if half > 10 else 2048 * 4096
        return _gauss(kind, *sides(64, most), half, bases, degree, form, precision)
    if kind == "delta":
        return _delta("difference", *sides(64, 4846 * 4868), rng.choice((2, 3, 4)), rng.choice((1, 2)),
                      "regrouped", rng.choice(("fp32", "fp32", "fp16x3")))
    if kind == "gradient":
        form, precision = rng.choice((("separable", "fp16x3"), ("separable", "bf16x3"),
                                      ("separable", "fp32"), ("basis", "fp32")))
        most = 512 * 1024 if form == "basis" else 1024 * 2048
        return _gauss(kind, *sides(64, most), half, bases, rng.choice((1, 2, 3)), form, precision)
    if kind == "equations":
        return _gauss(kind, *sides(128, 1024 * 2048), half, bases, rng.choice((1, 2)), "separable", "fp32")
    if kind == "fit":
        return _delta(kind, *sides(256, 1024 * 1024), rng.choice((2, 3)), rng.choice((1, 2)), "basis", "fp32")
    if kind == "stamps":
        return _gauss(kind, *sides(256, 2048 * 4096), half, bases, 2, "separable", "fp32")
    return _gauss("mosaic", *sides(256, 1024 * 2048), min(half, 10), bases, 2, "separable_regrouped",
                  "fp16x3", tiles=rng.choice((2, 3, 4)))


# ------------------------------------------------------------------ inputs --

def _degrees(case):
    return None if case["bases"] == "delta" else DEGREES[case["bases"]]


def _sizes(case):
    """(number of bases, number of spatial terms, kernel width)"""
    k = 2 * case["half_width"] + 1
    deg = _degrees(case)
    n = k * k if deg is None else sum((d + 1) * (d + 2) // 2 for d in deg)
    return n, (case["spatial_degree"] + 1) * (case["spatial_degree"] + 2) // 2, k


def _blur(img, taps):
    """Separable convolution with an odd symmetric filter, zero outside."""
    r = len(taps) // 2
    for axis in (0, 1):
        acc = taps[r] * img
        for d in range(1, r + 1):
            lo, hi = [slice(None)] * 2, [slice(None)] * 2
            n = img.shape[axis]
            if n <= d:
                break
            lo[axis], hi[axis] = slice(0, n - d), slice(d, n)
            acc[tuple(lo)] += taps[r + d] * img[tuple(hi)]
            acc[tuple(hi)] += taps[r + d] * img[tuple(lo)]
        img = acc
    return img


def _psf(fwhm, radius=6):
    s = fwhm / 2.3548200450309493
    t = [math.exp(-0.5 * (i / s) ** 2) for i in range(-radius, radius + 1)]
    z = sum(t)
    return [v / z for v in t]


def _stars(h, w, gen):
    n = max(4, int(round(STARS_PER_PIXEL * h * w)))
    at = torch.randint(0, h * w, (n,), generator=gen, device=DEV).unique()
    flux = 10.0 ** (3.0 + 2.0 * torch.rand(at.numel(), generator=gen, device=DEV))
    img = torch.zeros(h * w, device=DEV)
    img[at] = flux
    return _blur(img.view(h, w), _psf(2.5))


def _field(h, w, gen):
    sky = torch.poisson(torch.full((h, w), SKY, device=DEV), generator=gen)
    return (sky + _stars(h, w, gen)).contiguous()


def _coefficients(case, gen):
    """U(-0.05, 0.05) with 1 for the constant term of one near-central basis."""
    n, m, k = _sizes(case)
    a = 0.1 * torch.rand(n, m, generator=gen, device=DEV) - 0.05
    deg = _degrees(case)
    a[n // 2 if deg is None else (deg[0] + 1) * (deg[0] + 2) // 2, 0] = 1.0
    return a.contiguous()


def _fit_images(case, gen):
    """A reference and a second image that a smoothly varying kernel maps it to,
    with its own photon noise."""
    h, w = case["height"], case["width"]
    R = _field(h, w, gen)
    ramp = torch.linspace(-1.0, 1.0, w, device=DEV)[None, :]
    model = 0.7 * R + (0.3 + 0.05 * ramp) * _blur(R, _psf(2.0, 3))
    I = (model + model.clamp(min=1.0).sqrt() * torch.randn(h, w, generator=gen, device=DEV))
    return R, I.contiguous()


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _inputs(case, seed):
    gen = _generator(seed)
    h, w = case["height"], case["width"]
    kind = case["kind"]
    if kind in ("equations", "fit"):
        R, I = _fit_images(case, gen)
        return {"R": R, "I": I}
    if kind == "stamps":
        return {"R": _field(h, w, gen)}
    if kind == "mosaic":
        return {"R": [_field(h, w, gen) for _ in range(case["tiles"])],
                "I": [_field(h, w, gen) for _ in range(case["tiles"])],
                "a": [_coefficients(case, gen) for _ in range(case["tiles"])]}
    x = {"R": _field(h, w, gen), "I": _field(h, w, gen), "a": _coefficients(case, gen)}
    if kind == "gradient":
        x["G"] = 120.0 * torch.rand(h, w, generator=gen, device=DEV) - 60.0
    return x


def _plan(case):
    frame = None
    if "frame_width" in case:
        frame = (case["frame_x"], case["frame_y"], case["frame_width"], case["frame_height"])
    size = (case["height"], case["width"], case["half_width"])
    how = dict(precision=case["precision"], form=case["form"], frame=frame, pedestal=SKY)
    deg = _degrees(case)
    if deg is None:
        return svconv.Plan.dfb(*size, case["spatial_degree"], **how)
    return svconv.Plan(*size, SIGMAS, deg, case["spatial_degree"], **how)


def prepare(case, seed):
    state = dict(_inputs(case, seed), kind=case["kind"], plan=_plan(case))
    if case["kind"] == "gradient":
        state["R"].requires_grad_()
        state["a"].requires_grad_()
    elif case["kind"] == "fit":
        n, m, _ = _sizes(case)
        state["a0"] = torch.zeros(n, m, dtype=torch.float64, device=DEV)
        state["a0"][n // 2, 0] = 1.0
    elif case["kind"] == "mosaic":
        def pinned(t):
            p = svconv.pinned_empty(tuple(t.shape))
            p.copy_(t)
            return p
        for key in ("R", "I"):
            state[key] = [pinned(t) for t in state[key]]
        state["a"] = [t.cpu() for t in state["a"]]
        state["D"] = [svconv.pinned_empty(tuple(t.shape)) for t in state["R"]]
        state["pipeline"] = svconv.Pipeline(state["plan"], depth=3)
    torch.cuda.synchronize()
    return state


def run(state):
    kind, plan = state["kind"], state["plan"]
    if kind == "difference":
        return plan.difference(state["R"], state["I"], state["a"])
    if kind == "gradient":
        D = svconv.difference(plan, state["R"], state["I"], state["a"])
        gR, ga = torch.autograd.grad(D, (state["R"], state["a"]), state["G"])
        return {"D": D.detach(), "gR": gR, "ga": ga}
    if kind == "equations":
        JtJ, rhs = plan.normal_equations(state["R"], state["I"])
        return {"JtJ": JtJ, "rhs": rhs}
    if kind == "fit":
        a, D, _, _ = svfit.least_squares_fit(plan, state["R"], state["I"], state["a0"], iters=2)
        return {"a": a, "D": D}
    if kind == "stamps":
        mask, centres = plan.stamp_mask(state["R"], SKY, 300.0)
        return {"mask": mask, "centres": centres}
    state["pipeline"].run(state["R"], state["I"], state["a"], state["D"])
    return list(state["D"])


# ------------------------------------------------------------------- work --

def work(case):
    n, m, k = _sizes(case)
    px = case["height"] * case["width"]
    deg = _degrees(case)
    if deg is None:
        forward = 2 * m * k * k + 2 * m + 1
    else:
        # one-dimensional passes: a row pass per factor, then a column pass per
        # basis, or per row factor and spatial term, whichever is less
        rows = sum(d + 1 for d in deg)
        forward = 2 * rows * k + min(2 * n * k + 2 * n * m + 2 * n, 2 * rows * m * k + 2 * m) + 1
    kind = case["kind"]
    if kind == "difference":
        return {"bytes": 12 * px + 4 * n * m, "flops": forward * px}
    if kind == "gradient":
        # R, I, G in; D, gR out
        return {"bytes": 20 * px + 8 * n * m, "flops": 3 * forward * px}
    if kind == "equations" or kind == "fit":
        planes = n + 1
        # every pair of responses for each power of x; y is constant along a row
        gram = planes * (planes + 1) * (2 * case["spatial_degree"] + 1)
        responses = 0 if deg is None else 2 * (sum(d + 1 for d in deg) + n) * k
        if kind == "equations":
            return {"bytes": 8 * px + 8 * (n * m) * (n * m + 1), "flops": (gram + responses) * px}
        return {"bytes": 12 * px + 8 * (n * m) * (n * m + 1),
                "flops": (gram + responses + 3 * forward) * px + (n * m) ** 3 / 3}
    if kind == "stamps":
        return {"bytes": 5 * px, "flops": 10 * px}
    return {"bytes": 12 * px * case["tiles"], "flops": forward * px * case["tiles"]}


# ------------------------------------------------------------------ exact --

def _powers(case):
    return [(t - j, j) for t in range(case["spatial_degree"] + 1) for j in range(t + 1)]


def _axes(case):
    """Frame coordinates in [-1, 1] of the columns and rows, float64."""
    h, w = case["height"], case["width"]
    x0, y0 = case.get("frame_x", 0), case.get("frame_y", 0)
    wf, hf = case.get("frame_width", w), case.get("frame_height", h)
    x = torch.arange(w, dtype=torch.float64, device=DEV) + x0
    y = torch.arange(h, dtype=torch.float64, device=DEV) + y0
    return (2.0 * x / (wf - 1) - 1.0 if wf > 1 else 0.0 * x), (2.0 * y / (hf - 1) - 1.0 if hf > 1 else 0.0 * y)


def _term(case, power):
    x, y = _axes(case)
    return (y ** power[1])[:, None] * (x ** power[0])[None, :]


def _factor(sigma, e, half):
    w = torch.arange(-half, half + 1, dtype=torch.float64, device=DEV)
    f = torch.exp(-w * w / (2.0 * sigma * sigma)) * w ** e
    return f / f.abs().sum()


def _factors(case):
    """Per basis: (factor in x, factor in y), float64, in the basis' order."""
    out = []
    for s, d in zip(SIGMAS, _degrees(case)):
        f = [_factor(s, e, case["half_width"]) for e in range(d + 1)]
        out += [(f[t - j], f[j]) for t in range(d + 1) for j in range(t + 1)]
    return out


def _basis(case):
    """B[n][v + h][u + h], float64."""
    n, _, k = _sizes(case)
    if _degrees(case) is None:
        return torch.eye(n, dtype=torch.float64, device=DEV).view(n, k, k)
    return torch.stack([fy[:, None] * fx[None, :] for fx, fy in _factors(case)])


class _Fourier:
    """Linear convolution and correlation of a frame with small kernels."""

    def __init__(self, case):
        self.h, self.w, self.half = case["height"], case["width"], case["half_width"]

        def size(n):
            n += 2 * self.half
            while True:
                m = n
                for p in (2, 3, 5, 7):
                    while m % p == 0:
                        m //= p
                if m == 1:
                    return n
                n += 1
        self.shape = (size(self.h), size(self.w))

    def of(self, img):
        return torch.fft.rfft2(img.double(), s=self.shape)

    def of_kernel(self, K):
        out = torch.zeros(self.shape, dtype=torch.float64, device=DEV)
        k = K.shape[0]
        out[:k, :k] = K
        return torch.fft.rfft2(torch.roll(out, (-self.half, -self.half), (0, 1)))

    def back(self, F):
        return torch.fft.irfft2(F, s=self.shape)


def _kernels(case, a):
    return torch.einsum("nm,nvu->mvu", a.double(), _basis(case))


def _exact_difference(case, R, I, a):
    f = _Fourier(case)
    FR, K = f.of(R), _kernels(case, a)
    D = -I.double()
    for p, Km in zip(_powers(case), K):
        D += _term(case, p) * f.back(FR * f.of_kernel(Km))[:f.h, :f.w]
    return D


def _exact_gradients(case, x):
    f = _Fourier(case)
    k = 2 * f.half + 1
    FR, K, B = f.of(x["R"].detach()), _kernels(case, x["a"].detach()), _basis(case)
    gR, ga = torch.zeros(f.h, f.w, dtype=torch.float64, device=DEV), []
    for p, Km in zip(_powers(case), K):
        FG = f.of(x["G"].double() * _term(case, p))
        gR += f.back(FG * f.of_kernel(Km).conj())[:f.h, :f.w]
        # Q[v][u] = sum_p G P R(p - (u, v))
        Q = torch.roll(f.back(FG * FR.conj()), (f.half, f.half), (0, 1))[:k, :k]
        ga.append((B * Q).sum((1, 2)))
    return gR, torch.stack(ga, 1)


def _shifted(img, du, dv):
    """img(x - du, y - dv), zero outside."""
    h, w = img.shape
    out = torch.zeros_like(img)
    if abs(dv) < h and abs(du) < w:
        out[max(0, dv):h + min(0, dv), max(0, du):w + min(0, du)] = \
            img[max(0, -dv):h + min(0, -dv), max(0, -du):w + min(0, -du)]
    return out


def _responses(case, R):
    """T_n on the frame, float64."""
    R, half = R.double(), case["half_width"]
    if _degrees(case) is None:
        return [_shifted(R, u, v) for v in range(-half, half + 1) for u in range(-half, half + 1)]
    rows, out = {}, []
    for fx, fy in _factors(case):
        key = id(fx)
        if key not in rows:
            rows[key] = sum(fx[u + half] * _shifted(R, u, 0) for u in range(-half, half + 1))
        out.append(sum(fy[v + half] * _shifted(rows[key], 0, v) for v in range(-half, half + 1)))
    return out


def _exact_equations(case, R, I):
    n, m, _ = _sizes(case)
    half, powers = case["half_width"], _powers(case)
    inside = torch.zeros(R.shape, dtype=torch.bool, device=DEV)
    inside[half:R.shape[0] - half, half:R.shape[1] - half] = True
    px = int(inside.sum())
    T = torch.stack([t[inside] for t in _responses(case, R) + [I.double()]])
    step = 32768
    terms = {}
    for p in powers:
        for q in powers:
            e = (p[0] + q[0], p[1] + q[1])
            if e not in terms:
                Q = _term(case, e)[inside]
                S = torch.zeros(n + 1, n + 1, dtype=torch.float64, device=DEV)
                for at in range(0, px, step * 64):
                    part = T[:, at:at + step * 64]
                    pad = -part.shape[1] % step
                    left = torch.nn.functional.pad(part * Q[at:at + step * 64], (0, pad))
                    right = torch.nn.functional.pad(part, (0, pad))
                    left = left.view(n + 1, -1, step).transpose(0, 1).contiguous()
                    right = right.view(n + 1, -1, step).permute(1, 2, 0).contiguous()
                    S += torch.matmul(left, right).sum(0)
                terms[e] = S
    JtJ = torch.zeros(n, m, n, m, dtype=torch.float64, device=DEV)
    rhs = torch.zeros(n, m, dtype=torch.float64, device=DEV)
    for i, p in enumerate(powers):
        rhs[:, i] = terms[p][:n, n]
        for j, q in enumerate(powers):
            JtJ[:, i, :, j] = terms[(p[0] + q[0], p[1] + q[1])][:n, :n]
    return JtJ.reshape(n * m, n * m), rhs.reshape(n * m)


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    if kind == "difference":
        return _exact_difference(case, x["R"], x["I"], x["a"])
    if kind == "gradient":
        gR, ga = _exact_gradients(case, x)
        return {"D": _exact_difference(case, x["R"], x["I"], x["a"]), "gR": gR, "ga": ga}
    if kind == "equations":
        JtJ, rhs = _exact_equations(case, x["R"], x["I"])
        return {"JtJ": JtJ, "rhs": rhs}
    if kind == "fit":
        n, m, _ = _sizes(case)
        JtJ, rhs = _exact_equations(case, x["R"], x["I"])
        a = torch.linalg.solve(JtJ.cpu(), rhs.cpu()).to(DEV).view(n, m)
        return {"a": a, "D": _exact_difference(case, x["R"], x["I"], a.float())}
    if kind == "stamps":
        return None
    return [_exact_difference(case, R, I, a) for R, I, a in zip(x["R"], x["I"], x["a"])]
