"""The work this framework does for its users, as timed cases.

Each case is one call (or one gradient step) through the public entry points
of paper_1704_08364_amd: filtered and plain backprojection, raw counts, the
accuracy-matched cubic path, the projector, a least-squares gradient, uneven
batches and the brute-force comparison. `listed()` gives the fixed cases,
`draw(rng)` one more of the same ranges, `prepare` what a program holds before
the call, `run` one pass, `work` the bytes and operations a pass cannot do
without and `exact` the same result in 64-bit torch.

Inputs are analytic sinograms of random ellipses with 1 % noise, images those
ellipses' own values.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1704_08364_amd as P
from paper_1704_08364_amd import autograd as AG

# ---- cases -------------------------------------------------------------------
#
# kind   fbp     Plan.backproject, ramp filter
#        counts  Plan.backproject_counts: raw counts, Hann window, shifted axis
#        plain   Plan.backproject, no filter, monopole subtraction
#        project Plan.project (the adjoint projector)
#        lsgrad  loss and gradient of ||R f - g||^2 through autograd
#        uneven  Batch.backproject: sinograms of many sizes in one call
#        brute   Plan.ramp_filter, then Plan.bruteforce
# n detector bins = image side, V angles, B slices; interp linear or keys, pc
# the Cartesian padding, angles even or golden (golden-angle scan), angular
# linear or tent.


def listed():
    return [
        # a single slice looked at during a scan: latency and launches
        {"name": "fbp_256_one_slice", "kind": "fbp", "n": 256, "V": 256, "B": 1,
         "interp": "linear", "pc": 2, "angles": "even"},
        # a golden-angle scan, a handful of slices, an odd batch
        {"name": "fbp_512_golden", "kind": "fbp", "n": 512, "V": 377, "B": 5,
         "interp": "linear", "pc": 2, "angles": "golden"},
        # an ordinary detector, an odd number of angles
        {"name": "fbp_1024", "kind": "fbp", "n": 1024, "V": 1001, "B": 24,
         "interp": "linear", "pc": 2, "angles": "even"},
        # the benchmark: a block of 64 slices of a 2048^3 volume
        {"name": "fbp_2048_block", "kind": "fbp", "n": 2048, "V": 2048, "B": 64,
         "interp": "linear", "pc": 2, "angles": "even"},
        # the same block by the more accurate path: cubic taps, no oversampling
        {"name": "fbp_2048_cubic", "kind": "fbp", "n": 2048, "V": 2048, "B": 64,
         "interp": "keys", "pc": 1, "angles": "even"},
        # the largest detector, a pair of slices
        {"name": "fbp_4096_pair", "kind": "fbp", "n": 4096, "V": 3001, "B": 2,
         "interp": "linear", "pc": 2, "angles": "even"},
        # beamline data as it arrives: raw counts, flat and dark fields, the axis off centre
        {"name": "counts_2048", "kind": "counts", "n": 2048, "V": 2000, "B": 7},
        # plain backprojection as an operator, origin artifacts suppressed
        {"name": "plain_1024", "kind": "plain", "n": 1024, "V": 1024, "B": 16},
        # the projector of iterative reconstruction
        {"name": "project_1024", "kind": "project", "n": 1024, "V": 1024, "B": 32, "angular": "linear"},
        # one gradient step of a least-squares reconstruction
        {"name": "lsgrad_512_tent", "kind": "lsgrad", "n": 512, "V": 500, "B": 12, "angular": "tent"},
        # sinograms of many scans in one call
        {"name": "uneven_96", "kind": "uneven", "count": 96, "nmax": 2048, "sizes": 170408368},
        # the direct sum that results are compared with
        {"name": "brute_1024", "kind": "brute", "n": 1024, "V": 1024, "B": 2},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    cap = {"bytes": 0, "flops": 0}
    for c in listed():
        w = work(c)
        cap = {k: max(cap[k], w[k]) for k in cap}
    while True:
        kind = rng.choice(["fbp", "fbp", "fbp", "fbp", "counts", "plain", "project", "lsgrad", "uneven", "brute"])
        case = {"kind": kind}
        if kind == "uneven":
            case.update(count=_log_int(rng, 8, 96), nmax=rng.choice([512, 1024, 2048]), sizes=rng.randrange(1 << 30))
        else:
            big = {"fbp": 4096, "counts": 2048, "plain": 2048, "project": 1024, "lsgrad": 1024, "brute": 1024}[kind]
            n = rng.choice([s for s in (128, 256, 512, 1024, 2048, 4096) if s <= big])
            # an oversampled block of the largest detector would be many times the largest listed case
            case.update(n=n, V=_log_int(rng, n // 2, 2 * n),
                        B=_log_int(rng, 1, {4096: 6, 2048: 48}.get(n, 64) if kind != "brute" else 8))
            if kind == "fbp":
                interp, pc = rng.choice([("linear", 2), ("linear", 2), ("keys", 1), ("keys", 2)])
                case.update(interp=interp, pc=pc, angles=rng.choice(["even", "even", "golden"]))
            if kind in ("project", "lsgrad"):
                angular = rng.choice(["linear", "tent"])
                case.update(angular=angular)
        w = work(case)
        if w["bytes"] <= cap["bytes"] and w["flops"] <= cap["flops"]:
            return case


def _sizes(case):
    """(n, V) of the instances of an uneven batch."""
    rng = random.Random(case["sizes"])
    ns = [s for s in (256, 512, 1024, 2048) if s <= case["nmax"]]
    out = []
    for _ in range(case["count"]):
        n = rng.choice(ns)
        out.append((n, rng.randint(n // 2, 2 * n)))
    return out


def _angles(case):
    """Angle list of a golden-angle scan, sorted; None for even angles."""
    if case.get("angles") != "golden":
        return None
    j = np.arange(case["V"], dtype=np.float64)
    return np.sort(np.mod(j * (math.pi * (math.sqrt(5.0) - 1.0) / 2.0), math.pi))


_SHIFT = 2.5       # detector bins the rotation axis is off, raw counts
_MONOPOLE = 0.4    # width of the subtracted Gaussian, plain backprojection


def _options(case):
    """Keyword arguments of the case's plan."""
    kind = case["kind"]
    kw = {"max_batch": case["B"]}
    if kind == "fbp":
        kw["pad_cart"] = case["pc"]
        if case["interp"] == "keys":
            kw.update(interp="keys", taper="keys")
        ang = _angles(case)
        if ang is not None:
            kw["angles"] = ang
    elif kind == "counts":
        kw.update(apodization="hann", center_shift=_SHIFT)
    elif kind == "plain":
        kw.update(filter="none", monopole_width=_MONOPOLE)
    elif kind in ("project", "lsgrad"):
        kw.update(filter="none", adjoint=True, angular=case["angular"])
    return kw


# ---- inputs --------------------------------------------------------------------


def _ellipses(rng):
    out = []
    for _ in range(int(rng.integers(5, 13))):
        r, ph = 0.55 * math.sqrt(rng.random()), 2 * math.pi * rng.random()
        out.append((r * math.cos(ph), r * math.sin(ph), rng.uniform(0.04, 0.35), rng.uniform(0.04, 0.35),
                    rng.uniform(0, math.pi), rng.uniform(0.1, 1.0) * (1 if rng.random() < 0.7 else -1)))
    return out


def _sinogram(n, theta, rng, gen, shift=0.0):
    """Analytic parallel-beam projections [V][n] of random ellipses (Kak and
    Slaney's line integrals), 1 % noise; theta float32 on the GPU."""
    t = (torch.arange(n, device=theta.device, dtype=torch.float32) - n // 2 - shift) * (2.0 / n)
    y = torch.zeros(theta.numel(), n, device=theta.device)
    for x0, y0, a, b, rot, rho in _ellipses(rng):
        s2 = (a * torch.cos(theta - rot)) ** 2 + (b * torch.sin(theta - rot)) ** 2
        t0 = x0 * torch.cos(theta) + y0 * torch.sin(theta)
        d = s2[:, None] - (t[None, :] - t0[:, None]) ** 2
        y += (2.0 * rho * a * b / s2)[:, None] * d.clamp_(min=0.0).sqrt_()
    return y.add_(torch.randn(y.shape, generator=gen, device=y.device), alpha=0.01 * float(y.abs().max()))


def _image(n, rng):
    u = (torch.arange(n, device="cuda:0", dtype=torch.float32) - n // 2) * (2.0 / n)
    img = torch.zeros(n, n, device="cuda:0")
    for x0, y0, a, b, rot, rho in _ellipses(rng):
        dx, dy = u[None, :] - x0, u[:, None] - y0
        p = (dx * math.cos(rot) + dy * math.sin(rot)) / a
        q = (dy * math.cos(rot) - dx * math.sin(rot)) / b
        img += rho * (p * p + q * q <= 1.0)
    return img


def _theta(case, V):
    ang = _angles(case)
    if ang is None:
        ang = np.arange(V) * (math.pi / V)
    return torch.tensor(ang, dtype=torch.float32, device="cuda:0")


def _inputs(case, seed):
    """The tensors of a case, from the seed alone."""
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "uneven":
        return {"sinos": torch.cat([_sinogram(n, _theta({}, V), rng, gen).reshape(-1) for n, V in _sizes(case)])}
    n, V, B = case["n"], case["V"], case["B"]
    theta = _theta(case, V)
    x = {}
    if kind != "project":
        shift = _SHIFT if kind == "counts" else 0.0
        x["sino"] = torch.empty(B, V, n, device="cuda:0")
        for k in range(B):
            x["sino"][k] = _sinogram(n, theta, rng, gen, shift)
    if kind in ("project", "lsgrad"):
        x["img"] = torch.stack([_image(n, rng) for _ in range(B)])
    if kind == "counts":
        # Lambert-Beer counts at 1e5 photons over an uneven flat field
        y = x.pop("sino")
        x["dark"] = 100.0 + 5.0 * torch.rand(B, n, generator=gen, device="cuda:0")
        x["flat"] = 1e5 * (1.0 + 0.1 * torch.rand(B, n, generator=gen, device="cuda:0"))
        y *= 2.0 / y.abs().amax()
        x["counts"] = torch.exp_(y.neg_()).mul_((x["flat"] - x["dark"])[:, None, :]).add_(x["dark"][:, None, :])
    return x


def prepare(case, seed):
    st = {"case": case, **_inputs(case, seed)}
    if case["kind"] == "uneven":
        st["batch"] = P.Batch(_sizes(case))
        st["imgs"] = torch.empty(st["batch"].img_elems, device="cuda:0")
        st["ws"] = st["batch"].workspace()
        return st
    n, V, B = case["n"], case["V"], case["B"]
    st["plan"] = P.Plan(n, V, **_options(case))
    if case["kind"] in ("fbp", "counts", "plain"):
        st["out"] = torch.empty(B, n, n, device="cuda:0")
        st["ws"] = st["plan"].workspace(B)
    elif case["kind"] == "project":
        st["out"] = torch.empty(B, V, n, device="cuda:0")
        st["ws"] = st["plan"].workspace(B)
    elif case["kind"] == "lsgrad":
        st["img"].requires_grad_(True)
    elif case["kind"] == "brute":
        st["filtered"] = torch.empty(B, V, n, device="cuda:0")
        st["out"] = torch.empty(B, n, n, device="cuda:0")
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "uneven":
        return st["batch"].backproject(st["sinos"], st["imgs"], st["ws"])
    plan = st["plan"]
    if kind in ("fbp", "plain"):
        return plan.backproject(st["sino"], out=st["out"], workspace=st["ws"])
    if kind == "counts":
        return plan.backproject_counts(st["counts"], st["flat"], st["dark"], out=st["out"], workspace=st["ws"])
    if kind == "project":
        return plan.project(st["img"], out=st["out"], workspace=st["ws"])
    if kind == "lsgrad":
        r = AG.project(st["img"], plan) - st["sino"]
        loss = (r * r).sum()
        (grad,) = torch.autograd.grad(loss, st["img"])
        return loss.detach(), grad
    filtered = plan.ramp_filter(st["sino"], out=st["filtered"])
    return filtered, plan.bruteforce(filtered, out=st["out"])


# ---- work ----------------------------------------------------------------------


def _bst_flops(n, V, pc):
    """Transforms (5 L log2 L each, two real lines per complex one) and the
    polar-to-Cartesian interpolation of one slice."""
    M, G = 2 * n, pc * n
    fft = lambda L: 5.0 * L * math.log2(L)
    return V / 2 * fft(M) + G / 2 * fft(G) + n / 2 * fft(G) + 14.0 * math.pi / 8 * G * G


def work(case):
    kind = case["kind"]
    if kind == "uneven":
        sz = _sizes(case)
        return {"bytes": sum(4 * (V * n + n * n) for n, V in sz), "flops": sum(_bst_flops(n, V, 2) for n, V in sz)}
    n, V, B = case["n"], case["V"], case["B"]
    sino, img = 4 * V * n, 4 * n * n
    nbytes, flops = sino + img, _bst_flops(n, V, case.get("pc", 2))
    if kind == "counts":
        nbytes += 8 * n
    elif kind == "lsgrad":
        nbytes, flops = sino + 2 * img, 2 * flops
    elif kind == "brute":
        # the filtered sinogram is an output too; its convolution counted by transforms
        nbytes, flops = 2 * sino + img, 3.0 * V * n * n + V * 5.0 * 2 * n * math.log2(2 * n)
    return {"bytes": int(B * nbytes), "flops": float(B * flops)}


# ---- the same results in 64 bits ------------------------------------------------


class _Exact:
    """One slice's backprojection in float64 torch, a linear map of the
    sinogram [V][n] (monopole and normalisation aside)."""

    def __init__(self, n, V, pc=2, filter="ramp", interp="linear", angles=None, angular="linear", apodization="ramlak",
                 center_shift=0.0, dev="cuda:0"):
        self.n, self.V, self.M, self.G = n, V, 2 * n, pc * n
        f64 = dict(dtype=torch.float64, device=dev)
        M, G, Mh = self.M, self.G, n
        self.dt = self.d = 2.0 / n
        dsig, self.dk = 1.0 / (M * self.dt), 1.0 / (G * self.d)
        t = (torch.arange(n, **f64) - n // 2) * self.dt
        self.t = t
        sc = torch.sinc(t * dsig)
        if interp == "keys":
            self.w = 1.0 / (sc ** 3 * (3.0 * sc - 2.0 * torch.cos(math.pi * t * dsig)))
        else:
            self.w = 1.0 / sc ** 2
        m = torch.arange(Mh, **f64)
        K = torch.ones_like(m)
        if filter == "none":
            K = torch.where(m > 0, M * self.dt / m.clamp(min=1.0), torch.zeros_like(m))
        if apodization == "hann":
            K = K * 0.5 * (1.0 + torch.cos(2.0 * math.pi * m / M))
        self.kc = torch.polar(self.dt * K, 2.0 * math.pi * m * center_shift / M)
        self.dc = (1.0 if filter == "ramp" else 4.0 * math.asinh(1.0) / self.dk) / V
        th_j = None if angles is None else torch.tensor(angles, **f64)
        # Cartesian points (b, a): rows in FFT order, the half-plane's columns
        b = torch.arange(G, **f64)
        b = torch.where(b < G // 2, b, b - G)[:, None]
        a = torch.arange(G // 2, **f64)[None, :]
        rho = torch.sqrt(a * a + b * b)
        r = rho * (M / G)
        keep = (r < Mh + (1 if interp == "keys" else 0)) & (rho > 0)
        wide = torch.zeros_like(keep)
        if angular == "tent":
            wide = keep & (a * a + b * b < (V / math.pi) ** 2)
        th = torch.atan2(b, a)
        th = torch.where(b < 0, th + math.pi, th)
        lower = (b < 0).expand(G, G // 2)
        self.near = torch.nonzero((keep & ~wide).reshape(-1)).squeeze(1)
        pick = lambda x: x.expand(G, G // 2).reshape(-1)[self.near]
        thp, rp, lo = pick(th), pick(r), pick(lower)
        flip0 = torch.zeros_like(lo)
        if th_j is None:
            q = thp * (V / math.pi)
            j0 = q.floor().clamp(max=V - 1)
            f = q - j0
            j0 = j0.long()
        else:
            j0 = torch.searchsorted(th_j, thp, right=True) - 1
            flip0 = j0 < 0
            j0 = torch.where(flip0, V - 1, j0)
            left = torch.where(flip0, th_j[j0] - math.pi, th_j[j0])
            j1 = (j0 + 1) % V
            right = torch.where((j0 + 1 == V) & ~flip0, th_j[j1] + math.pi, th_j[j1])
            f = (thp - left) / (right - left)
        wrap = j0 + 1 == V
        j1 = torch.where(wrap, 0, j0 + 1)
        m0 = rp.floor()
        g = rp - m0
        m0 = m0.long()
        self.taps = []
        for j, wa, c in ((j0, 1.0 - f, lo ^ flip0), (j1, f, lo ^ (wrap & ~flip0))):
            for k in ((0, 1) if interp == "linear" else (-1, 0, 1, 2)):
                if interp == "linear":
                    wr = g if k else 1.0 - g
                else:
                    x = (g - k).abs()
                    wr = torch.where(x <= 1.0, (1.5 * x - 2.5) * x * x + 1.0, ((-0.5 * x + 2.5) * x - 4.0) * x + 2.0)
                mm = m0 + k
                cc = c ^ (mm < 0)
                mm = mm.abs()
                w = torch.where(mm < Mh, wa * wr, 0.0)
                self.taps.append((j * Mh + mm.clamp(max=Mh - 1), torch.stack((w, torch.where(cc, -w, w)), 1)))
        self.wide = torch.nonzero(wide.reshape(-1)).squeeze(1)
        if self.wide.numel():
            pick = lambda x: x.expand(G, G // 2).reshape(-1)[self.wide]
            q, h, rw, lo = pick(th) * (V / math.pi), V / (math.pi * pick(rho)), pick(r), pick(lower)
            first = (q - h).floor().long()
            cnt = (q + h).ceil().long() - first + 1
            pt = torch.repeat_interleave(torch.arange(q.numel(), device=dev), cnt)
            jc = torch.arange(pt.numel(), device=dev) - (cnt.cumsum(0) - cnt)[pt] + first[pt]
            w = (1.0 - (q[pt] - jc).abs() / h[pt]).clamp(min=0.0)
            tot = torch.zeros_like(q).index_add_(0, pt, w)
            w = w / tot[pt]
            cc = lo[pt] ^ (torch.div(jc, V, rounding_mode="floor") % 2 != 0)
            mw = rw.floor().long()
            gw = (rw - mw)[pt]
            mw = mw[pt]
            self.tent = []
            for k, wr in ((0, 1.0 - gw), (1, gw)):
                ww = torch.where(mw + k < Mh, w * wr, 0.0)
                self.tent.append((pt, (jc % V) * Mh + (mw + k).clamp(max=Mh - 1),
                                  torch.stack((ww, torch.where(cc, -ww, ww)), 1)))

    def __call__(self, y):
        n, M, G = self.n, self.M, self.G
        z = y * self.w
        z = torch.cat((z[:, n // 2:], torch.zeros(self.V, M - n, dtype=y.dtype, device=y.device), z[:, : n // 2]), 1)
        Y = torch.fft.rfft(z, dim=1)[:, : M // 2]
        S = torch.view_as_real((Y * self.kc).contiguous()).reshape(-1, 2)
        C = torch.zeros(G * (G // 2), 2, dtype=y.dtype, device=y.device)
        val = sum(S.index_select(0, i) * w for i, w in self.taps)
        C = C.index_copy(0, self.near, val)
        if self.wide.numel():
            tv = torch.zeros(self.wide.numel(), 2, dtype=y.dtype, device=y.device)
            for pt, i, w in self.tent:
                tv = tv.index_add(0, pt, S.index_select(0, i) * w)
            C = C.index_copy(0, self.wide, tv)
        origin = torch.stack((self.dc * self.dt * Y[:, 0].real.sum(), Y.new_zeros(()).real))[None, :]
        C = C.index_copy(0, torch.zeros(1, dtype=torch.long, device=y.device), origin)
        col = torch.fft.ifft(torch.view_as_complex(C).reshape(G, G // 2), dim=0) * G
        col = torch.cat((col[G - n // 2:], col[: n // 2]), 0)
        # real rows from the half-plane: column 0 once (its real part), the others twice
        re = torch.fft.ifft(torch.cat((0.5 * col[:, :1], col[:, 1:], torch.zeros_like(col)), 1), dim=1).real * (2.0 * G)
        return torch.cat((re[:, G - n // 2:], re[:, : n // 2]), 1) * self.dk ** 2

    def project(self, img):
        """R img = c B^T img, B^T by automatic differentiation."""
        y = torch.zeros(self.V, self.n, dtype=img.dtype, device=img.device, requires_grad=True)
        (g,) = torch.autograd.grad((self(y) * img).sum(), y)
        return g * self.c

    @property
    def c(self):
        return self.d * self.d / (self.dt * math.pi / self.V)


def _exact_brute(sino, n, V):
    """Band-limited ramp filter (linear convolution) and the direct sum of
    linearly interpolated projections of one slice."""
    dt = 2.0 / n
    f64 = dict(dtype=torch.float64, device=sino.device)
    k = torch.arange(2 * n, device=sino.device)
    k = torch.minimum(k, 2 * n - k)
    h = torch.where(k % 2 == 1, -1.0 / (math.pi * k.to(torch.float64) * dt).clamp(min=1e-300) ** 2, 0.0)
    h[0] = 1.0 / (4.0 * dt * dt)
    h[n] = 0.0
    filtered = torch.fft.irfft(torch.fft.rfft(sino, n=2 * n, dim=1) * torch.fft.rfft(h), n=2 * n, dim=1)[:, :n] * dt
    return filtered, _direct_sum(filtered, n, V, f64)


def _direct_sum(y, n, V, f64):
    u = torch.arange(n, **f64) - n // 2
    pad = torch.nn.functional.pad(y, (2, 3))
    img = torch.zeros(n, n, **f64)
    for j in range(V):
        th = j * math.pi / V
        s = (n / 2 + (u[None, :] * math.cos(th) + u[:, None] * math.sin(th))).clamp(-2.0, n + 1.0)
        i = s.floor()
        f = s - i
        i = i.long() + 2
        img += (1.0 - f) * pad[j][i] + f * pad[j][i + 1]
    return img * (math.pi / V)


def exact(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind == "uneven":
        ops, out, at = {}, [], 0
        for n, V in _sizes(case):
            op = _Exact(n, V)
            out.append(op(x["sinos"][at: at + n * V].reshape(V, n).double()).reshape(-1))
            at += n * V
        return torch.cat(out)
    n, V, B = case["n"], case["V"], case["B"]
    if kind == "brute":
        pairs = [_exact_brute(y.double(), n, V) for y in x["sino"]]
        return torch.stack([p[0] for p in pairs]), torch.stack([p[1] for p in pairs])
    kw = _options(case)
    for k in ("max_batch", "monopole_width", "adjoint", "taper"):
        kw.pop(k, None)
    op = _Exact(n, V, pc=kw.pop("pad_cart", 2), **kw)
    if kind == "fbp":
        return torch.stack([op(y.double()) for y in x["sino"]])
    if kind == "counts":
        out = []
        for k in range(B):
            fl, dk = x["flat"][k].double(), x["dark"][k].double()
            out.append(op(-torch.log((x["counts"][k].double() - dk) / (fl - dk))))
        return torch.stack(out)
    if kind == "plain":
        s = _MONOPOLE
        phi = torch.exp(-op.t ** 2 / (2 * s * s)) / (math.sqrt(2 * math.pi) * s)
        u2 = op.t[None, :] ** 2 + op.t[:, None] ** 2
        blob = math.pi / (math.sqrt(2 * math.pi) * s) * torch.special.i0e(u2 / (4 * s * s))
        out = []
        for y in x["sino"].double():
            m = y.sum() / (V * phi.sum())
            out.append(op(y - m * phi) + m * blob)
        return torch.stack(out)
    img = x["img"].double()
    if kind == "project":
        return torch.stack([op.project(f) for f in img])
    loss, grads = 0.0, []
    for f, g in zip(img, x["sino"].double()):
        r = op.project(f) - g
        loss = loss + (r * r).sum()
        grads.append(2.0 * op.c * op(r))
    return loss, torch.stack(grads)
