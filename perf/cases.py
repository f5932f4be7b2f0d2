"""Performance cases of the framework: what a user has it do, through its public entry points.

A case is a dict of plain values; "kind" names the entry point:

  objective    Context.objective: candidates -> (J, image), the evaluation of the outer loop
  grad         Context.objective_grad: J and its unrolled gradient
  envelope     Context.objective_grad_ex(mode="envelope"): J and the gradient at the fixed image
  mlem         Context.mlem: reconstructions for given attenuation maps
  project      Context.project: one attenuated projection per (map, image)
  backproject  Context.backproject: its transpose
  batch        Context.evaluate_batch: slices of uneven sizes in one call, objective and gradient
  gp_ei        Context.gp_ei: surrogate mean, deviation and expected improvement at many queries
  gp_search    Context.gp_chaos_search: the whole acquisition search of a cycle

Geometry: n x n image, `angles` over the full circle, `bins` detector bins, `samples` per ray, a field of
view of 25.6 cm (0.2 cm pixels at 128). Inputs are the simulation study's: head candidates from the search
box, an activity of 1 with hot disks of 4 inside the head, Poisson counts at 30 per bin.
"""
import math
import random

import numpy as np
import torch

from paper_2109_11920_amd import api

DELTA_R = 0.8
TRUE_HEAD = (7.5, 0.0, 1.2, 0.0, -0.3, 0.0, 0.150, 0.250)
BOX_LO = np.array([6.5, -1.5, -1.5, -1.5, -1.5, -1.5, 0.13, 0.20])
BOX_HI = np.array([8.5, 1.5, 1.5, 1.5, 1.5, 1.5, 0.17, 0.30])
LENGTH_GRID = np.geomspace(0.03, 3.0, 16)
# the outer loop's settings of the acquisition search
SEARCH = dict(n_global=16, n_local=32, centres=8, radius0=0.1, shrink=0.85, exclusion=0.02)
CHAINS = 4096


def _img(kind, n, angles, cands, iters=0, bins=None, samples=None, name=None):
    c = {"kind": kind, "n": n, "angles": angles, "bins": bins or n, "samples": samples or n, "cands": cands,
         "iters": iters}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest evaluation: one candidate map on a 64-pixel slice; launches and latency
        _img("objective", 64, 64, 1, 20, name="objective_1_n64"),
        # the plain method: one candidate at the study's image size, 50 iterations, image wanted
        _img("objective", 128, 128, 1, 50, name="objective_1_n128"),
        # the main line: a large batch of candidates on the 128-angle slice
        _img("objective", 128, 128, 256, 30, name="objective_256_n128"),
        # the same evaluation on sizes that are a multiple of nothing: a cropped slice, 37 candidates
        _img("objective", 109, 90, 37, 30, name="objective_37_n109_ragged"),
        # reconstructions for maps the caller brings, at an image size beyond one tile stage
        _img("mlem", 192, 96, 16, 20, name="mlem_16_n192"),
        # single projections and backprojections of a large image; a detector finer than the pixels, an odd
        # number of angles and rays longer than the image for the transpose
        _img("project", 256, 128, 32, name="project_32_n256"),
        _img("backproject", 120, 75, 24, bins=125, samples=150, name="backproject_24_n120_odd"),
        # gradient-based search: 64 candidates, exact gradient through 20 iterations
        _img("grad", 128, 128, 64, 20, name="grad_64_n128"),
        # a gradient-aware cycle of the outer loop at the paper's 72 angles
        _img("envelope", 128, 72, 64, 30, name="envelope_64_n128_a72"),
        # a study's slices in one call: uneven image sizes and angle counts, objective and gradient
        {"name": "batch_8_uneven", "kind": "batch", "slices": 8, "cands": 32, "iters": 40, "layout": 10, "ragged": False},
        # the surrogate at many queries, as a host-driven search asks for it
        {"name": "gp_ei_512", "kind": "gp_ei", "obs": 512, "queries": 65536, "d": 8},
        # the acquisition search of one cycle after five cycles of 64
        {"name": "gp_search_384", "kind": "gp_search", "obs": 384, "batch": 64, "d": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["objective", "objective", "objective", "grad", "envelope", "mlem", "project", "backproject",
                       "batch", "gp_ei", "gp_search"])
    if kind == "gp_ei":
        return {"kind": kind, "obs": _log_int(rng, 40, 512), "queries": _log_int(rng, 1000, 65536), "d": 8}
    if kind == "gp_search":
        return {"kind": kind, "obs": _log_int(rng, 64, 512), "batch": rng.choice([16, 32, 48, 64]), "d": 8}
    if kind == "batch":
        return {"kind": kind, "slices": rng.randint(2, 6), "cands": _log_int(rng, 4, 32), "iters": rng.randint(5, 30),
                "layout": rng.randint(0, 10 ** 6), "ragged": rng.random() < 0.5}
    n, angles = _log_int(rng, 48, 256), _log_int(rng, 36, 256)
    if rng.random() < 0.5:  # half of them on round sizes
        n, angles = rng.choice([64, 96, 128, 192, 256]), rng.choice([64, 72, 96, 128, 256])
    bins = samples = n
    if rng.random() < 0.3:
        bins = int(round(n * rng.uniform(0.8, 1.4)))
        samples = int(round(n * rng.uniform(1.0, 1.4)))
    iters = {"project": 0, "backproject": 0}.get(kind, _log_int(rng, 5, 50))
    c = _img(kind, n, angles, _log_int(rng, 1, 256), iters, bins, samples)
    # at most the largest listed case's work
    most = max(work(x)["flops"] for x in listed() if x["kind"] not in ("gp_ei", "gp_search", "batch"))
    while work(c)["flops"] > most and c["cands"] > 1:
        c["cands"] //= 2
    while work(c)["flops"] > most and c["iters"] > 1:
        c["iters"] //= 2
    return c


# ---------------------------------------------------------------- work
def _slices(case):
    """(n, angles) of a batch's slices."""
    r = random.Random(case["layout"])
    if case["ragged"]:
        return [(r.randint(72, 224), r.randint(48, 200)) for _ in range(case["slices"])]
    return [(r.choice([96, 128, 192, 256]), r.choice([64, 96, 128, 256])) for _ in range(case["slices"])]


def _image_work(kind, n, angles, bins, samples, cands, iters):
    """Bytes: arguments and results. Operations: a sample costs 10 in a projection or its transpose (8 of
    the bilinear read, the attenuation's multiply and add) and 12 in the attenuation's scan; a reverse
    step is a read of two images, a transpose, and a recomputed iteration."""
    s, px, rays = float(angles) * bins * samples * cands, 4.0 * n * n * cands, 4.0 * angles * bins
    if kind == "project" or kind == "backproject":
        return 2 * px + rays * cands, 22 * s
    if kind == "mlem":
        return 3 * px + rays, s * (12 + 10 + 20 * iters)
    fwd = s * (12 + 20 + 20 * iters)
    small = 72.0 * cands + rays
    if kind == "objective":
        return small + px, fwd
    if kind == "envelope":
        return small, fwd + 32 * s
    return small, fwd + s * (32 + 60 * iters)


def work(case):
    if case["kind"] == "gp_ei":
        n, m, d = case["obs"], case["queries"], case["d"]
        return {"bytes": 8.0 * (n * n / 2 + n * (d + 1) + m * (d + 3)), "flops": float(m) * n * (n + 1 + 3 * d + 4)}
    if case["kind"] == "gp_search":
        n, d = case["obs"], case["d"]
        m = CHAINS * (SEARCH["n_global"] + SEARCH["n_local"])
        return {"bytes": 8.0 * (n * n / 2 + n * (d + 1) + CHAINS * d), "flops": float(m) * n * (n + 1 + 3 * d + 4)}
    if case["kind"] == "batch":
        parts = [_image_work("grad", n, a, n, n, case["cands"], case["iters"]) for n, a in _slices(case)]
    else:
        parts = [_image_work(*(case[k] for k in ("kind", "n", "angles", "bins", "samples", "cands", "iters")))]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ---------------------------------------------------------------- the method in 64 bits (inputs and exact)
class _Ref:
    """The discretised method of one geometry in plain torch FP64; images are [n * n, C]."""

    def __init__(self, n, angles, bins, samples, pixel, device):
        self.n, self.angles, self.bins, self.samples, self.dx, self.dev = n, angles, bins, samples, pixel, device
        f64 = dict(dtype=torch.float64, device=device)
        sig = (torch.arange(bins, **f64) - (bins - 1) / 2) * (n / bins)
        tau = torch.arange(samples, **f64) - (samples - 1) / 2
        self.blocks = []  # (first angle, angles, taps), about 2^21 samples each
        step = max(1, (1 << 21) // (bins * samples))
        for a0 in range(0, angles, step):
            a1 = min(angles, a0 + step)
            phi = torch.arange(a0, a1, **f64) * (2 * math.pi / angles)
            c, s = torch.cos(phi)[:, None, None], torch.sin(phi)[:, None, None]
            u = (sig[None, :, None] * c - tau[None, None, :] * s + (n - 1) / 2).reshape(-1)
            v = (sig[None, :, None] * s + tau[None, None, :] * c + (n - 1) / 2).reshape(-1)
            l0, i0 = torch.floor(u), torch.floor(v)
            fu, fv = u - l0, v - i0
            taps = []
            for di, dl, w in ((0, 0, (1 - fu) * (1 - fv)), (0, 1, fu * (1 - fv)), (1, 0, (1 - fu) * fv), (1, 1, fu * fv)):
                i, l = (i0 + di).long(), (l0 + dl).long()
                ok = (i >= 0) & (i < n) & (l >= 0) & (l < n)
                taps.append((torch.where(ok, i * n + l, 0), torch.where(ok, w, 0.0)[:, None]))
            self.blocks.append((a0, a1, taps))

    def sample(self, k, img):
        """W img on block k: [angles, bins, samples, C]."""
        a0, a1, taps = self.blocks[k]
        out = sum(w * img.index_select(0, i) for i, w in taps)
        return out.view(a1 - a0, self.bins, self.samples, -1)

    def spread(self, k, field, out):
        """out += W^T field on block k."""
        f = field.reshape(-1, field.shape[-1])
        for i, w in self.blocks[k][2]:
            out.index_add_(0, i, w * f)

    def attenuation(self, mu):
        att = []
        for k in range(len(self.blocks)):
            m = self.sample(k, mu)
            later = torch.flip(torch.cumsum(torch.flip(m, [2]), 2), [2]) - m
            att.append(torch.exp(-self.dx * (0.5 * m + later)))
        return att

    def project(self, att, img):
        return self.dx * torch.cat([(att[k] * self.sample(k, img)).sum(2) for k in range(len(att))])

    def backproject(self, att, sino):
        out = torch.zeros(self.n * self.n, sino.shape[-1], dtype=torch.float64, device=self.dev)
        for k, (a0, a1, _) in enumerate(self.blocks):
            self.spread(k, att[k] * sino[a0:a1, :, None, :], out)
        return self.dx * out

    def raster(self, theta, delta_r):
        """theta [C, 8], delta_r a number or [C, 1, 1, 1] -> mu [n * n, C]."""
        n, dx = self.n, self.dx
        sub = (torch.arange(4 * n, dtype=torch.float64, device=self.dev) - (4 * n - 1) / 2) * (dx / 4)
        r = torch.sqrt(sub[None, :] ** 2 + sub[:, None] ** 2)
        x = torch.where(r > 1e-12, sub[None, :] / r.clamp_min(1e-300), 1.0)
        p = [torch.ones_like(x), x]
        for m in range(1, 5):
            p.append(((2 * m + 1) * x * p[m] - m * p[m - 1]) / (m + 1))
        d = sum(theta[:, m, None, None] * p[m] for m in range(6)) - r
        h = dx / 4

        def mean_cover(e):
            t = torch.clamp(e / h + 0.5, 0.0, 1.0)
            return (t * t * (3 - 2 * t)).view(-1, n, 4, n, 4).mean((2, 4))

        fb, fo = mean_cover(d), mean_cover(d + delta_r)
        mu = theta[:, 6, None, None] * fb + theta[:, 7, None, None] * (fo - fb)
        return mu.reshape(len(theta), -1).T.contiguous()

    @staticmethod
    def ratio(meas, y):
        return torch.where(y > 0, meas[..., None] / torch.where(y > 0, y, 1.0), 0.0)

    def mlem(self, att, meas, iters, img, keep=None):
        s = self.backproject(att, torch.ones(self.angles, self.bins, img.shape[1], dtype=torch.float64, device=self.dev))
        pos = s > 0
        safe = torch.where(pos, s, 1.0)
        for _ in range(iters):
            y = self.project(att, img)
            r = self.ratio(meas, y)
            b = self.backproject(att, r)
            if keep is not None:
                keep.append((img, y, r, b))
            img = torch.where(pos, img * b / safe, 0.0)
        return img, pos, safe

    @staticmethod
    def score(meas, y):
        S = meas[..., None]
        t = torch.where(S > 0, y - S * torch.log(torch.where(y > 0, y, 1.0)), y)
        bad = ((y <= 0) & (S > 0)).any(0).any(0)
        J = t.sum((0, 1)) + torch.lgamma(meas + 1.0).sum()
        return torch.where(bad, math.inf, J)

    def evaluate(self, meas, theta, iters, grad=None):
        """(J [C], image [n * n, C], gradient [C, 9] for grad "unrolled" or "envelope")."""
        if grad:
            theta = theta.clone().requires_grad_(True)
        dr = torch.full((len(theta), 1, 1), DELTA_R, dtype=torch.float64, device=self.dev, requires_grad=bool(grad))
        mu = self.raster(theta, dr)
        with torch.no_grad():
            att = self.attenuation(mu.detach())
            kept = [] if grad == "unrolled" else None
            one = torch.ones(self.n * self.n, len(theta), dtype=torch.float64, device=self.dev)
            img, pos, safe = self.mlem(att, meas, iters, one, kept)
            y = self.project(att, img)
            J = self.score(meas, y)
            if not grad:
                return J, img, None
            ybar = torch.where(y > 0, 1.0 - self.ratio(meas, y), (meas == 0).double()[..., None])
            # att_bar is kept as a list of (weights of a sinogram, image) terms, summed block by block at the end
            terms = [(ybar, img)]
            if grad == "unrolled":
                fbar, sbar = self.backproject(att, ybar), torch.zeros_like(img)
                for F, yn, rn, b in reversed(kept):
                    sbar -= torch.where(pos, fbar * (F * b / safe) / safe, 0.0)
                    bbar = torch.where(pos, fbar * F / safe, 0.0)
                    fbar = torch.where(pos, fbar * b / safe, 0.0)
                    terms.append((rn, bbar))
                    rbar = self.project(att, bbar)
                    yb = torch.where(yn > 0, -rbar * rn / torch.where(yn > 0, yn, 1.0), 0.0)
                    terms.append((yb, F))
                    fbar = fbar + self.backproject(att, yb)
                terms.append((torch.ones_like(ybar), sbar))
            mubar = torch.zeros_like(one)
            for k, (a0, a1, _) in enumerate(self.blocks):
                ab = sum(w[a0:a1, :, None, :] * self.sample(k, g) for w, g in terms)
                lbar = -att[k] * self.dx * ab
                before = torch.cumsum(lbar, 2) - lbar
                self.spread(k, self.dx * (0.5 * lbar + before), mubar)
        mu.backward(mubar)
        return J, img, torch.cat([theta.grad, dr.grad.view(-1, 1)], 1)


def _device():
    return torch.device("cuda", 0)


def _pixel(n):
    return float(np.float32(25.6 / n))


def _heads(rng, count):
    return torch.tensor(BOX_LO + (BOX_HI - BOX_LO) * rng.random((count, 8)), dtype=torch.float32)


def _activity(rng, n, inside):
    """1 inside the head, three hot disks of 4 (radius 0.8 to 1.5 cm); inside [n, n] in 0..1."""
    x = (np.arange(n) - (n - 1) / 2) * _pixel(n)
    f = inside.copy()
    for _ in range(3):
        r, rad, phi = rng.uniform(0.8, 1.5), rng.uniform(0.0, 4.5), rng.uniform(0.0, 2 * math.pi)
        d2 = (x[None, :] - rad * math.cos(phi)) ** 2 + (x[:, None] - rad * math.sin(phi)) ** 2
        f = np.where(d2 < r * r, 4.0 * inside, f)
    return f


def _measure(rng, ref):
    """A noisy sinogram [angles, bins] of the true head at 30 counts per bin (float32, on the device)."""
    theta = torch.tensor([TRUE_HEAD], dtype=torch.float64, device=ref.dev)
    mu = ref.raster(theta, DELTA_R)
    inside = torch.clamp(mu[:, 0] / TRUE_HEAD[6], 0.0, 1.0).view(ref.n, ref.n).cpu().numpy()
    img = torch.tensor(_activity(rng, ref.n, inside), dtype=torch.float64, device=ref.dev).view(-1, 1)
    y = ref.project(ref.attenuation(mu), img)[..., 0].cpu().numpy()
    y = np.maximum(y, 0.0) * (30.0 * y.size / y.sum())
    return torch.tensor(rng.poisson(np.round(y, 6)).astype(np.float32), device=ref.dev)


def _ref(case):
    return _Ref(case["n"], case["angles"], case["bins"], case["samples"], _pixel(case["n"]), _device())


def _inputs(case, seed, ref):
    """The arguments of an image case: (attenuation maps or candidates, second argument)."""
    rng = np.random.default_rng([seed, 1])
    C, n, kind = case["cands"], case["n"], case["kind"]
    if kind in ("objective", "grad", "envelope"):
        meas = _measure(rng, ref)
        return _heads(rng, C).to(ref.dev), meas
    mu = torch.cat([ref.raster(h[None].double().to(ref.dev), DELTA_R) for h in _heads(rng, C)], 1)
    mu = mu.T.reshape(C, n, n).float().contiguous()
    if kind == "mlem":
        return mu, _measure(rng, ref)
    if kind == "project":
        inside = (mu > 0.05).double().cpu().numpy()
        img = np.stack([_activity(rng, n, x) * rng.uniform(0.8, 1.2, (n, n)) for x in inside])
        return mu, torch.tensor(img, dtype=torch.float32, device=ref.dev)
    # ratios of measured to expected counts: around 1, some zeros
    sino = rng.poisson(30.0, (C, case["angles"], case["bins"])) / 30.0
    sino[rng.random(sino.shape) < 0.2] = 0.0
    return mu, torch.tensor(sino, dtype=torch.float32, device=ref.dev)


def _observations(case, seed):
    """Unit-box points and objective values as a search leaves them: half spread out, half gathered
    around the smallest value."""
    rng = np.random.default_rng([seed, 2])
    n, d = case["obs"], case["d"]
    best = rng.uniform(0.25, 0.75, d)
    u = rng.random((n, d))
    half = n // 2
    u[half:] = np.clip(best + rng.normal(0.0, 0.12, (n - half, d)), 0.0, 1.0)
    scale = rng.uniform(200.0, 2000.0, d)
    y = 33000.0 + ((u - best) ** 2) @ scale + 120.0 * np.sin(5.0 * u).sum(1)
    z = rng.uniform(0.01, 0.99, (CHAINS, d))
    q = rng.random((case.get("queries", 1), d))
    return u, y, z, q


_CONTEXT = []


def _context():
    """The program's one context."""
    if not _CONTEXT:
        _CONTEXT.append(api.Context(0))
    return _CONTEXT[0]


def prepare(case, seed):
    st = {"case": case, "ctx": _context()}
    if case["kind"] in ("gp_ei", "gp_search"):
        u, y, z, q = _observations(case, seed)
        f64 = dict(dtype=torch.float64, device=_device())
        st["model"] = api.gp_fit(u, y, LENGTH_GRID, n_select=256, noise=1e-6)
        st["model"].on(_device())
        st["best"] = float(y.min())
        st["z"], st["q"], st["taken"] = torch.tensor(z, **f64), torch.tensor(q, **f64), torch.tensor(u, **f64)
        return st
    if case["kind"] == "batch":
        st["slices"] = []
        for k, (n, angles) in enumerate(_slices(case)):
            rng = np.random.default_rng([seed, 3, k])
            ref = _Ref(n, angles, n, n, _pixel(n), _device())
            meas = _measure(rng, ref)
            g = api.Geometry(n, angles, n, n, _pixel(n))
            st["slices"].append(api.SliceBatch.make(g, meas, _heads(rng, case["cands"]).to(_device()), True))
        st["stream"] = torch.cuda.Stream(_device())
        return st
    st["geom"] = api.Geometry(case["n"], case["angles"], case["bins"], case["samples"], _pixel(case["n"]))
    st["a"], st["b"] = _inputs(case, seed, _ref(case))
    return st


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "gp_ei":
        ei, mu, sd = ctx.gp_ei(state["model"], state["q"], state["best"], 0.0, want_mu_sigma=True)
        return {"ei": ei, "mu": mu, "sigma": sd}
    if kind == "gp_search":
        props, vmax, queries = ctx.gp_chaos_search(state["model"], state["best"], 0.0, state["z"], state["taken"],
                                                   case["batch"], per_step=max(4 * case["batch"], 256), **SEARCH)
        return {"proposals": props, "max_ei": vmax, "queries": queries}
    if kind == "batch":
        # the batch is captured once per shape and replayed; a stream other than the default one allows it
        now = torch.cuda.current_stream()
        state["stream"].wait_stream(now)
        with torch.cuda.stream(state["stream"]):
            ctx.evaluate_batch(state["slices"], DELTA_R, case["iters"], 5)
        now.wait_stream(state["stream"])
        return [{"J": s.obj, "grad": s.grad, "status": s.status} for s in state["slices"]]
    g, a, b = state["geom"], state["a"], state["b"]
    if kind == "objective":
        J, img, status = ctx.objective(g, b, a, DELTA_R, case["iters"], want_image=True)
        return {"J": J, "image": img, "status": status}
    if kind == "grad":
        J, grad, status = ctx.objective_grad(g, b, a, DELTA_R, case["iters"], 5)
        return {"J": J, "grad": grad, "status": status}
    if kind == "envelope":
        J, grad, status = ctx.objective_grad_ex(g, b, a, DELTA_R, case["iters"], mode="envelope")
        return {"J": J, "grad": grad, "status": status}
    if kind == "mlem":
        return ctx.mlem(g, a, b, case["iters"])
    if kind == "project":
        return ctx.project(g, a, b)
    return ctx.backproject(g, a, b)


# ---------------------------------------------------------------- outputs in 64 bits
def _ei_of(case, seed):
    """The surrogate's (EI, mean, deviation) at rows of a unit-box tensor, and the data it was fitted to."""
    u, y, z, q = _observations(case, seed)
    f64 = dict(dtype=torch.float64, device=_device())
    m0, s = y.mean(), y.std(ddof=1) or 1.0
    t = (y - m0) / s

    def fit(U, T, length):
        d2 = ((U[:, None, :] - U[None, :, :]) ** 2).sum(2)
        L = np.linalg.cholesky(np.exp(-d2 / (2 * length * length)) + 1e-6 * np.eye(len(U)))
        w = np.linalg.solve(L, T)
        return L, w, -0.5 * w @ w - np.log(np.diag(L)).sum()

    pick = np.argsort(y, kind="stable")[:256]
    yp = y[pick]
    tp = (yp - yp.mean()) / (yp.std(ddof=1) or 1.0)
    length = max((fit(u[pick], tp, h)[2], -k, h) for k, h in enumerate(LENGTH_GRID))[2]
    L, w, _ = fit(u, t, length)
    Lg, wg, U = torch.tensor(L, **f64), torch.tensor(w, **f64), torch.tensor(u, **f64)

    def ei_of(Q):
        out = []
        for c in Q.split(16384):
            K = torch.exp(-((c[:, None, :] - U[None, :, :]) ** 2).sum(2) / (2 * length * length))
            v = torch.linalg.solve_triangular(Lg, K.T, upper=False)
            mu, sd = m0 + s * (v.T @ wg), s * torch.sqrt(torch.clamp(1.0 - (v * v).sum(0), min=0.0))
            g = (y.min() - mu) / torch.where(sd > 0, sd, 1.0)
            ei = sd * (g * 0.5 * torch.erfc(-g / math.sqrt(2.0)) + torch.exp(-0.5 * g * g) / math.sqrt(2 * math.pi))
            out.append(torch.stack([torch.where(sd > 0, ei.clamp_min(0.0), (y.min() - mu).clamp_min(0.0)), mu, sd]))
        return torch.cat(out, 1)

    return ei_of, u, z, q


def _greedy(pts, vals, q, taken):
    ref, chosen = [np.asarray(t) for t in taken], []
    for i in np.argsort(-vals, kind="stable"):
        if len(chosen) == q:
            break
        if not ref or np.min(((np.asarray(ref) - pts[i]) ** 2).sum(1)) >= SEARCH["exclusion"] ** 2:
            chosen.append(int(i))
            ref.append(pts[i])
    return chosen


def _search(case, seed):
    ei_of, taken, z, _ = _ei_of(case, seed)
    keep, pts, vals = max(4 * case["batch"], 256), [], []

    def values(U):
        return ei_of(torch.tensor(U, dtype=torch.float64, device=_device()))[0].cpu().numpy()

    def pool(U, e):
        top = np.sort(np.argsort(-e, kind="stable")[:keep])
        pts.append(U[top])
        vals.append(e[top])

    for _ in range(SEARCH["n_global"]):
        pool(z, values(z))
        z = 4.0 * z * (1.0 - z)
    allp, allv = np.concatenate(pts), np.concatenate(vals)
    pick = _greedy(allp, allv, min(max(SEARCH["centres"], case["batch"]), CHAINS), [])
    C, Ce, r = allp[pick].copy(), allv[pick].copy(), SEARCH["radius0"]
    per = CHAINS // len(C)
    for _ in range(SEARCH["n_local"]):
        zz = z[:per * len(C)].reshape(len(C), per, -1)
        U = np.clip(C[:, None, :] + r * (2.0 * zz - 1.0), 0.0, 1.0).reshape(per * len(C), -1)
        e = values(U)
        pool(U, e)
        j = np.argmax(e.reshape(len(C), per), axis=1) + per * np.arange(len(C))
        better = e[j] > Ce
        C[better], Ce[better] = U[j][better], e[j][better]
        z = 4.0 * z * (1.0 - z)
        r *= SEARCH["shrink"]
    allp, allv = np.concatenate(pts), np.concatenate(vals)
    queries = CHAINS * SEARCH["n_global"] + per * len(C) * SEARCH["n_local"]
    return {"proposals": allp[_greedy(allp, allv, case["batch"], taken)], "max_ei": float(allv.max()), "queries": queries}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gp_ei":
        ei_of, _, _, q = _ei_of(case, seed)
        ei, mu, sd = ei_of(torch.tensor(q, dtype=torch.float64, device=_device()))
        return {"ei": ei, "mu": mu, "sigma": sd}
    if kind == "gp_search":
        return _search(case, seed)
    if kind == "batch":
        return None  # its slices are the other cases' sizes; all of them in 64 bits take over 20 seconds
    ref = _ref(case)
    a, b = _inputs(case, seed, ref)
    C, n = case["cands"], case["n"]
    # candidates at a time: about 4 GB for one field of the samples
    step = max(1, min(32, (1 << 29) // (case["angles"] * case["bins"] * case["samples"])))
    parts = []
    for c in range(0, C, step):
        x = a[c:c + step].double()
        if kind in ("objective", "grad", "envelope"):
            J, img, grad = ref.evaluate(b.double(), x, case["iters"],
                                        {"grad": "unrolled", "envelope": "envelope"}.get(kind))
            parts.append((J, img.T.reshape(-1, n, n), grad))
            continue
        att = ref.attenuation(x.reshape(len(x), -1).T.contiguous())
        if kind == "mlem":
            one = torch.ones(n * n, len(x), dtype=torch.float64, device=ref.dev)
            out = ref.mlem(att, b.double(), case["iters"], one)[0].T.reshape(-1, n, n)
        elif kind == "project":
            out = ref.project(att, b[c:c + step].double().reshape(len(x), -1).T.contiguous()).permute(2, 0, 1)
        else:
            out = ref.backproject(att, b[c:c + step].double().permute(1, 2, 0).contiguous()).T.reshape(-1, n, n)
        parts.append((out,))
    whole = [torch.cat(p).contiguous() if p[0] is not None else None for p in zip(*parts)]
    if kind == "objective":
        return {"J": whole[0], "image": whole[1], "status": None}
    if kind in ("grad", "envelope"):
        return {"J": whole[0], "grad": whole[2][:, :8].contiguous() if kind == "grad" else whole[2], "status": None}
    return whole[0]
