"""Timing cases of the framework: what its users run, through the package's entry points.

`listed()` gives the fixed cases, `draw(rng)` further ones of the same ranges.
`prepare(case, seed)` makes what a program holds before the call (sample
locations and values on the device, the plan, batch or network), `run(state)`
is one pass, `work(case)` the bytes and operations it cannot do without, and
`exact(case, seed)` what it returns in 64 bits, from plain torch and numpy.

Every input is drawn on the device from the seed: polar-format annular-sector
rasters (pulses at jittered angles, range wavenumbers around 2.25 n) with the
Fourier data of 40 point scatterers plus speckle, jittered 1D rasters, and
noisy grids for the dense frame approximation.
"""
from __future__ import annotations

import math
import os
import random

import numpy as np
import torch

DEV = "cuda"
NPARAM = 6337
NET = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1706_08575_amd", "models", "mlp_sas.bin")
PAIR_BUDGET = 1 << 25   # pairs formed at once by exact()


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------

def listed():
    return [
        # one 1D reconstruction of a jittered raster: the smallest call, all latency
        dict(name="line_256_f64", kind="image", dim=1, n=256, G=512, m=512, dtype="f64", weights="plain"),
        # one sonar image from new samples: binning, weights, spreading, transform
        dict(name="image_512", kind="image", dim=2, n=512, G=1024, pulses=256, m=256 * 512, dtype="f32",
             weights="plain"),
        # the large survey image, 8.4 M samples
        dict(name="image_4096", kind="image", dim=2, n=4096, G=8192, pulses=2048, m=2048 * 4096, dtype="f32",
             weights="plain"),
        # double precision, an image size that is no power of two, a last pulse cut short
        dict(name="image_1000_f64", kind="image", dim=2, n=1000, G=2048, pulses=611, m=611 * 1237 - 13, dtype="f64",
             weights="plain"),
        # the next ping on a raster whose weights are already there
        dict(name="ping_1024", kind="ping", dim=2, n=1024, G=2048, pulses=512, m=512 * 2048, dtype="f32",
             weights="plain"),
        # image to samples: the data model of iterative reconstructions
        dict(name="forward_4096", kind="forward", dim=2, n=4096, G=8192, pulses=2048, m=2048 * 4096, dtype="f32",
             weights="none"),
        # banded coefficient matrix, 15 entries a column
        dict(name="band8_512", kind="image", dim=2, n=512, G=1024, pulses=256, m=256 * 512, dtype="f32",
             weights="band", r=8),
        # iterative density compensation, the comparator of the frame weights
        dict(name="density20_512", kind="image", dim=2, n=512, G=1024, pulses=256, m=256 * 512, dtype="f32",
             weights="density", iters=20),
        # weights from the trained network, accepted by the audit
        dict(name="learned_1024", kind="image", dim=2, n=1024, G=2048, pulses=512, m=512 * 2048, dtype="f32",
             weights="learned"),
        # pings of uneven size in one batch, new rasters
        dict(name="batch_16", kind="batch", items=16, pattern=5, lo=16.0, hi=20.0),
        # training data and one gradient of the network: features, labels, forward and backward
        dict(name="train_65536", kind="train", n=256, pulses=128, m=128 * 512),
        # dense frame approximation, the accuracy reference of small rasters
        dict(name="frame_32", kind="frame", n=32, side=30),
    ]


def _image_size(rng, lo, hi):
    """A grid of 2^j points and an image of half its edge, or an even size near that."""
    G = 1 << rng.randint(lo, hi)
    if rng.random() < 0.5:
        return G // 2, G
    return 2 * rng.randint(int(0.2 * G), int(0.27 * G)), G


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["line", "image", "image", "image", "ping", "forward", "band", "density", "learned", "batch",
                       "train", "frame"])
    if kind == "line":
        n, G = _image_size(rng, 5, 13)
        return dict(kind="image", dim=1, n=n, G=G, m=_log(rng, n / 2, 8 * n), dtype=rng.choice(["f32", "f64"]),
                    weights="plain")
    if kind in ("image", "ping", "forward"):
        dtype = rng.choice(["f32", "f32", "f64"])
        n, G = _image_size(rng, 7, 12 if dtype == "f32" else 11)
        m = _log(rng, max(256, n * n / 16), min(3 << 20, 4 * n * n))
        w = {"image": "plain", "ping": rng.choice(["plain", "none"]), "forward": "none"}[kind]
        return dict(kind=kind, dim=2, n=n, G=G, pulses=max(1, int(math.sqrt(m / 2) * rng.uniform(0.7, 1.4))), m=m,
                    dtype=dtype, weights=w)
    if kind in ("band", "density", "learned"):
        n, G = _image_size(rng, 7, 10 if kind != "learned" else 11)
        # the samples of a band have to stay apart for its columns to be independent
        m = _log(rng, n * n / 8, (0.5 if kind == "band" else 1.5) * n * n)
        c = dict(kind="image", dim=2, n=n, G=G, pulses=max(1, int(math.sqrt(m / 2) * rng.uniform(0.7, 1.4))), m=m,
                 dtype="f32" if kind == "learned" else rng.choice(["f32", "f32", "f64"]), weights=kind)
        if kind == "band":
            # the paper's bands are r = 8 and 12
            c.update(r=rng.choice([2, 3, 5, 8, 12]), pulses=max(1, int(math.sqrt(m / 2))))
        if kind == "density":
            c.update(iters=rng.choice([5, 10, 20, 30]))
        return c
    if kind == "batch":
        return dict(kind="batch", items=rng.randint(2, 16), pattern=rng.randint(0, 10 ** 6), lo=12.0,
                    hi=rng.choice([16.0, 18.0, 19.0]))
    if kind == "train":
        p = rng.randint(32, 128)
        return dict(kind="train", n=256, pulses=p, m=p * 512 - rng.randint(0, 300))
    n = rng.choice([8, 16, 16, 32])
    return dict(kind="frame", n=n, side=rng.randint(n // 2, min(34, n + n // 4)))


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _sector(g, n, pulses, m, jitter=1.0):
    """m samples of a polar-format raster, the last pulse cut short."""
    per = -(-m // pulses)
    k0 = 2.25 * n
    kc = k0 * (0.8 * math.cos(math.radians(10.0)) + 1.2) / 2.0
    p = torch.arange(pulses, device=DEV, dtype=torch.float64)
    th = torch.deg2rad(-10.0 + 20.0 * (p + 0.5) / pulses) + math.radians(0.02 * jitter) * _normal(g, pulses)
    r = k0 * (0.8 + 0.4 * (torch.arange(per, device=DEV, dtype=torch.float64) + 0.5) / per)
    k = torch.stack([(r[None, :] * torch.cos(th)[:, None] - kc).reshape(-1),
                     (r[None, :] * torch.sin(th)[:, None]).reshape(-1)], dim=1)
    return (k + 0.01 * jitter * _normal(g, *k.shape))[:m].contiguous()


def _scene_data(g, k, scatterers=40):
    """Fourier data of point scatterers, plus speckle of variance 1."""
    d = k.shape[1]
    pos = _uniform(g, -0.4, 0.4, scatterers, d)
    mag, ph = _uniform(g, 5.0, 20.0, scatterers), _uniform(g, 0.0, 2 * math.pi, scatterers)
    out = _normal(g, k.shape[0], 2) * math.sqrt(0.5)
    for s in range(scatterers):
        a = ph[s] - 2 * math.pi * (k * pos[s]).sum(1)
        out[:, 0] += mag[s] * torch.cos(a)
        out[:, 1] += mag[s] * torch.sin(a)
    return torch.view_as_complex(out)


def _locations(case, g):
    if case["dim"] == 1:
        m = case["m"]
        j = torch.arange(m, device=DEV, dtype=torch.float64)
        return (j - m // 2 + _uniform(g, -0.25, 0.25, m)).reshape(m, 1)
    return _sector(g, case["n"], case["pulses"], case["m"])


def _batch_items(case):
    """(n, m, pulses) of every item."""
    r = random.Random(case["pattern"])
    out = []
    for _ in range(case["items"]):
        m = int(round(2.0 ** r.uniform(case["lo"], case["hi"])))
        per = int(math.ceil(math.sqrt(2 * m)))
        out.append((r.choice([256, 512, 1024, 2048]), m, -(-m // per)))
    return out


def _batch_inputs(case, seed):
    g = _gen(seed)
    ks = [_sector(g, n, p, m) for n, m, p in _batch_items(case)]
    return ks, [_scene_data(g, k, 12).to(torch.complex64) for k in ks]


def _cdtype(case):
    return torch.complex64 if case["dtype"] == "f32" else torch.complex128


def _image_inputs(case, seed):
    g = _gen(seed)
    k = _locations(case, g)
    return k, _scene_data(g, k).to(_cdtype(case))


def _forward_inputs(case, seed):
    g = _gen(seed)
    k = _locations(case, g)
    n = case["n"]
    x = (torch.arange(n, device=DEV, dtype=torch.float64) - n // 2) / n
    e = torch.exp(-x * x / 0.05)
    img = torch.view_as_complex(_normal(g, n, n, 2) * (e[:, None] * e[None, :])[:, :, None])
    return k, img.to(_cdtype(case))


def _frame_inputs(case, seed):
    """Noisy grid of Sec. V-A with the data of sin(4 pi x1) sin(2 pi x2)."""
    g = _gen(seed)
    s = case["side"]
    a = torch.arange(s, device=DEV, dtype=torch.float64) - s // 2
    k = torch.stack([t.reshape(-1) for t in torch.meshgrid(a, a, indexing="ij")], dim=1)
    k = (k + _uniform(g, -0.25, 0.25, s * s, 2)).contiguous()
    f = [(torch.sinc(k[:, a] - c) - torch.sinc(k[:, a] + c)) / 2j for a, c in ((0, 2.0), (1, 1.0))]
    noise = torch.view_as_complex(0.01 * _normal(g, s * s, 2))
    return k, (f[0] * f[1] + noise).contiguous()


def _train_inputs(case, seed):
    """A training raster with its own jitter scale, and initial parameters."""
    g = _gen(seed)
    js = float(2.0 ** _uniform(g, -1.0, 1.0, 1).item())
    k = _sector(g, case["n"], case["pulses"], case["m"], js)
    r = np.random.default_rng(seed)
    params = {}
    for name, shape, fan in (("W1", (32, 64), 32), ("b1", (64,), 32), ("W2", (64, 64), 64), ("b2", (64,), 64),
                             ("W3", (64, 1), 64), ("b3", (1,), 64)):
        v = r.uniform(-1, 1, size=shape) / math.sqrt(fan)
        params[name] = (0.1 * v if name in ("W3", "b3") else v).astype(np.float32)
    return k, params


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def prepare(case, seed):
    from paper_1706_08575_amd.batch import Batch
    from paper_1706_08575_amd.ftcg import Plan
    from paper_1706_08575_amd.mlp import Mlp

    kind = case["kind"]
    st = {"kind": kind}
    if kind == "batch":
        ks, fs = _batch_inputs(case, seed)
        items = _batch_items(case)
        st.update(plan=Batch([n for n, _, _ in items]), m=[m for _, m, _ in items], k=torch.cat(ks), f=torch.cat(fs))
        return st
    if kind == "train":
        k, params = _train_inputs(case, seed)
        st.update(net=Mlp(params), k=k)
        return st
    if kind == "frame":
        k, f = _frame_inputs(case, seed)
        st.update(plan=Plan(case["n"], dim=2, dtype="f64", weights="none"), k=k, f=f)
        return st
    k, f = (_forward_inputs if kind == "forward" else _image_inputs)(case, seed)
    P = Plan(case["n"], dim=case["dim"], sigma=case["G"] / case["n"], dtype=case["dtype"], weights=case["weights"])
    if case["weights"] == "band":
        P.set_band(case["r"])
    if case["weights"] == "density":
        P.set_density_iterations(case["iters"])
    if case["weights"] == "learned":
        net = Mlp()
        with open(NET, "rb") as fh:
            net.load(fh.read())
        P.set_mlp(net, audit_threshold=1.0)
    if kind != "image":
        P.set_points(k)
    st.update(plan=P, k=k, f=f)
    return st


def run(state):
    kind = state["kind"]
    if kind == "image":
        state["plan"].set_points(state["k"])
        return state["plan"].execute(state["f"])
    if kind == "ping":
        return state["plan"].execute(state["f"])
    if kind == "forward":
        return state["plan"].forward(state["f"])
    if kind == "batch":
        state["plan"].set_points(state["m"], state["k"])
        return state["plan"].execute(state["f"])
    if kind == "train":
        feat, base, target = state["net"].features(state["k"], with_target=True)
        loss, grad = state["net"].loss_grad(feat, target)
        return {"feat": feat, "base": base, "target": target, "loss": loss, "grad": grad}
    return state["plan"].frame_approx(state["k"], state["f"])


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _pairs(n, m, dim=2):
    """Unordered pairs of samples in one another's weight box, at the raster's mean density."""
    if dim == 1:
        return m * min(m, 16) / 2
    return 0.5 * m * min(m, 256.0 * m / (0.707 * n * n))


def _image_work(n, G, m, dim, cs, weights, r=1, iters=0):
    b = m * (8 * dim + cs) + n ** dim * cs
    taps = 12 ** dim * m * 4.0
    fft = 5.0 * G ** dim * math.log2(G) * dim
    fl = taps + fft
    if weights in ("plain", "band"):
        fl += 15.0 * _pairs(n, m, dim)
    if weights == "band":
        fl += 2 * _pairs(n, m, dim) * (2 * r - 1) * 2.0 + m * ((2 * r - 1) ** 3 / 3.0 + 8.0 * r)
    if weights == "density":
        fl += iters * m * 12 ** dim * 8.0
    if weights == "learned":
        fl += m * 2.0 * NPARAM
    return b, fl


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = fl = 0.0
        for n, m, _ in _batch_items(case):
            x = _image_work(n, 2 * n, m, 2, 8, "plain")
            b, fl = b + x[0], fl + x[1]
        return {"bytes": b, "flops": fl}
    if kind == "train":
        m = case["m"]
        return {"bytes": m * (16 + 128 + 8 + 4) + 4.0 * NPARAM * 2,
                "flops": 15.0 * _pairs(case["n"], m) + 6.0 * NPARAM * m}
    if kind == "frame":
        m, modes = case["side"] ** 2, case["n"] ** 2
        lo, hi = min(m, modes), max(m, modes)
        return {"bytes": m * 32.0 + modes * 16.0, "flops": 2.0 * hi * lo * lo - 2.0 * lo ** 3 / 3.0}
    n, G, m, dim = case["n"], case["G"], case["m"], case["dim"]
    cs = 8 if case["dtype"] == "f32" else 16
    w = case["weights"] if kind == "image" else "none"
    b, fl = _image_work(n, G, m, dim, cs, w, case.get("r", 1), case.get("iters", 0))
    if kind != "image":
        b += m * 8.0   # the weights (ping); the forward transform reads none
    return {"bytes": b, "flops": fl}


# ----------------------------------------------------------------------------
# the same in 64 bits, from plain torch and numpy
# ----------------------------------------------------------------------------

W = 6
RADIUS = 8.0


def _beta(sigma):
    return math.pi * (sigma - 0.5) / (sigma * W)


class _Box:
    """Candidate pairs of samples within RADIUS of each other along both axes."""

    def __init__(self, k):
        k = k if k.shape[1] == 2 else torch.cat([torch.zeros_like(k), k], dim=1)
        lo = k.min(0).values
        self.row = torch.floor((k[:, 0] - lo[0]) / RADIUS)
        self.span = float((k[:, 1].max() - lo[1]).item()) + 4 * RADIUS
        self.x = k[:, 1] - lo[1]
        key, self.order = torch.sort(self.row * self.span + self.x)
        self.lo, self.cnt = [], []
        for dr in (-1, 0, 1):
            c = (self.row + dr) * self.span + self.x
            a = torch.searchsorted(key, c - (RADIUS + 1e-6))
            self.lo.append(a)
            self.cnt.append(torch.searchsorted(key, c + (RADIUS + 1e-6)) - a)
        self.total = self.cnt[0] + self.cnt[1] + self.cnt[2]

    def chunks(self, budget=PAIR_BUDGET):
        """(first, last) ranges of samples with at most `budget` candidates together."""
        ends = torch.cumsum(self.total, 0).cpu().numpy()
        a = 0
        while a < len(ends):
            base = ends[a - 1] if a else 0
            b = max(a + 1, int(np.searchsorted(ends, base + budget, side="right")))
            yield a, b
            a = b

    def pairs(self, a, b):
        """(i, j): every sample i of a..b-1 with each of its candidates j."""
        ii, jj = [], []
        for lo, cnt in zip(self.lo, self.cnt):
            c = cnt[a:b]
            i = torch.repeat_interleave(torch.arange(a, b, device=c.device), c)
            first = torch.cumsum(c, 0) - c
            at = torch.arange(i.numel(), device=c.device) - first[i - a] + lo[i]
            ii.append(i)
            jj.append(self.order[at])
        return torch.cat(ii), torch.cat(jj)


def _gram(k, i, j):
    """T_ij: product of sincs inside the box, else 0."""
    t = None
    for a in range(k.shape[1]):
        d = k[i, a] - k[j, a]
        s = torch.where(d.abs() <= RADIUS, torch.sinc(d), torch.zeros_like(d))
        t = s if t is None else t * s
    return t


def _weights(k):
    box = _Box(k)
    out = torch.zeros(k.shape[0], dtype=torch.float64, device=k.device)
    for a, b in box.chunks():
        i, j = box.pairs(a, b)
        out.index_add_(0, i, _gram(k, i, j) ** 2)
    return 1.0 / out


def _taps(k, G, sigma):
    """Per axis and tap, the grid index and the kernel value."""
    beta = _beta(sigma)
    u = sigma * k + G // 2
    f = torch.floor(u)
    g = f[:, :, None] + torch.arange(1 - W, W + 1, device=k.device, dtype=torch.float64)
    return torch.remainder(g, G).to(torch.int64), torch.exp(-beta * (g - u[:, :, None]) ** 2)


def _spread(k, c, G, sigma):
    d = k.shape[1]
    H = torch.zeros(G ** d, 2, dtype=torch.float64, device=k.device)
    step = 1 << 21
    for s in range(0, k.shape[0], step):
        g, e = _taps(k[s:s + step], G, sigma)
        v = torch.view_as_real(c[s:s + step].to(torch.complex128))
        for a in range(2 * W):
            if d == 1:
                H.index_add_(0, g[:, 0, a], v * e[:, 0, a, None])
                continue
            va = v * e[:, 0, a, None]
            for b in range(2 * W):
                H.index_add_(0, g[:, 0, a] * G + g[:, 1, b], va * e[:, 1, b, None])
    return torch.view_as_complex(H).reshape((G,) * d)


def _interpolate(k, H, G, sigma):
    d = k.shape[1]
    out = torch.zeros(k.shape[0], dtype=H.dtype, device=k.device)
    step = 1 << 21
    for s in range(0, k.shape[0], step):
        g, e = _taps(k[s:s + step], G, sigma)
        o = out[s:s + step]
        for a in range(2 * W):
            if d == 1:
                o += H[g[:, 0, a]] * e[:, 0, a]
                continue
            for b in range(2 * W):
                o += H.reshape(-1)[g[:, 0, a] * G + g[:, 1, b]] * (e[:, 0, a] * e[:, 1, b])
    return out


def _window(n, sigma):
    beta = _beta(sigma)
    x = (torch.arange(n, device=DEV, dtype=torch.float64) - n // 2) / n / sigma
    return math.sqrt(math.pi / beta) * torch.exp(-math.pi ** 2 * x * x / beta)


def _grid_to_image(H, n, G, sigma):
    d = H.dim()
    J = torch.fft.fftshift(torch.fft.ifftn(torch.fft.ifftshift(H), norm="forward"))
    lo = G // 2 - n // 2
    w = _window(n, sigma)
    return J[lo:lo + n] / w if d == 1 else J[lo:lo + n, lo:lo + n] / (w[:, None] * w[None, :])


def _image(case, k, c):
    sigma = case["G"] / case["n"]
    return _grid_to_image(_spread(k, c, case["G"], sigma), case["n"], case["G"], sigma)


def _band_values(k, f, r):
    """C f with C the (2r-1)-banded minimiser of ||T C - I||_F."""
    m, nb = k.shape[0], 2 * r - 1
    box = _Box(k)
    P = torch.zeros(m, nb, dtype=torch.float64, device=k.device)
    at = torch.arange(m, device=k.device)
    for a, b in box.chunks(PAIR_BUDGET // 4):
        i, j = box.pairs(a, b)
        t = _gram(k, i, j)
        for e in range(nb):
            o = i + e
            ok = o < m
            v = t * _gram(k, o.clamp(max=m - 1), j)
            P[:, e].index_add_(0, i, torch.where(ok, v, torch.zeros_like(v)))
    J = at[:, None] + torch.arange(1 - r, r, device=k.device)       # m x nb
    ok = (J >= 0) & (J < m)
    Jc = J.clamp(0, m - 1)
    lo, hi = torch.minimum(Jc[:, :, None], Jc[:, None, :]), torch.maximum(Jc[:, :, None], Jc[:, None, :])
    both = ok[:, :, None] & ok[:, None, :]
    A = torch.where(both, P[lo, (hi - lo).clamp(max=nb - 1)], torch.zeros((), dtype=torch.float64, device=k.device))
    A = A + torch.diag_embed((~ok).to(torch.float64))
    rhs = torch.where(ok, _gram(k, at[:, None].expand(m, nb), Jc), torch.zeros_like(A[:, :, 0]))
    col = np.linalg.solve(A.cpu().numpy(), rhs.cpu().numpy()[:, :, None])[:, :, 0]
    col = torch.where(ok, torch.from_numpy(col).to(k.device), torch.zeros_like(rhs))
    out = torch.zeros(m, 2, dtype=torch.float64, device=k.device)
    fr = torch.view_as_real(f.to(torch.complex128))
    for p in range(nb):
        out.index_add_(0, Jc[:, p], col[:, p, None] * fr)
    return torch.view_as_complex(out)


def _density_weights(case, k):
    sigma, G = case["G"] / case["n"], case["G"]
    w = torch.ones(k.shape[0], dtype=torch.float64, device=k.device)
    for _ in range(case["iters"]):
        w = w / _interpolate(k, _spread(k, w, G, sigma).real.contiguous(), G, sigma)
    return w * (math.pi / (sigma * _beta(sigma))) ** k.shape[1]


def _features(k):
    """32 offsets of the 16 nearest samples in the box (nearest first) and the estimate from them."""
    m = k.shape[0]
    box = _Box(k)
    feat = torch.full((m, 16, 2), RADIUS, dtype=torch.float64, device=k.device)
    for a, b in box.chunks():
        i, j = box.pairs(a, b)
        d = k[j] - k[i]
        q = d[:, 0].float() ** 2 + d[:, 1].float() ** 2
        q = torch.where((i != j) & (d.abs() <= RADIUS).all(1), q, torch.full_like(q, math.inf))
        s = torch.sort(j, stable=True).indices                # ties: the smaller index
        s = s[torch.sort(q[s], stable=True).indices]
        s = s[torch.sort(i[s], stable=True).indices]
        i, q, d = i[s], q[s], d[s]
        cnt = box.total[a:b]
        rank = torch.arange(i.numel(), device=k.device) - (torch.cumsum(cnt, 0) - cnt)[i - a]
        keep = (rank < 16) & torch.isfinite(q)
        feat[i[keep], rank[keep]] = d[keep]
    s = torch.where(feat.abs() < RADIUS, torch.sinc(feat), torch.zeros_like(feat)) ** 2
    return feat.reshape(m, 32), 1.0 / (1.0 + (s[:, :, 0] * s[:, :, 1]).sum(1))


def _network(x, p):
    a = torch.nn.functional.silu(x @ p[0] + p[1])
    a = torch.nn.functional.silu(a @ p[2] + p[3])
    return (a @ p[4] + p[5]).reshape(-1)


def _split(v):
    out, o = [], 0
    for s in ((32, 64), (64,), (64, 64), (64,), (64, 1), (1,)):
        c = int(np.prod(s))
        out.append(torch.from_numpy(np.asarray(v[o:o + c], dtype=np.float64).reshape(s)).to(DEV))
        o += c
    return out


def _learned_weights(k):
    with open(NET, "rb") as fh:
        blob = fh.read()                                        # header, parameters, two Adam moments
    p = _split(np.frombuffer(blob[-12 * NPARAM:-8 * NPARAM], dtype="<f4"))
    feat, base = _features(k)
    return base * torch.exp(_network(feat, p))


def _frame(case, seed):
    k, f = _frame_inputs(case, seed)
    n, sigma = case["n"], 2.0
    t, w = np.polynomial.legendre.leggauss(4 * n + 64)
    x = torch.from_numpy(0.5 * t).to(DEV)
    beta = _beta(sigma)
    v = torch.from_numpy(0.5 * w).to(DEV) / (math.sqrt(math.pi / beta) *
                                             torch.exp(-math.pi ** 2 * (x / sigma) ** 2 / beta))
    modes = torch.arange(n, device=DEV, dtype=torch.float64) - n // 2
    g = [(torch.cos(2 * math.pi * (k[:, a, None] - modes)[:, :, None] * x) * v).sum(2) for a in (0, 1)]
    Psi = (g[0][:, :, None] * g[1][:, None, :]).reshape(k.shape[0], n * n)
    B = np.linalg.lstsq(Psi.cpu().numpy(), torch.view_as_real(f).cpu().numpy(), rcond=None)[0]
    c = torch.view_as_complex(torch.from_numpy(np.ascontiguousarray(B)).to(DEV)).reshape(n, n)
    w = _window(n, sigma)
    img = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(c), norm="forward"))
    return img / (w[:, None] * w[None, :])


def _train(case, seed):
    k, params = _train_inputs(case, seed)
    feat, base = _features(k)
    target = torch.log(_weights(k) / base)
    p = [torch.from_numpy(params[n].astype(np.float64)).to(DEV).requires_grad_()
         for n in ("W1", "b1", "W2", "b2", "W3", "b3")]
    loss = torch.mean((_network(feat, p) - target) ** 2)
    grad = torch.cat([g.reshape(-1) for g in torch.autograd.grad(loss, p)])
    return {"feat": feat, "base": base, "target": target, "loss": float(loss.item()), "grad": grad}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for (n, _, _), k, f in zip(_batch_items(case), *_batch_inputs(case, seed)):
            out.append(_image(dict(n=n, G=2 * n), k, _weights(k) * f).reshape(-1))
        return torch.cat(out)
    if kind == "train":
        return _train(case, seed)
    if kind == "frame":
        return _frame(case, seed)
    n, G = case["n"], case["G"]
    if kind == "forward":
        k, img = _forward_inputs(case, seed)
        w = _window(n, G / n)
        J = torch.zeros(G, G, dtype=torch.complex128, device=DEV)
        lo = G // 2 - n // 2
        J[lo:lo + n, lo:lo + n] = img / (w[:, None] * w[None, :])
        H = torch.fft.fftshift(torch.fft.fft2(torch.fft.ifftshift(J)))
        return _interpolate(k, H, G, G / n)
    k, f = _image_inputs(case, seed)
    w = case["weights"]
    if w == "band":
        c = _band_values(k, f, case["r"])
    elif w == "none":
        c = f
    else:
        c = f * {"plain": _weights, "learned": _learned_weights, "density": lambda q: _density_weights(case, q)}[w](k)
    return _image(case, k, c)
