"""Workloads of the field-map estimator for timing, each through the public Python entry points.

A case names a volume (grid, coils, echo times, mask), the solver options and the call.  Inputs are
synthetic acquisitions made on the GPU from a seed: an ellipsoid phantom with smooth phase, a smooth field
of some hundred Hz with a local dipole, Gaussian coil maps on a ring, complex noise.  `exact` is the method
itself in plain torch and float64 (the iteration of Lin & Fessler, arXiv 2005.08661, Sec. III), written for
any device and independent of the kernels.
"""
import math

import numpy as np
import torch

from paper_2005_08661_amd import fmap

DEV = "cuda" if torch.cuda.is_available() else "cpu"

# six fat peaks at 3 T: offsets in Hz, amplitudes
FAT_HZ = [-3.80 * 127.732434, -3.40 * 127.732434, -2.70 * 127.732434, -2.00 * 127.732434, -0.50 * 127.732434,
          0.60 * 127.732434]
FAT_AMP = [0.08, 0.70, 0.12, 0.02, 0.03, 0.05]
WF_TE = "1.2,2.2,3.2,4.2,5.2,6.2"
BATCH16 = ("152x120x48 80x72x72 144x80x96 96x80x72 104x144x88 128x96x96 136x152x96 72x104x72 120x136x64 "
           "160x152x48 96x80x80 152x128x88 112x160x80 88x128x80 152x96x40 120x64x64")


def _case(name, call, shapes, coils, te, beta, mask, niter, precision, order, precond, model="fieldmap", reg=1,
          rtol=0.0):
    c = dict(call=call, shapes=shapes, coils=coils, te_ms=te, beta=beta, mask=mask, niter=niter,
             precision=precision, order=order, precond=precond, model=model, reg=reg, rtol=rtol)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one coil, every solver option at its default (FP64, natural-order IC(0));
        # what a first script or a per-slab loop runs, where launches and waits are all there is
        _case("small 32x32x16 f64 natural", "solve", "32x32x16", 1, "0,2,10", 0.125, "head", 50, "f64", "natural",
              "ic0"),
        # a thin many-coil phantom scan (74x74x10, 32 coils, echoes 0/1/2.3 ms): a column length that is no
        # multiple of 4, few voxels, much coil data for its size
        _case("phantom 74x74x10 mix redblack", "solve", "74x74x10", 32, "0,1,2.3", 0.125, "head", 50, "mix",
              "redblack", "ic0"),
        # the ordinary volume of the package's benchmark
        _case("head 128x128x64 mix redblack", "solve", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 100, "mix",
              "redblack", "ic0"),
        # odd sizes in full precision on a head-shaped mask, as after resampling to a 2 mm template grid
        _case("odd 91x109x91 f64 redblack", "solve", "91x109x91", 4, "0,2,5", 0.0625, "head", 40, "f64", "redblack",
              "ic0"),
        # a volume above the 256 MB last-level cache
        _case("large 256x256x128 mix redblack", "solve", "256x256x128", 2, "0,2.2,4.4", 0.0625, "full", 100, "mix",
              "redblack", "ic0"),
        # the default elimination order at the ordinary size, to a 1e-4 cost gap
        _case("head 128x128x64 mix natural", "solve", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 40, "mix",
              "natural", "ic0"),
        # the paper's own preconditioner, IC with a drop tolerance, to a 1e-3 cost gap
        _case("head 128x128x64 mix ict", "solve", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 10, "mix", "natural",
              "ict"),
        # block red-black order: natural order's iteration count at a fraction of its waits
        _case("head 128x128x64 mix blockrb", "solve", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 40, "mix",
              "blockrb", "ic0"),
        # water-fat imaging: six echoes, the swept and smoothed start of Sec. III-A
        _case("waterfat 192x192x64 mix", "solve", "192x192x64", 8, WF_TE, 0.0625, "full", 100, "mix", "redblack",
              "ic0", model="waterfat"),
        # a reconstruction queue: sixteen volumes of different sizes in one call
        _case("batch of 16 mix redblack", "batch", BATCH16, 4, "0,2,5", 0.0625, "full", 100, "mix", "redblack", "ic0"),
        # second-order differences with three-colour IC(0)
        _case("second order 128x128x64 mix", "solve", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 100, "mix",
              "color3", "ic0", reg=2),
        # a training step: the solve and its implicit gradient with respect to the images and beta
        _case("train step 128x128x64 mix", "train", "128x128x64", 8, "0,2.2,4.4", 0.0625, "full", 100, "mix",
              "redblack", "ic0", rtol=1e-6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of a listed kind: sizes over the kind's range, odd ones among them."""
    kind = rng.choice(["small", "redblack", "redblack", "f64", "large", "natural", "ict", "blockrb", "waterfat",
                       "batch", "second", "train"])
    beta = round(2.0 ** rng.uniform(-6, -2), 5)
    mask = rng.choice(["full", "head"])
    te = rng.choice(["0,2.2,4.4", "0,2,5", "0,1,2.3", "0,2.5", "0,1.5,3,5"])

    def grid(xy, z):
        return "%dx%dx%d" % (_log(rng, *xy), _log(rng, *xy), _log(rng, *z))

    if kind == "small":
        return _case(None, "solve", grid((12, 48), (8, 32)), rng.choice([1, 2, 4]), te, beta, mask, 50,
                     rng.choice(["f64", "mix"]), rng.choice(["natural", "redblack", "blockrb"]), "ic0")
    if kind == "redblack":
        return _case(None, "solve", grid((48, 150), (10, 64)), rng.choice([4, 8, 16]), te, beta, mask, 50, "mix",
                     "redblack", rng.choice(["ic0", "ic0", "ic0", "diag"]))
    if kind == "f64":
        return _case(None, "solve", grid((48, 128), (10, 90)), rng.choice([2, 4, 8]), te, beta, mask, 40, "f64",
                     "redblack", "ic0")
    if kind == "large":
        return _case(None, "solve", grid((160, 256), (80, 128)), 2, te, beta, mask, 60, "mix", "redblack", "ic0")
    if kind == "natural":
        return _case(None, "solve", grid((48, 128), (16, 64)), rng.choice([2, 8]), te, beta, mask, 20,
                     rng.choice(["f64", "mix"]), "natural", "ic0")
    if kind == "ict":
        return _case(None, "solve", grid((40, 120), (16, 64)), rng.choice([2, 8]), te, beta, mask, 8,
                     rng.choice(["f64", "mix"]), "natural", "ict")
    if kind == "blockrb":
        return _case(None, "solve", grid((48, 128), (16, 64)), rng.choice([2, 8]), te, beta, mask, 40,
                     rng.choice(["f64", "mix"]), "blockrb", "ic0")
    if kind == "waterfat":
        return _case(None, "solve", grid((64, 180), (16, 64)), rng.choice([4, 8]), WF_TE, beta, mask, 50,
                     rng.choice(["f64", "mix"]), "redblack", "ic0", model="waterfat")
    if kind == "batch":
        n = rng.randint(3, 12)
        shapes = " ".join("%dx%dx%d" % (rng.randrange(64, 161, 8), rng.randrange(64, 161, 8), rng.randrange(32, 97, 8))
                          for _ in range(n))
        return _case(None, "batch", shapes, 4, te, beta, mask, 60, "mix", "redblack", "ic0")
    if kind == "second":
        return _case(None, "solve", grid((48, 128), (16, 64)), rng.choice([2, 8]), te, beta, mask, 50, "mix", "color3",
                     "ic0", reg=2)
    return _case(None, "train", grid((48, 128), (16, 64)), rng.choice([2, 8]), te, beta, mask, 80, "mix", "redblack",
                 "ic0", rtol=1e-6)


# --- inputs --------------------------------------------------------------------------------------

def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split()]


def _te(case):
    return [1e-3 * float(v) for v in case["te_ms"].split(",")]


def _smooth(gen, shape, k, span):
    """Sum of k random anisotropic Gaussians, scaled to max |.| = span."""
    r = torch.rand((k, 7), generator=gen, device=DEV)
    out = torch.zeros(shape, device=DEV)
    for i in range(k):
        e = [torch.exp(-0.5 * ((torch.arange(n, device=DEV) - (0.2 + 0.6 * r[i, a]) * n)
                               / ((0.1 + 0.2 * r[i, 3 + a]) * n)) ** 2) for a, n in enumerate(shape)]
        out += (2 * r[i, 6] - 1) * e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
    return out * (span / out.abs().max().clamp_min(1e-12))


def _acquire(case, shape, seed):
    """y complex64 [ncoil, L, X, Y, Z], sens (None for one coil), mask uint8, the true field."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    wf = case["model"] == "waterfat"
    g = torch.meshgrid(*[torch.arange(n, device=DEV, dtype=torch.float32) for n in shape], indexing="ij")
    ctr = [(n - 1) / 2 for n in shape]
    r2 = sum(((g[a] - ctr[a]) / max(0.4 * n, 0.5)) ** 2 for a, n in enumerate(shape))
    mag = torch.where(r2 <= 1, 1.0, 0.05)
    f = _smooth(gen, shape, 8, 300.0 if wf else 120.0 if min(shape) < 24 else 250.0)
    if not wf and min(shape) >= 24:  # a susceptibility-like dipole of +-400 Hz
        c = torch.rand(3, generator=gen, device=DEV)
        d = [g[a] - (0.35 + 0.3 * c[a]) * n for a, n in enumerate(shape)]
        q = (d[0] ** 2 + d[1] ** 2 + d[2] ** 2).clamp_min(16.0)
        f = f + (400.0 * 32.0 * (3 * d[2] ** 2 - q) / q ** 2.5).clamp(-400, 400)
    phase = torch.polar(torch.ones(shape, device=DEV), _smooth(gen, shape, 3, math.pi))
    te = _te(case)
    if wf:
        ff = 0.25 + 0.25 * _smooth(gen, shape, 4, 1.0)
        cl = [sum(a * complex(math.cos(2 * math.pi * h * t), math.sin(2 * math.pi * h * t))
                  for a, h in zip(FAT_AMP, FAT_HZ)) for t in te]
        img = [mag * phase * ((1 - ff) + ff * c) for c in cl]
    else:
        img = [mag * phase] * len(te)
    nc = case["coils"]
    sens = None
    if nc > 1:
        R, u = max(shape[:2]), torch.rand((nc, 4), generator=gen, device=DEV)
        sens = torch.empty((nc,) + shape, dtype=torch.complex64, device=DEV)
        for k in range(nc):
            th = 2 * math.pi * k / nc
            p = (ctr[0] + 0.6 * R * math.cos(th), ctr[1] + 0.6 * R * math.sin(th),
                 ctr[2] + (0.25 if k % 2 == 0 else -0.25) * shape[2])
            m = torch.exp(-2.0 * sum((g[a] - p[a]) ** 2 for a in range(3)) / R ** 2)
            sens[k] = torch.polar(m, 2 * math.pi * u[k, 0] + sum(2 * (u[k, 1 + a] - 0.5) * g[a] / n
                                                                 for a, n in enumerate(shape)))
        sens /= (sens.abs() ** 2).sum(0).sqrt()
    y = torch.empty((nc, len(te)) + shape, dtype=torch.complex64, device=DEV)
    sigma = 10 ** (-25.0 / 20) / math.sqrt(nc)
    for l, t in enumerate(te):
        im = img[l] * torch.polar(torch.ones(shape, device=DEV), 2 * math.pi * t * f)
        for k in range(nc):
            y[k, l] = im if sens is None else sens[k] * im
            y[k, l] += sigma * torch.randn(shape, dtype=torch.complex64, generator=gen, device=DEV)
    if case["mask"] == "full":
        mask = torch.ones(shape, dtype=torch.uint8, device=DEV)
    else:  # the phantom's hull, two voxels wider on each side
        mask = (sum(((g[a] - ctr[a]) / (0.4 * n + 2)) ** 2 for a, n in enumerate(shape)) <= 1).to(torch.uint8)
    return y, sens, mask, f.double() * mask


def _betas(case):
    """Volumes of a batch differ in beta."""
    n = len(_shapes(case))
    return [case["beta"] * 2.0 ** (0 if n == 1 else (v % 5) - 2) for v in range(n)]


def _params(case, shape, beta):
    wf = case["model"] == "waterfat"
    return fmap.make_params(
        shape, case["coils"], _te(case), beta, case["niter"], model=fmap.WATERFAT if wf else fmap.FIELDMAP,
        fat_hz=FAT_HZ if wf else None, fat_amp=FAT_AMP if wf else None,
        precision=dict(f64=fmap.F64, mix=fmap.MIX)[case["precision"]],
        ordering=dict(natural=fmap.NATURAL, redblack=fmap.REDBLACK, color3=fmap.COLOR3,
                      blockrb=fmap.BLOCKRB)[case["order"]],
        precond=dict(ic0=fmap.IC0, diag=fmap.DIAG, ict=fmap.ICT)[case["precond"]], reg_order=case["reg"])


def prepare(case, seed):
    shapes, betas = _shapes(case), _betas(case)
    vols = [_acquire(case, s, seed * 1000 + v) for v, s in enumerate(shapes)]
    prms = [_params(case, s, b) for s, b in zip(shapes, betas)]
    st = dict(case=case, y=[v[0] for v in vols], s=[v[1] for v in vols], m=[v[2] for v in vols])
    if case["call"] == "batch":
        st["handle"] = fmap.Batch(prms)
    else:
        st["handle"] = fmap.Plan(prms[0])
    if case["call"] == "train":
        st["y"][0].requires_grad_(True)
        st["beta"] = torch.tensor(case["beta"], device=DEV, requires_grad=True)
        st["target"] = vols[0][3]
    return st


def run(state):
    c, h = state["case"], state["handle"]
    if c["call"] == "batch":
        return h.solve(state["y"], state["s"], state["m"])
    if c["call"] == "train":
        y, beta = state["y"][0], state["beta"]
        f = fmap.fieldmap_solve(y, state["s"][0], state["m"][0], beta, h, rtol=c["rtol"])
        dy, db = torch.autograd.grad(((f - state["target"]) ** 2).sum(), (y, beta))
        return dict(f=f.detach(), dy=dy, dbeta=db)
    return h.solve(state["y"][0], state["s"][0], state["m"][0])


def work(case):
    """Images, coil maps and mask once, the map once, and per iteration the sweeps that the method's data
    dependences force: a forward one (echo data, f and z in; f, g, D, an FP64 pivot and a vector out), a
    backward one, the direction, and two line-search passes over echo data, f and z."""
    te = _te(case)
    L, nc = len(te), case["coils"]
    pairs = L * (L - 1) // 2
    t = 4 if case["precision"] == "mix" else 8
    frac = 1.0 if case["mask"] == "full" else 4 / 3 * math.pi * 0.42 ** 3
    vox = sum(a * b * c for a, b, c in _shapes(case))
    n = vox * frac
    io = vox * (8.0 * nc * (L + (nc > 1)) + 1 + 8)
    fwd = 2 * L * t + 2 * t + 4 * t + 8
    it = fwd + (5 * t + 8) + 5 * t + 2 * (2 * L * t + 2 * t)
    flops = n * case["niter"] * (3 * 28 * pairs + 60)
    nbytes = io + n * case["niter"] * it
    if case["model"] == "waterfat":
        flops += n * 100 * pairs * 45
    if case["call"] == "train":
        nbytes += vox * 8.0 * nc * L
    return dict(bytes=nbytes, flops=flops)


# --- the method in float64 torch ------------------------------------------------------------------

class _Volume:
    """In-mask voxels as flat vectors of m values; index m is a slot that reads 0."""

    def __init__(self, mask):
        self.mask = mask.bool()
        self.shape = tuple(mask.shape)
        self.xyz = torch.nonzero(self.mask).T.contiguous()
        self.m = self.xyz.shape[1]
        self.vol = torch.full(self.shape, self.m, dtype=torch.int64, device=mask.device)
        self.vol[self.mask] = torch.arange(self.m, device=mask.device)
        e = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
        self.nb = {(a, s): self.at(tuple(s * v for v in e[a])) for a in range(3) for s in (-1, 1)}
        self.deg = sum((v < self.m).double() for v in self.nb.values())

    def at(self, off):
        """Index of the voxel at an offset, m where there is none."""
        q = [self.xyz[a] + off[a] for a in range(3)]
        ok = torch.ones_like(q[0], dtype=torch.bool)
        for a in range(3):
            ok &= (q[a] >= 0) & (q[a] < self.shape[a])
            q[a] = q[a].clamp(0, self.shape[a] - 1)
        return torch.where(ok, self.vol[q[0], q[1], q[2]], self.m)

    @staticmethod
    def pad(v):
        return torch.cat([v, v.new_zeros(1)])

    def levels(self, key):
        """Index lists of equal key in ascending order."""
        o = torch.argsort(key, stable=True)
        _, n = torch.unique_consecutive(key[o], return_counts=True)
        return list(torch.split(o, n.tolist()))


class _Reg1:
    def __init__(self, V):
        self.V = V
        self.diag = V.deg

    def ctc(self, f):
        p = self.V.pad(f)
        out = self.V.deg * f
        for i in self.V.nb.values():
            out -= p[i]
        return out

    def norm2(self, z):
        p, V = self.V.pad(z), self.V
        return sum((((p[V.nb[a, 1]] - z) * (V.nb[a, 1] < V.m)) ** 2).sum() for a in range(3))


class _Reg2:
    def __init__(self, V):
        self.V = V
        self.r = [((V.nb[a, -1] < V.m) & (V.nb[a, 1] < V.m)).double() for a in range(3)]
        self.diag = sum(4 * self.r[a] + V.pad(self.r[a])[V.nb[a, -1]] + V.pad(self.r[a])[V.nb[a, 1]] for a in range(3))

    def rows(self, f):
        p, V = self.V.pad(f), self.V
        return [self.r[a] * (p[V.nb[a, -1]] - 2 * f + p[V.nb[a, 1]]) for a in range(3)]

    def ctc(self, f):
        V = self.V
        return sum(-2 * d + V.pad(d)[V.nb[a, -1]] + V.pad(d)[V.nb[a, 1]] for a, d in enumerate(self.rows(f)))

    def norm2(self, z):
        return sum((d * d).sum() for d in self.rows(z))


def _ic0(V, order, beta):
    """p = P^{-1} g with IC(0) of diag(D) + beta C^T C on the 7-point stencil."""
    x, y, z = V.xyz
    if order == "natural":
        key = x + y + z
    elif order == "redblack":
        key = (x + y + z) % 2
    else:  # 8x8 column tiles in a checkerboard, natural order inside one
        key = ((x // 8 + y // 8) % 2) * (1 << 20) + x % 8 + y % 8 + z
    nb = torch.stack(list(V.nb.values()))
    kp = torch.cat([key, key.new_full((1,), 1 << 40)])[nb]
    early = torch.where((kp < key) & (nb < V.m), nb, V.m)
    late = torch.where((kp > key) & (nb < V.m), nb, V.m)
    lev = [(i, early[:, i].contiguous(), late[:, i].contiguous()) for i in V.levels(key)]

    def apply(D, g):
        h = D + beta * V.deg
        ip = h.new_zeros(V.m + 1)
        u = h.new_zeros(V.m + 1)
        p = h.new_zeros(V.m + 1)
        for i, e, _ in lev:
            q = 1.0 / (h[i] - beta * beta * ip[e].sum(0))
            ip[i] = q
            u[i] = (g[i] + beta * u[e].sum(0)) * q
        for i, _, l in reversed(lev):
            p[i] = u[i] + beta * ip[i] * p[l].sum(0)
        return p[:-1]

    return apply


def _ic0_second(V, R, beta):
    """The same on the 13-point stencil, colours (x + y + z) mod 3 in turn."""
    col = V.xyz.sum(0) % 3
    is_c = [(col == c) for c in range(3)]
    unit = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
    at = {(a, o): V.at(tuple(o * v for v in unit[a])) for a in range(3) for o in (-2, -1, 1, 2)}
    rp = [V.pad(r) for r in R.r]
    H = {}
    for a in range(3):
        for s in (-1, 1):
            H[a, s] = -2 * beta * (R.r[a] + rp[a][at[a, s]]) * (at[a, s] < V.m)
            H[a, 2 * s] = beta * rp[a][at[a, s]] * (at[a, 2 * s] < V.m)

    def apply(D, g):
        d = torch.cat([D + beta * R.diag, D.new_ones(1)])
        Lp = {k: D.new_zeros(V.m + 1) for k in at}

        def put(k, val, c):
            Lp[k][:-1] = torch.where(is_c[c], val, Lp[k][:-1])

        for a in range(3):
            for o in (-1, 2):
                put((a, o), H[a, o] / d[at[a, o]], 1)
        d1 = d[:-1] - sum(Lp[a, o][:-1] ** 2 * d[at[a, o]] for a in range(3) for o in (-1, 2))
        d[:-1] = torch.where(is_c[1], d1, d[:-1])
        for a in range(3):
            for o in (1, -2):
                put((a, o), H[a, o] / d[at[a, o]], 2)
        for a in range(3):
            k, m, q = at[a, -1], at[a, -2], at[a, 1]
            low = (H[a, -1] - Lp[a, -2][:-1] * Lp[a, -1][k] * d[m] - Lp[a, 1][:-1] * Lp[a, 2][k] * d[q]) / d[k]
            k = at[a, 2]
            high = (H[a, 2] - Lp[a, 1][:-1] * Lp[a, -1][k] * d[q]) / d[k]
            put((a, -1), low, 2)
            put((a, 2), high, 2)
        d2 = d[:-1] - sum(Lp[k][:-1] ** 2 * d[at[k]] for k in at)
        d[:-1] = torch.where(is_c[2], d2, d[:-1])
        u = V.pad(g)
        for c in (1, 2):
            v = g - sum(Lp[k][:-1] * u[at[k]] for k in at)
            u[:-1] = torch.where(is_c[c], v, u[:-1])
        w = u[:-1] / d[:-1]
        p = V.pad(w)
        for c in (1, 0):
            v = w - sum(Lp[a, -o][at[a, o]] * p[at[a, o]] for a, o in at)
            p[:-1] = torch.where(is_c[c], v, p[:-1])
        return p[:-1]

    return apply


def _ict(V, beta, factor=1e-3):
    """IC with a drop tolerance on the level-1 fill pattern (natural order)."""
    off = [(1, 0, 0), (1, 0, -1), (1, -1, 0), (0, 1, 0), (0, 1, -1), (0, 0, 1)]
    x, y, z = V.xyz
    lower = torch.stack([V.at(tuple(-v for v in o)) for o in off])
    upper = torch.stack([V.at(o) for o in off])
    lev = [(i, lower[:, i].contiguous(), upper[:, i].contiguous()) for i in V.levels(3 * x + 2 * y + z)]
    pair = {(u, v): off.index(d) for u in range(6) for v in range(u)
            if (d := tuple(p - q for p, q in zip(off[v], off[u]))) in off}
    stencil = [sum(o) == 1 and min(o) >= 0 for o in off]
    after = sum((V.nb[a, 1] < V.m).double() for a in range(3))

    def apply(D, g):
        h = D + beta * V.deg
        tol = factor * max(float(h.abs().max()), beta if bool((V.deg > 0).any()) else 0.0)
        cn = V.pad((h.abs() + beta * after) * tol)
        lo, ld = D.new_zeros(6, V.m + 1), D.new_ones(V.m + 1)
        yv, p = D.new_zeros(V.m + 1), D.new_zeros(V.m + 1)
        for i, k, _ in lev:
            lkk, ck = ld[k], cn[k]
            row = []
            for u in range(6):
                s = torch.full_like(h[i], -beta if stencil[u] else 0.0)
                for v in range(u):
                    if (u, v) in pair:
                        s = s - row[v] * lo[pair[u, v], k[u]]
                s = s / lkk[u]
                row.append(torch.where((s.abs() < ck[u]) | (k[u] == V.m), 0.0, s))
            r = torch.stack(row)
            ljj = (h[i] - (r * r).sum(0)).sqrt()
            lo[:, i] = r
            ld[i] = ljj
            yv[i] = (g[i] - (r * yv[k]).sum(0)) / ljj
        for i, _, k in reversed(lev):
            s = yv[i] - sum(lo[u][k[u]] * p[k[u]] for u in range(6))
            p[i] = s / ld[i]
        return p[:-1]

    return apply


class _Data:
    """The coil-combined echo-pair data term of one volume."""

    def __init__(self, case, V, y, sens):
        self.te = te = _te(case)
        L = len(te)
        y = y.detach()[:, :, V.mask].to(torch.complex128)
        self.s = None if sens is None else sens[:, V.mask].to(torch.complex128)
        if sens is None:
            self.ss = torch.ones(V.m, dtype=torch.float64, device=y.device)
            self.zh = y[0]
        else:
            self.ss = (self.s.abs() ** 2).sum(0)
            self.zh = (self.s.conj()[:, None] * y).sum(0) / self.ss.sqrt()
        if case["model"] == "waterfat":
            c = [sum(a * np.exp(2j * math.pi * h * t) for a, h in zip(FAT_AMP, FAT_HZ)) for t in te]
            A = np.stack([np.ones(L), np.array(c)], 1)
        else:
            A = np.ones((L, 1), complex)
        self.G = A @ np.linalg.pinv(A)
        self.pairs = [(m, n, 2 * abs(self.G[m, n]), float(np.angle(self.G[m, n])) / (2 * math.pi), te[m] - te[n])
                      for m in range(L) for n in range(m + 1, L)]
        self.rho, self.tau = self.zh.abs(), torch.angle(self.zh) / (2 * math.pi)
        self.absy = None
        if case["model"] == "waterfat":
            sa = 1.0 if self.s is None else self.s.abs()[:, None]
            self.absy = (sa * y.abs()).sum(0)

    def turns(self, f):
        for m, n, w, ang, dt in self.pairs:
            xi = ang + self.tau[n] - self.tau[m] + f * dt
            yield w * self.rho[m] * self.rho[n], xi - torch.round(xi), 2 * math.pi * dt

    def cost(self, f):
        return sum(w * (1 - torch.cos(2 * math.pi * h)) for w, h, _ in self.turns(f))

    def grad_curv(self, f):
        d = c = 0.0
        for w, h, k in self.turns(f):
            d = d + w * k * torch.sin(2 * math.pi * h)
            c = c + w * k * k * torch.sinc(2 * h)
        return d, c

    def hess(self, f):
        return sum(w * k * k * torch.cos(2 * math.pi * h) for w, h, k in self.turns(f))


def _start(case, d, R, beta):
    if case["model"] != "waterfat":
        return torch.angle(d.zh[0].conj() * d.zh[1]) / (2 * math.pi * (d.te[1] - d.te[0]))
    half = abs(FAT_HZ[int(np.argmax(FAT_AMP))]) / 2
    best = torch.full_like(d.rho[0], math.inf)
    ft = torch.zeros_like(best)
    for q in range(100):
        fs = -half + 2.0 * half * q / 99
        c = d.cost(torch.full_like(best, fs))
        ft = torch.where(c < best, fs, ft)
        best = torch.minimum(c, best)
    G = torch.from_numpy(abs(d.G)).to(best.device)
    rho = ((G @ d.absy) * d.absy).sum(0) / d.ss
    op = lambda v: 2 * rho * v + beta * R.ctc(v)  # noqa: E731
    f, r = ft.clone(), 2 * rho * ft - op(ft)
    p, rs = r.clone(), (r * r).sum()
    for _ in range(10):
        ap = op(p)
        a = rs / (p * ap).sum()
        f, r = f + a * p, r - a * ap
        rn = (r * r).sum()
        p, rs = r + (rn / rs) * p, rn
    return f


def _minimise(case, y, sens, mask, beta):
    V = _Volume(mask)
    d = _Data(case, V, y, sens)
    R = _Reg2(V) if case["reg"] == 2 else _Reg1(V)
    if case["precond"] == "ict":
        pre = _ict(V, beta)
    elif case["precond"] == "diag":
        pre = lambda D, g: g / (D + beta * R.diag)  # noqa: E731
    elif case["reg"] == 2:
        pre = _ic0_second(V, R, beta)
    else:
        pre = _ic0(V, case["order"], beta)
    f = _start(case, d, R, beta)
    z = gprev = torch.zeros_like(f)
    gtp_prev = 0.0
    for it in range(case["niter"]):
        dphi, D = d.grad_curv(f)
        g = dphi + beta * R.ctc(f)
        p = pre(D, g)
        gtp = (g * p).sum()
        mu = (gtp - (gprev * p).sum()) / gtp_prev if it else torch.zeros_like(gtp)
        ztg = -gtp + mu * (z * g).sum()
        if bool(ztg >= 0):
            mu, ztg = torch.zeros_like(gtp), -gtp
        z = -p + mu * z
        A, B = (z * R.ctc(f)).sum(), R.norm2(z)
        alpha = -ztg / ((z * z * D).sum() + beta * B)
        for _ in range(2):
            s1, s2 = d.grad_curv(f + alpha * z)
            alpha = alpha - ((z * s1).sum() + beta * A + alpha * beta * B) / ((z * z * s2).sum() + beta * B)
        f = f + alpha * z
        gprev, gtp_prev = g, gtp
    return V, d, R, f


def _out(V, f):
    v = torch.zeros(V.shape, dtype=f.dtype, device=f.device)
    v[V.mask] = f
    return v


def _gradient(V, d, R, f, dldf, beta):
    """dL/dy and dL/dbeta at the minimiser: H v = dL/df with the exact Hessian, by CG."""
    h = d.hess(f)
    diag = d.grad_curv(f)[1] + beta * R.diag
    op = lambda v: h * v + beta * R.ctc(v)  # noqa: E731
    v, r = torch.zeros_like(f), dldf.clone()
    z = r / diag
    p, rz, stop = z.clone(), (r * z).sum(), 1e-12 * float(dldf.norm())
    for k in range(20000):
        ap = op(p)
        a = rz / (p * ap).sum()
        v, r = v + a * p, r - a * ap
        if k % 20 == 0 and float(r.norm()) <= stop:
            break
        z = r / diag
        rn = (r * z).sum()
        p, rz = z + (rn / rz) * p, rn
    zh = d.zh.detach().clone().requires_grad_(True)
    g = 0.0
    for m, n, w, ang, dt in d.pairs:  # |Gamma| terms: Im(Gamma conj(z_m) z_n e^{i 2 pi f dt})
        e = torch.polar(torch.full_like(f, w * 2 * math.pi * dt), 2 * math.pi * (ang + f * dt))
        g = g + (e * zh[m].conj() * zh[n]).imag
    dz, = torch.autograd.grad(g, zh, -v)
    s = torch.ones((1, V.m), dtype=torch.complex128, device=f.device) if d.s is None else d.s
    dy = torch.zeros((s.shape[0], dz.shape[0]) + V.shape, dtype=torch.complex128, device=f.device)
    for c in range(s.shape[0]):
        dy[c][:, V.mask] = dz * (s[c] / d.ss.sqrt())
    return dy, -(v * R.ctc(f)).sum()


def exact(case, seed):
    outs = []
    for k, (shape, beta) in enumerate(zip(_shapes(case), _betas(case))):
        y, s, m, target = _acquire(case, shape, seed * 1000 + k)
        if case["call"] == "train":
            beta = float(torch.tensor(beta))
        V, d, R, f = _minimise(case, y, s, m, beta)
        if case["call"] == "train":
            dy, db = _gradient(V, d, R, f, 2 * (f - target[V.mask]), beta)
            return dict(f=_out(V, f), dy=dy, dbeta=db)
        outs.append(_out(V, f))
    return outs if case["call"] == "batch" else outs[0]
