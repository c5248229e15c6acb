"""Timing cases of the wavelet Sobolev-prior operators, over the range that they are used in.

A case is a dict: `kind` names the call (below), the other entries are its arguments (`n0`, `n1`, `n2`:
the sides of the grid, as many as it has).  Kinds:

  cov      matern_cov_apply of a batch of images or volumes, as a reconstruction loop calls it
  sample   matern_sample and its backward: a MAP estimate in the sampler's white-noise coordinates
  embed    es_adjoint and its backward (es_apply): a data term on E_s^* x
  norm     the squared H^s norm of a batch, the penalty that a solver monitors
  sym      the non-periodic operator and its backward (its transpose), any side lengths
  pcg      Tikhonov / MAP solve by preconditioned conjugate gradients, a fixed number of iterations
  gmres    the same in the paper's form by GMRES, 15 iterations as in the paper
  ragged   matern_cov_apply of instances of different sizes through a plan that the program keeps

The grids are those of the repository's workloads and tests: 128^2 (small image), 512^2 (the paper's
reconstruction grid), 1024^2 batches, 64^3 to 256^3 volumes, and sides that are no powers of two.  Images
are random discs plus noise, sampler inputs and incoming gradients are white noise, masks Bernoulli(0.3).

The Fourier form is left out: its time is that of the FFT library's transforms.
"""
import itertools
import math

import numpy as np
import torch

import paper_2507_02401_amd as es
from paper_2507_02401_amd import solver

MASK_DENSITY = 0.3
ALPHA = 0.05  # regularisation weight of the solver cases
PCG_ITERS, GMRES_ITERS = 12, 15


def listed():
    return [
        # one small image: latency and launches count
        dict(name="cov_one_128", kind="cov", batch=1, n0=128, n1=128, order=4, levels=5, s=1.0),
        # the benchmark's batch: the largest ordinary call
        dict(name="cov_64x1024", kind="cov", batch=64, n0=1024, n1=1024, order=8, levels=7, s=1.5),
        # sides that are no powers of two, levels whose rows are not multiples of four
        dict(name="cov_7x360x600", kind="cov", batch=7, n0=360, n1=600, order=3, levels=3, s=0.5),
        # a few volumes with a long filter
        dict(name="cov_4x128cube", kind="cov", batch=4, n0=128, n1=128, n2=128, order=8, levels=4, s=1.0),
        # MAP gradient through the sampler, the paper's grid, a large batch
        dict(name="sample_256x512", kind="sample", batch=256, n0=512, n1=512, order=6, levels=6, s=1.5),
        # one large volume, full filter bank in both directions
        dict(name="embed_256cube", kind="embed", batch=1, n0=256, n1=256, n2=256, order=4, levels=5, s=2.0),
        # the penalty's value for every image of a batch
        dict(name="norm_64x1024", kind="norm", batch=64, n0=1024, n1=1024, order=8, levels=7, s=1.5),
        # non-periodic operator, forward and backward, on images and on volumes of odd level sizes
        dict(name="sym_64x1024", kind="sym", batch=64, n0=1024, n1=1024, order=8, levels=7, s=1.5),
        dict(name="sym_2x96x112x160", kind="sym", batch=2, n0=96, n1=112, n2=160, order=8, levels=3, s=1.5),
        # one reconstruction as in the paper: 512^2, 15 GMRES iterations
        dict(name="gmres_one_512", kind="gmres", batch=1, n0=512, n1=512, order=6, levels=6, s=1.5),
        # a batch of reconstructions by conjugate gradients
        dict(name="pcg_16x512", kind="pcg", batch=16, n0=512, n1=512, order=6, levels=6, s=1.0),
        # many instances of different sizes, dimensions, filters and depths in one plan
        dict(name="ragged_48", kind="ragged", count=48, pick=1),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["cov", "cov", "sample", "embed", "norm", "sym", "pcg", "gmres", "ragged"])
    if kind == "ragged":
        return dict(kind=kind, count=rng.randint(4, 48), pick=rng.randint(2, 10 ** 6))
    order, s = rng.randint(1, 8), rng.choice([0.5, 1.0, 1.5, 2.0])
    if kind == "pcg":
        s = min(s, 1.0)  # above it the finest weights leave a solution of few exact digits in FP32
    ndim = rng.choice([2, 2, 3])
    if kind in ("pcg", "gmres"):
        ndim, largest = 2, 1 << (22 if kind == "pcg" else 21)
    else:
        largest = 1 << 26 if ndim == 2 else 1 << 24
    lo, hi = (64, 1024) if ndim == 2 else (32, 256)
    sides = [_log_uniform(rng, lo, hi) for _ in range(ndim)]
    levels = max(2, int(math.log2(min(sides))) - rng.choice([3, 3, 4]))
    if kind == "sym":
        sides = [int(v) for v in sides]  # any side length
    elif rng.random() < 0.4:
        sides = [2 ** round(math.log2(v)) for v in sides]  # as most grids are chosen
        levels = min(levels, int(math.log2(min(sides))))
    else:
        sides = [max(1, round(v / 2 ** levels)) * 2 ** levels for v in sides]
    most = max(1, largest // math.prod(sides))
    batch = max(1, int(_log_uniform(rng, 1, most)))
    case = dict(kind=kind, batch=batch, order=order, levels=levels, s=s)
    case.update({"n%d" % k: v for k, v in enumerate(sides)})
    return case


# ---- inputs --------------------------------------------------------------------------------------------

RAGGED_2D = (128, 192, 256, 360, 512, 640, 1024, 2048)
RAGGED_3D = (64, 96, 128)


def _ragged_descs(case):
    """(shape, order, levels, s) of every instance: mostly images of mixed sides, some cubes."""
    gen = np.random.default_rng(np.random.SeedSequence([7, int(case["pick"])]))
    out = []
    for _ in range(case["count"]):
        if gen.integers(10) == 0:
            shape = (int(gen.choice(RAGGED_3D)),) * 3
        else:
            shape = (int(gen.choice(RAGGED_2D)), int(gen.choice(RAGGED_2D)))
        order, s = int(gen.choice((2, 4, 8))), float(gen.choice((0.5, 1.0, 2.0)))
        levels = int(math.log2(min(shape))) - 3
        while any(v % 2 ** levels for v in shape):
            levels -= 1
        out.append((shape, order, levels, s))
    return out


def _grid(case):
    return tuple(case["n%d" % k] for k in range(3) if "n%d" % k in case)


def _phantom(batch, grid, gen, device, noise=0.05):
    """Random discs (balls in 3-D) of amplitude U[0.5, 1] plus white noise, per instance."""
    x = noise * torch.randn((batch,) + grid, generator=gen, device=device)
    nd = len(grid)
    for _ in range(20):
        radius = min(grid) * (0.02 + 0.1 * torch.rand(batch, generator=gen, device=device))
        amp = 0.5 + 0.5 * torch.rand(batch, generator=gen, device=device)
        d2 = 0.0
        for k, n in enumerate(grid):
            c = n * torch.rand(batch, generator=gen, device=device)
            axis = (torch.arange(n, device=device)[None, :] - c[:, None]) ** 2
            d2 = d2 + axis.reshape((batch,) + tuple(n if j == k else 1 for j in range(nd)))
        one = (batch,) + (1,) * nd
        x += amp.reshape(one) * (d2 <= (radius ** 2).reshape(one))
    return x


def _inputs(case, seed, device):
    gen = torch.Generator(device).manual_seed(int(seed))
    kind = case["kind"]

    def noise(*shape):
        return torch.randn(shape, generator=gen, device=device)

    if kind == "ragged":
        return [noise(*d[0]) for d in _ragged_descs(case)]
    grid = _grid(case)
    shape = (case["batch"],) + grid
    if kind == "sample":
        return [noise(*shape), noise(*shape)]
    x = _phantom(case["batch"], grid, gen, device)
    if kind in ("embed", "sym"):
        return [x, noise(*shape)]
    if kind in ("pcg", "gmres"):
        mask = (torch.rand(shape, generator=gen, device=device) < MASK_DENSITY).float()
        return [mask * x, mask]
    return [x]


def prepare(case, seed):
    xs = _inputs(case, seed, "cuda")
    kind = case["kind"]
    if kind == "ragged":
        return dict(kind=kind, xs=xs, plan=es.RaggedPlan(_ragged_descs(case), es.OP_COV))
    if kind in ("sample", "embed", "sym"):
        xs[0].requires_grad_(True)
    return dict(kind=kind, xs=xs, args=(len(_grid(case)), case["order"], case["levels"], case["s"]))


def run(state):
    kind, xs = state["kind"], state["xs"]
    if kind == "ragged":
        return state["plan"](xs)
    args = state["args"]
    if kind == "cov":
        return es.matern_cov_apply(xs[0], *args)
    if kind == "norm":
        return es.hs_norm_sq(xs[0], *args)
    if kind == "pcg":
        x, info = solver.tikhonov_pcg(xs[0], xs[1], *args, ALPHA, iters=PCG_ITERS, rtol=0.0)
        return x, info["iterations"]
    if kind == "gmres":
        x, info = solver.tikhonov_gmres(xs[0], xs[1], *args, ALPHA, iters=GMRES_ITERS, restart=GMRES_ITERS, rtol=0.0)
        return x, info["iterations"]
    fn = {"sample": es.autograd.matern_sample, "embed": es.autograd.es_adjoint, "sym": es.autograd.sym_cov_apply}[kind]
    y = fn(xs[0], *args)
    grad, = torch.autograd.grad(y, xs[0], xs[1])
    return y.detach(), grad


# ---- the work a pass cannot do without -----------------------------------------------------------------


def _transform_flops(voxels, ndim, taps, levels, low_only):
    """Multiply-adds (two operations each) of one analysis or synthesis sweep over `levels` levels."""
    total, size = 0.0, float(voxels)
    for _ in range(levels):
        for axis in range(ndim):  # every axis halves what the next one sees where only low bands are kept
            total += 2 * taps * size * (0.5 ** (axis + 1) if low_only else 1.0)
        size /= 2 ** ndim
    return total


def work(case):
    kind = case["kind"]
    if kind == "ragged":
        got = [work(dict(kind="cov", batch=1, order=o, levels=m, **{"n%d" % k: v for k, v in enumerate(shape)}))
               for shape, o, m, _ in _ragged_descs(case)]
        return {"bytes": sum(g["bytes"] for g in got), "flops": sum(g["flops"] for g in got)}
    grid, taps, m = _grid(case), 2 * case["order"], case["levels"]
    n = case["batch"] * math.prod(grid)
    bank = _transform_flops(n, len(grid), taps, m, False)
    cov = 2 * _transform_flops(n, len(grid), taps, max(0, m - 1), True) + 2.0 * n  # projection form: low bands, two sweeps
    if kind == "cov":
        return {"bytes": 8.0 * n, "flops": cov}
    if kind == "norm":
        return {"bytes": 4.0 * n, "flops": bank + 2.0 * n}
    if kind in ("sample", "sym"):
        return {"bytes": 16.0 * n, "flops": 2 * cov}
    if kind == "embed":
        return {"bytes": 16.0 * n, "flops": 2 * bank}
    if kind == "pcg":  # two operators a step, and x, r, d, z read and x, r, d written
        return {"bytes": 12.0 * n + PCG_ITERS * (16.0 + 28.0) * n, "flops": PCG_ITERS * (2 * cov + 12.0 * n)}
    steps = range(1, GMRES_ITERS + 1)  # an operator a step, and the basis read for its products
    return {"bytes": 12.0 * n + sum((8.0 + 4.0 * k) * n for k in steps), "flops": sum(cov + 8.0 * k * n for k in steps)}


# ---- the same in 64 bits, from the definitions ----------------------------------------------------------


def _daubechies(order):
    """Low-pass taps of the minimum-phase filter with `order` vanishing moments (spectral factorisation)."""
    y = np.roots([math.comb(order - 1 + k, k) for k in range(order - 1, -1, -1)])
    poly = np.array([1.0 + 0j])
    for _ in range(order):
        poly = np.convolve(poly, [1.0, 1.0])
    for v in y:
        b = 2 - 4 * v
        z = (b + np.sqrt(b * b - 4 + 0j)) / 2
        poly = np.convolve(poly, [1.0, -(z if abs(z) < 1 else 1 / z)])
    h = poly.real
    return h * math.sqrt(2.0) / h.sum()


def _matrices(n, h, periodic, device):
    """(analysis, synthesis) matrices of one axis, each [low, high]: analysis l x n, synthesis n x l."""
    L = len(h)
    taps = [h, np.array([(-1) ** t * h[L - 1 - t] for t in range(L)])]
    ana, syn = [], []
    for f in taps:
        l = n // 2 if periodic else (n + L - 1) // 2
        a, b = np.zeros((l, n)), np.zeros((n, l))
        k = np.arange(l)
        for t in range(L):
            if periodic:
                np.add.at(a, (k, (2 * k + t) % n), f[t])
                continue
            p = (2 * k + t - (L - 2)) % (2 * n)  # half-point symmetric extension, period 2 n
            np.add.at(a, (k, np.where(p < n, p, 2 * n - 1 - p)), f[t])
            i = 2 * k + t - (L - 2)
            ok = (i >= 0) & (i < n)
            b[i[ok], k[ok]] += f[t]
        ana.append(torch.from_numpy(a).to(device))
        syn.append(torch.from_numpy(a.T.copy() if periodic else b).to(device))
    return ana, syn


def _along(mat, x, axis):
    moved = x.movedim(axis, -1)
    y = moved.reshape(-1, moved.shape[-1]) @ mat.t().contiguous()
    return y.reshape(moved.shape[:-1] + (mat.shape[0],)).movedim(-1, axis)


class _Exact:
    """The operators of one geometry in 64 bits: level by level, every band a product with one matrix an axis."""

    def __init__(self, grid, order, levels, device, periodic=True):
        self.nd, self.m, self.levels = len(grid), levels, []
        h, sides = _daubechies(order), tuple(grid)
        for _ in range(levels):
            self.levels.append([_matrices(n, h, periodic, device) for n in sides])
            sides = tuple(n // 2 if periodic else (n + len(h) - 1) // 2 for n in sides)

    def _patterns(self):
        return itertools.product((0, 1), repeat=self.nd)

    def _band(self, mats, x):
        for k, mat in enumerate(mats):
            x = _along(mat, x, k - self.nd)
        return x

    def weighted(self, x, weight, transpose=False, i=0):
        """W^{-1} D W x (transposed: (W^{-1} D W)^T x); `weight` of a level, 1 = finest."""
        if i == self.m:
            return x
        axes, out = self.levels[i], None
        for p in self._patterns():
            ana = [axes[k][0][e] for k, e in enumerate(p)]
            syn = [axes[k][1][e] for k, e in enumerate(p)]
            if transpose:
                ana, syn = [b.t() for b in syn], [a.t() for a in ana]
            c = self._band(ana, x)
            c = c * weight(i + 1) if any(p) else self.weighted(c, weight, transpose, i + 1)
            y = self._band(syn, c)
            out = y if out is None else out + y
        return out

    def coefficients(self, x, weight, i=0):
        """D W x in the packed layout."""
        if i == self.m:
            return x
        out = torch.empty_like(x)
        for p in self._patterns():
            c = self._band([self.levels[i][k][0][e] for k, e in enumerate(p)], x)
            c = c * weight(i + 1) if any(p) else self.coefficients(c, weight, i + 1)
            out[self._at(out, p)] = c
        return out

    def image(self, c, weight, i=0):
        """W^T D c of packed coefficients."""
        if i == self.m:
            return c
        out = 0.0
        for p in self._patterns():
            b = c[self._at(c, p)]
            b = b * weight(i + 1) if any(p) else self.image(b, weight, i + 1)
            out = out + self._band([self.levels[i][k][1][e] for k, e in enumerate(p)], b)
        return out

    def _at(self, x, p):
        half = [x.shape[k - self.nd] // 2 for k in range(self.nd)]
        return (Ellipsis,) + tuple(slice(e * h, (e + 1) * h) for e, h in zip(p, half))

    def detail(self, s, tau):
        return lambda i: 2.0 ** (-tau * s * (self.m - i))


def _dot(a, b):
    return (a * b).flatten(1).sum(1).reshape((-1,) + (1,) * (a.dim() - 1))


def _pcg(p, mask, op, s):
    b = mask * p
    x, r = torch.zeros_like(b), b.clone()
    z = op.weighted(r, op.detail(s, 2))
    d, rz = z.clone(), _dot(r, z)
    for _ in range(PCG_ITERS):
        ad = ALPHA * op.weighted(d, op.detail(-s, 2)) + mask * d
        a = rz / _dot(d, ad)
        x, r = x + a * d, r - a * ad
        z = op.weighted(r, op.detail(s, 2))
        new = _dot(r, z)
        d, rz = z + (new / rz) * d, new
    return x


def _gmres(p, mask, op, s):
    def apply(v):
        return op.weighted(mask * mask * v, op.detail(s, 2)) + ALPHA * v

    b = op.weighted(mask * p, op.detail(s, 2))
    beta = _dot(b, b).sqrt()
    basis = [b / beta]
    hess = torch.zeros((b.shape[0], GMRES_ITERS + 1, GMRES_ITERS), dtype=b.dtype)
    for k in range(GMRES_ITERS):
        w = apply(basis[k])
        for _ in range(2):
            for j, v in enumerate(basis):
                c = _dot(v, w)
                hess[:, j, k] += c.flatten().cpu()
                w = w - c * v
        norm = _dot(w, w).sqrt()
        hess[:, k + 1, k] = norm.flatten().cpu()
        basis.append(w / norm)
    rhs = torch.zeros((b.shape[0], GMRES_ITERS + 1, 1), dtype=b.dtype)
    rhs[:, 0, 0] = beta.flatten().cpu()
    y = torch.linalg.lstsq(hess, rhs).solution.to(b.device)
    return sum(y[:, k, 0].reshape(beta.shape) * basis[k] for k in range(GMRES_ITERS))


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    xs = [x.double() for x in _inputs(case, seed, device)]
    if kind == "ragged":
        out = []
        for x, (shape, order, levels, s) in zip(xs, _ragged_descs(case)):
            op = _Exact(shape, order, levels, device)
            out.append(op.weighted(x, op.detail(s, 2)))
        return out
    s = case["s"]
    op = _Exact(_grid(case), case["order"], case["levels"], device, periodic=kind != "sym")
    if kind == "cov":
        return op.weighted(xs[0], op.detail(s, 2))
    if kind == "norm":
        return op.coefficients(xs[0], op.detail(-s, 1)).square().flatten(1).sum(1)
    if kind == "sample":
        return op.weighted(xs[0], op.detail(s, 1)), op.weighted(xs[1], op.detail(s, 1))
    if kind == "embed":
        return op.coefficients(xs[0], op.detail(s, 1)), op.image(xs[1], op.detail(s, 1))
    if kind == "sym":
        return op.weighted(xs[0], op.detail(s, 2)), op.weighted(xs[1], op.detail(s, 2), transpose=True)
    return (_pcg if kind == "pcg" else _gmres)(xs[0], xs[1], op, s), None
