"""The work that users of this framework have it do, as timed cases.

A case is a dict of plain values; ``prepare`` makes what a user's program holds
before the call (context, microstructure, fields), ``run`` is one pass through
the public entry points, ``work`` what that pass cannot do without and
``exact`` the same outputs in float64 from plain torch.

Kinds of cases:

* ``apply``     one application of the operator of eq. (13), the call of an
                outer Krylov solver written by the user;
* ``solve``     a new microstructure: the material is set, the batched loads
                are solved and the fields come out, with the effective matrix;
* ``gradient``  forward and backward of the homogenised matrix with respect to
                per-voxel moduli, through torch.autograd;
* ``ensemble``  a few realisations solved together, each on its own stream.
"""
import math
import os

import numpy as np
import torch

import paper_1411_0330_amd as pkg
from paper_1411_0330_amd import inputs, lsh
from paper_1411_0330_amd.autograd import homogenized_gram, young_to_bulk_shear

DEV = "cuda:0"
TUNE_CACHE = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "tune_cache.txt")
AXES = (2, 4, 8, 16, 32, 48, 64, 80, 96, 128, 160, 192, 256, 512, 1024)


def _case(kind, name=None, **kw):
    c = {"kind": kind, "physics": "scalar", "nz": 0, "ny": 64, "nx": 64, "loads": 1, "precision": "fp64",
         "green": "filtered", "medium": "phases", "contrast": 10.0, "reference": "soft", "solver": "cg",
         "tol": 1e-10, "tuned": False, "strain": False, "members": 1}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a user's own Krylov loop on a small box, where latency counts
        _case("apply", "apply_scalar_16_f64", nz=16, ny=16, nx=16, contrast=100.0),
        # an odd box (axes of 3 and 5 times a power of two), per-voxel conductivities, FP32
        _case("apply", "apply_scalar_48x48x80_f32", nz=48, ny=48, nx=80, loads=3, precision="mixed", medium="voxel"),
        # an ordinary elastic box in FP64, the six unit strains together
        _case("apply", "apply_elastic_64_f64", physics="elastic", nz=64, ny=64, nx=64, loads=6),
        # the operator at the benchmark's full size in FP32
        _case("apply", "apply_elastic_256_f32", physics="elastic", nz=256, ny=256, nx=256, loads=6, precision="mixed",
              tuned=True),
        # the smallest whole solve: a 64 x 64 cell in 2D, both loads, reference between the phases
        _case("solve", "cell_64_cg_f64", ny=64, nx=64, loads=2, green="truncated", reference="between"),
        # a finely resolved 2D plate
        _case("solve", "plate_512_cg_f64", ny=512, nx=512, loads=2, contrast=20.0),
        # the quick start: elastic 64^3, six loads, mixed precision
        _case("solve", "elastic_64_cg_mixed", physics="elastic", nz=64, ny=64, nx=64, loads=6, precision="mixed",
              tol=1e-6),
        # conduction at contrast 100, 128^3, mixed precision to a tight tolerance
        _case("solve", "boolean_128_cg_mixed", nz=128, ny=128, nx=128, loads=3, precision="mixed", contrast=100.0,
              tol=1e-8),
        # the benchmark's step: elastic 256^3, six loads, fields and strains out, tuned shapes from the cache
        _case("solve", "elastic_256_cg_mixed", physics="elastic", nz=256, ny=256, nx=256, loads=6, precision="mixed",
              tol=1e-6, tuned=True, strain=True),
        # a reference between the phases: the symmetric indefinite system
        _case("solve", "indefinite_64_minres_f64", nz=64, ny=64, nx=64, loads=3, green="truncated",
              reference="between", solver="minres"),
        # sensitivities of two effective moduli with respect to every voxel's stiffness
        _case("gradient", "sensitivity_192_f64", physics="elastic", nz=192, ny=192, nx=192, loads=2, medium="voxel"),
        # stochastic homogenisation: realisations of mixed sizes, four in flight
        _case("ensemble", "ensemble_8_cg_mixed", nz=160, ny=160, nx=160, loads=3, precision="mixed", medium="voxel",
              contrast=20.0, tol=1e-6, members=8),
    ]


def _log_axis(rng, lo, hi):
    """An axis length of the supported ones, spread over the logarithm."""
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(AXES, key=lambda n: abs(math.log(n / want)))


def draw(rng):
    limit = 0.7 * work(listed()[8])["bytes"]
    while True:
        kind = rng.choice(("apply", "apply", "apply", "solve", "solve", "solve", "solve", "gradient", "ensemble"))
        physics = rng.choice(("scalar", "elastic"))
        two_d = physics == "scalar" and kind != "ensemble" and rng.random() < 0.3
        if two_d:
            shape = dict(nz=0, ny=_log_axis(rng, 8, 1024), nx=_log_axis(rng, 8, 1024))
        elif rng.random() < 0.5:
            n = _log_axis(rng, 16, 192)
            shape = dict(nz=n, ny=n, nx=n)
        else:
            shape = dict(nz=_log_axis(rng, 4, 256), ny=_log_axis(rng, 8, 256), nx=_log_axis(rng, 8, 256))
        c = 6 if physics == "elastic" else (2 if two_d else 3)
        precision = rng.choice(("fp64", "mixed"))
        kw = dict(physics=physics, loads=rng.randint(1, c), precision=precision,
                  medium=rng.choice(("phases", "phases", "voxel")),
                  green=rng.choice(("filtered", "filtered", "truncated")),
                  contrast=round(math.exp(rng.uniform(math.log(3.0), math.log(100.0))), 1),
                  tol=1e-10 if precision == "fp64" else rng.choice((1e-6, 1e-8)), **shape)
        if kind == "apply" and physics == "scalar" and rng.random() < 0.2:
            kw["green"] = "fd"
        if kind == "solve":
            kw["strain"] = rng.random() < 0.3
            if precision == "fp64" and rng.random() < 0.3:
                kw["solver"] = rng.choice(("minres", "symmlq", "eyre_milton"))
                kw["contrast"] = min(kw["contrast"], 10.0)
                if kw["solver"] == "eyre_milton" and (physics == "elastic" or kw["medium"] == "voxel"):
                    kw["solver"] = "minres"
        if kind == "gradient":
            kw.update(medium="voxel", green="filtered", loads=min(2, c), precision="fp64", tol=1e-10)
        if kind == "ensemble":
            n = _log_axis(rng, 48, 160)
            kw.update(physics="scalar", nz=n, ny=n, nx=n, loads=3, precision="mixed", medium="voxel", contrast=20.0,
                      tol=1e-6, members=rng.randint(2, 8), green="filtered")
        case = _case(kind, **kw)
        if work(case)["bytes"] <= limit:
            return case


# ---------------------------------------------------------------------------
# inputs, made on the GPU from the seed
# ---------------------------------------------------------------------------
def _shape(case):
    return ((case["nz"],) if case["nz"] else ()) + (case["ny"], case["nx"])


def _comps(case):
    return 6 if case["physics"] == "elastic" else len(_shape(case))


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _gaussian(shape, corr, gen):
    """Periodic Gaussian random field of correlation length ``corr`` voxels, mean 0 and variance 1."""
    w = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64)
    k2 = torch.zeros((), device=DEV, dtype=torch.float64)
    for a, n in enumerate(shape):
        f = torch.fft.fftfreq(n, device=DEV, dtype=torch.float64)
        k2 = k2 + (f * f).view([-1 if i == a else 1 for i in range(len(shape))])
    g = torch.fft.ifftn(torch.fft.fftn(w) * torch.exp(-2.0 * math.pi ** 2 * corr ** 2 * k2)).real
    return ((g - g.mean()) / g.std()).contiguous()


def _member_sizes(case):
    """Cube sizes of an ensemble: the four sizes of its range in turn, up to the case's own."""
    sizes = [n for n in (64, 96, 128, 160) if n <= case["nx"]] or [case["nx"]]
    return [sizes[-1 - i % len(sizes)] for i in range(case["members"])]


def _medium(case, shape, gen):
    """Material of one box: phase map and moduli, or per-voxel coefficients, with the reference A0."""
    el = case["physics"] == "elastic"
    d = len(shape)
    k = case["contrast"]
    g = _gaussian(shape, min(4.0, max(1.0, min(shape) / 16.0)), gen)
    if case["medium"] == "voxel":
        if el:
            E = 1.0 + (k - 1.0) * torch.sigmoid(2.0 * g)
            K, mu = young_to_bulk_shear(E, 0.3)
            return {"coef": torch.stack([K, mu]).contiguous(), "A0": inputs.elastic_from_young(0.5, 0.3)}
        a = torch.exp(0.25 * math.log(k) * g)
        return {"coef": a[None].contiguous(), "A0": inputs.scalar_isotropic(0.5 * float(a.min()), d)}
    phase = (g > 0.6).to(torch.uint8).contiguous()
    if el:
        soft, hard = inputs.elastic_from_young(1.0, 0.3), inputs.elastic_from_young(k, 0.2)
        mu0 = 0.5 * inputs.lame_from_young(1.0, 0.3)[1]
        if case["reference"] == "between":
            mu0 = 0.5 * (inputs.lame_from_young(1.0, 0.3)[1] + inputs.lame_from_young(k, 0.2)[1])
        A0 = inputs.elastic_isotropic_mandel(2.0 * mu0 * 0.3 / 0.4, mu0)
    else:
        soft, hard = inputs.scalar_isotropic(1.0, d), inputs.scalar_isotropic(k, d)
        a0 = 0.5 * (1.0 + k) if case["reference"] == "between" else 0.5
        if case["solver"] == "eyre_milton":
            a0 = math.sqrt(k)
        A0 = inputs.scalar_isotropic(a0, d)
    return {"phase": phase, "moduli": np.stack([soft, hard]), "A0": A0}


def _context(case, shape, med, stream=None):
    ctx = lsh.Context(shape, case["physics"], case["precision"], max_loads=case["loads"], device=DEV, stream=stream)
    ctx.set_reference(med["A0"])
    _set_medium(ctx, med)
    ctx.set_green(case["green"])
    if case["tuned"]:
        ctx.autotune(case["loads"], cache=TUNE_CACHE)
    return ctx


def _set_medium(ctx, med):
    if "coef" in med:
        ctx.set_voxel_moduli(med["coef"])
    else:
        ctx.set_phases(med["phase"], med["moduli"])


def _loads(case, c):
    if case["kind"] == "gradient":
        return inputs.unit_loads(c)[[0, c - 1]][: case["loads"]]
    return inputs.unit_loads(c)[: case["loads"]]


def _inputs(case, seed):
    """Everything random of one case, made alike for prepare and exact."""
    gen = _gen(seed)
    if case["kind"] == "ensemble":
        return [_medium(case, (n, n, n), gen) for n in _member_sizes(case)]
    shape = _shape(case)
    if case["kind"] == "gradient":
        theta = _gaussian(shape, 2.0, gen)
        if case["physics"] == "elastic":
            return {"theta": theta, "A0": inputs.elastic_from_young(0.5, 0.3)}
        return {"theta": theta, "A0": inputs.scalar_isotropic(0.5, len(shape))}
    med = _medium(case, shape, gen)
    if case["kind"] == "apply":
        dt = torch.float64 if case["precision"] == "fp64" else torch.float32
        med["tau"] = torch.randn((case["loads"], _comps(case)) + shape, generator=gen, device=DEV, dtype=dt)
    return med


def _coef_of(theta, elastic):
    """Per-voxel coefficients of a design field theta: E = 1 + 9 sigmoid(theta) at fixed Poisson's ratio, or a alike."""
    E = 1.0 + 9.0 * torch.sigmoid(theta)
    if elastic:
        return torch.stack(young_to_bulk_shear(E, 0.3))
    return E[None]


def prepare(case, seed):
    made = _inputs(case, seed)
    kind = case["kind"]
    if kind == "ensemble":
        streams = [torch.cuda.Stream() for _ in made]
        ctxs = [_context(case, tuple(m["coef"].shape[1:]), m, s) for m, s in zip(made, streams)]
        return {"case": case, "ctxs": ctxs, "media": made, "streams": streams,
                "loads": [_loads(case, 3) for _ in made]}
    shape = _shape(case)
    if kind == "gradient":
        el = case["physics"] == "elastic"
        ctx = lsh.Context(shape, case["physics"], "fp64", max_loads=case["loads"], device=DEV)
        ctx.set_reference(made["A0"])
        ctx.set_green(case["green"])
        return {"case": case, "ctx": ctx, "theta": made["theta"].requires_grad_(True), "elastic": el,
                "loads": _loads(case, _comps(case))}
    ctx = _context(case, shape, made)
    return {"case": case, "ctx": ctx, "medium": made, "loads": _loads(case, _comps(case))}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "apply":
        return state["ctx"].apply(state["medium"]["tau"])
    if kind == "gradient":
        G = homogenized_gram(_coef_of(state["theta"], state["elastic"]), state["ctx"], state["loads"],
                             tol=case["tol"])
        J = G[0, 0] + 0.5 * G[-1, -1] if G.shape[0] > 1 else G[0, 0]
        (grad,) = torch.autograd.grad(J, state["theta"])
        return {"G": G.detach(), "grad": grad}
    # a mixed solve's fields and matrix are read in FP32, an FP64 one's in FP64
    out_t = "f64" if case["precision"] == "fp64" else "f32"
    np_t = np.float64 if case["precision"] == "fp64" else np.float32
    if kind == "ensemble":
        for ctx, med in zip(state["ctxs"], state["media"]):
            _set_medium(ctx, med)
        lsh.solve_many(state["ctxs"], state["loads"], solver=case["solver"], tol=case["tol"], maxit=2000, threads=4)
        return {"effective": [c.effective().astype(np_t) for c in state["ctxs"]],
                "tau": [c.field(l, "tau", dtype=out_t) for c in state["ctxs"] for l in range(case["loads"])]}
    ctx = state["ctx"]
    _set_medium(ctx, state["medium"])
    ctx.solve(state["loads"], case["solver"], tol=case["tol"], maxit=4000)
    out = {"effective": ctx.effective().astype(np_t),
           "tau": [ctx.field(l, "tau", dtype=out_t) for l in range(case["loads"])]}
    if case["strain"]:
        out["strain"] = [ctx.field(l, "strain", dtype=out_t) for l in range(case["loads"])]
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _iterations(case):
    """Iterations that such a solve takes, near enough: the conjugate-gradient estimate with the condition number
    of the contrast against a reference of half the softest phase."""
    return max(1, round(0.7 * math.sqrt(2.0 * case["contrast"]) * math.log(2.0 / case["tol"])))


def work(case):
    """An application reads and writes a field and reads the material; an iteration of a solve reads and writes the
    solution, the residual and the direction once, and reads the material.  A transform of n points is 5 n log2 n
    operations (half of that on real data), there and back for every component, and a c x c product per wave-vector
    and voxel."""
    if case["kind"] == "ensemble":
        one = [work(dict(case, kind="solve", nz=n, ny=n, nx=n, members=1)) for n in _member_sizes(case)]
        return {k: sum(w[k] for w in one) for k in ("bytes", "flops")}
    shape, c, nl = _shape(case), _comps(case), case["loads"]
    vox = float(np.prod(shape))
    s = 8 if case["precision"] == "fp64" else 4
    mat = 1.0 if case["medium"] == "phases" else s * (2.0 if case["physics"] == "elastic" else 1.0)
    field = c * s * vox * nl
    flops = nl * vox * (2 * 2.5 * c * math.log2(vox) + 2.0 * c * c + 3.0 * c)
    if case["kind"] == "apply":
        return {"bytes": 2 * field + mat * vox, "flops": flops}
    its = _iterations(case)
    out = (2 if case["strain"] else 1) * field
    return {"bytes": its * (6 * field + mat * vox) + out, "flops": its * (flops + 10.0 * c * nl * vox)}


# ---------------------------------------------------------------------------
# the same in float64, with plain torch
# ---------------------------------------------------------------------------
class _Exact:
    """The operator of eq. (13) on one box in float64: rfftn, the Green operator as a real symmetric matrix per
    wave-vector (complex Hermitian for finite differences), and the local inverse per voxel."""

    def __init__(self, case, shape, med, A0):
        self.case, self.shape, self.A0 = case, shape, np.asarray(A0)
        self.el = case["physics"] == "elastic"
        self.c = 6 if self.el else len(shape)
        self.axes = tuple(range(1, 1 + len(shape)))
        f64 = dict(device=DEV, dtype=torch.float64)
        d = len(shape)
        self.k = []     # index per physical axis (x first), broadcast over the half spectrum
        for p in range(d):
            a = d - 1 - p
            n = shape[a]
            k = torch.arange(n // 2 + 1 if p == 0 else n, **f64)
            self.k.append(k.view([-1 if i == a else 1 for i in range(d)]))
        self.n = [shape[d - 1 - p] for p in range(d)]
        self._local(med, f64)
        self._green(f64)

    def _local(self, med, f64):
        A0 = self.A0
        if "coef" in med:
            coef = med["coef"].to(torch.float64)
            if self.el:
                mu0 = 0.5 * A0[3, 3]
                K0 = A0[0, 1] + 2.0 * mu0 / 3.0
                dK, dm = coef[0] - K0, coef[1] - mu0
            else:
                dK, dm = None, coef[0] - A0[0, 0]
        else:
            ph = med["phase"].to(torch.int64)
            mods = np.asarray(med["moduli"])
            if self.el:
                mu0 = 0.5 * A0[3, 3]
                K0 = A0[0, 1] + 2.0 * mu0 / 3.0
                mu = 0.5 * mods[:, 3, 3]
                K = mods[:, 0, 1] + 2.0 * mu / 3.0
                dK, dm = torch.tensor(K - K0, **f64)[ph], torch.tensor(mu - mu0, **f64)[ph]
            else:
                dK, dm = None, torch.tensor(mods[:, 0, 0] - A0[0, 0], **f64)[ph]
        self.dK, self.dm = dK, dm

    def dinv(self, t):
        """(A - A0)^{-1} t"""
        if not self.el:
            return t / self.dm
        tr = (t[0] + t[1] + t[2]) / 3.0
        out = t / (2.0 * self.dm)
        out[:3] += tr * (1.0 / (3.0 * self.dK) - 1.0 / (2.0 * self.dm))
        return out

    def dmul(self, e):
        """(A - A0) e"""
        if not self.el:
            return e * self.dm
        tr = e[0] + e[1] + e[2]
        out = e * (2.0 * self.dm)
        out[:3] += tr * (self.dK - 2.0 * self.dm / 3.0)
        return out

    def _term(self, xi):
        """Upper triangle of the continuous operator along xi (zero at xi = 0)."""
        n2 = sum(x * x for x in xi)
        c = self.c
        if not self.el:
            den = sum(self.A0[i, j] * xi[i] * xi[j] for i in range(c) for j in range(c))
            inv = torch.where(den > 0, 1.0 / torch.where(den > 0, den, torch.ones_like(den)), torch.zeros_like(den))
            return [xi[i] * xi[j] * inv for i in range(c) for j in range(i, c)]
        r = torch.where(n2 > 0, 1.0 / torch.sqrt(torch.where(n2 > 0, n2, torch.ones_like(n2))), torch.zeros_like(n2))
        u = [x * r for x in xi]
        lam, mu = self.A0[0, 1], 0.5 * self.A0[3, 3]
        kappa = (lam + mu) / (mu * (lam + 2.0 * mu))
        ij = [(0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1)]
        w = [1.0, 1.0, 1.0, math.sqrt(2.0), math.sqrt(2.0), math.sqrt(2.0)]
        on = (n2 > 0).to(torch.float64)
        out = []
        for a in range(6):
            for b in range(a, 6):
                (i, j), (k, l) = ij[a], ij[b]
                v = -kappa * u[i] * u[j] * u[k] * u[l]
                for (p, q, s, t) in ((i, k, j, l), (i, l, j, k), (j, k, i, l), (j, l, i, k)):
                    if p == q:
                        v = v + on * u[s] * u[t] / (4.0 * mu)
                out.append(w[a] * w[b] * v)
        return out

    def _green(self, f64):
        k, n, d, c = self.k, self.n, len(self.n), self.c
        self.V = None
        if self.case["green"] == "fd":
            V = [(torch.exp(2j * math.pi * k[a] / n[a]) - 1.0) * n[a] for a in range(d)]
            den = sum((V[i].conj() * V[j]).real * self.A0[i, j] for i in range(d) for j in range(d))
            self.V = V
            self.iden = torch.where(den > 0, 1.0 / torch.where(den > 0, den, torch.ones_like(den)),
                                    torch.zeros_like(den))
            return
        if self.case["green"] == "truncated":
            xi = [torch.where(k[a] <= n[a] // 2, k[a], k[a] - n[a]) for a in range(d)]
            M = self._term(xi)
            nyq = sum((k[a] == n[a] // 2).to(torch.float64) for a in range(d)) > 0
            inv = np.linalg.inv(self.A0)
            flat = [inv[i, j] for i in range(c) for j in range(i, c)]
            self.M = [torch.where(nyq, torch.full_like(m, f), m) for m, f in zip(M, flat)]
            return
        total = None
        for alias in range(1 << d):
            w, xi = 1.0, []
            for a in range(d):
                t = math.pi * k[a] / (2.0 * n[a])
                lo = (alias >> a) & 1
                w = w * (torch.sin(t) if lo else torch.cos(t)) ** 2
                xi.append(k[a] - n[a] if lo else k[a])
            term = self._term(xi)
            total = [w * m for m in term] if total is None else [s + w * m for s, m in zip(total, term)]
        self.M = total

    def gamma(self, t):
        h = torch.fft.rfftn(t, dim=self.axes)
        if self.V is not None:
            s = sum(v.conj() * h[i] for i, v in enumerate(self.V)) * self.iden
            o = torch.stack([v * s for v in self.V])
        else:
            c, q = self.c, 0
            o = torch.zeros_like(h)
            for i in range(c):
                for j in range(i, c):
                    m = self.M[q]
                    o[i] += m * h[j]
                    if i != j:
                        o[j] += m * h[i]
                    q += 1
        return torch.fft.irfftn(o, s=self.shape, dim=self.axes)

    def L(self, t):
        return self.dinv(t) + self.gamma(t)

    def cg(self, p, tol=1e-13, maxit=2000):
        """tau of the load p, by conjugate gradients in float64 (A0 softer than every voxel)."""
        b = torch.as_tensor(p, device=DEV, dtype=torch.float64).view([-1] + [1] * len(self.shape))
        b = b.expand((self.c,) + tuple(self.shape)).contiguous()
        x, r = torch.zeros_like(b), b.clone()
        q = r.clone()
        rr = float((r * r).sum())
        stop = tol * tol * rr
        for _ in range(maxit):
            Lq = self.L(q)
            alpha = rr / float((q * Lq).sum())
            x += alpha * q
            r -= alpha * Lq
            new = float((r * r).sum())
            if new <= stop:
                break
            q = r + (new / rr) * q
            rr = new
        return x

    def strain(self, p, t):
        return torch.as_tensor(p, device=DEV, dtype=torch.float64).view([-1] + [1] * len(self.shape)) - self.gamma(t)


def _exact_solve(case, shape, med, loads):
    """tau, strain and effective rows of every load.  With the reference between the phases (truncated operator) the
    strain does not depend on the reference: it is solved against a soft one and tau formed from it."""
    ex = _Exact(case, shape, med, med["A0"])
    soft = ex
    if case["reference"] == "between" or case["solver"] == "eyre_milton":
        if case["green"] != "truncated":
            return None
        m2 = _medium(dict(case, reference="soft", solver="cg"), shape, _gen(0))
        soft = _Exact(case, shape, med, m2["A0"])
    taus, eps, eff = [], [], []
    for p in loads:
        t = soft.cg(p)
        e = soft.strain(p, t)
        if soft is not ex:
            t = ex.dmul(soft.dinv(t))
        taus.append(t)
        eps.append(e)
        eff.append(ex.A0 @ np.asarray(p) + t.flatten(1).mean(dim=1).cpu().numpy())
    return taus, eps, np.stack(eff)


def exact(case, seed):
    its = 0.7 * math.sqrt(2.0 * case["contrast"]) * math.log(2e13)
    boxes = [n ** 3 for n in _member_sizes(case)] if case["kind"] == "ensemble" else [float(np.prod(_shape(case)))]
    vox = sum(boxes) * case["loads"] * _comps(case)
    if case["kind"] != "apply" and its * vox > 10e9 * (2.0 if case["physics"] == "scalar" else 1.0):
        return None     # over about 20 seconds
    made = _inputs(case, seed)
    if case["kind"] == "apply":
        ex = _Exact(case, _shape(case), made, made["A0"])
        out = torch.empty(made["tau"].shape, device=DEV, dtype=torch.float64)
        for l in range(case["loads"]):
            out[l] = ex.L(made["tau"][l].to(torch.float64))
        return out
    if case["kind"] == "ensemble":
        eff, tau = [], []
        for m in made:
            t, _, e = _exact_solve(case, tuple(m["coef"].shape[1:]), m, _loads(case, 3))
            eff.append(e)
            tau += t
        return {"effective": eff, "tau": tau}
    shape, loads = _shape(case), _loads(case, _comps(case))
    if case["kind"] == "gradient":
        el = case["physics"] == "elastic"
        theta = made["theta"].requires_grad_(True)
        coef = _coef_of(theta, el)
        med = {"coef": coef.detach(), "A0": made["A0"]}
        _, eps, eff = _exact_solve(case, shape, med, loads)
        G = np.asarray(loads) @ eff.T
        w = [1.0] if len(eps) == 1 else [1.0] + [0.0] * (len(eps) - 2) + [0.5]
        vox = float(np.prod(shape))
        ee = sum(wl * (e * e).sum(dim=0) for wl, e in zip(w, eps)) / vox
        if el:
            tt = sum(wl * (e[0] + e[1] + e[2]) ** 2 for wl, e in zip(w, eps)) / vox
            g = torch.stack([tt, 2.0 * (ee - tt / 3.0)])
        else:
            g = ee[None]
        (grad,) = torch.autograd.grad(coef, theta, grad_outputs=g)
        return {"G": torch.tensor(0.5 * (G + G.T), device=DEV), "grad": grad}
    solved = _exact_solve(case, shape, made, loads)
    if solved is None:
        return None
    taus, eps, eff = solved
    out = {"effective": eff, "tau": taus}
    if case["strain"]:
        out["strain"] = eps
    return out
