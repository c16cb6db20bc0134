"""The plane passes (x and y transforms of a plane in one workgroup) against the
oracle's operator and against the separate passes (LSH_PLANE=0): square planes
of every compiled length, planes with run-time lengths down to the smallest,
phase maps with a masked phase and per-voxel moduli, and whole solves through
every epilogue (conjugate gradients, refinement, strain, MINRES's q = Lv)."""
import numpy as np
import pytest

from oracle import operator as op
from paper_1411_0330_amd import inputs as I

from .gpu_util import context, problem, rel_max_err, to_dev

pytestmark = pytest.mark.gpu

SCAL = np.stack([I.scalar_isotropic(a, 3) for a in (1.0, 10.0, 0.5)])
ELAS = np.stack([I.elastic_from_young(1.0, 0.3), I.elastic_from_young(10.0, 0.2), I.elastic_from_young(0.5, 0.3)])
A0 = {"scalar": SCAL[2], "elastic": ELAS[2]}   # the third phase lies outside I0


def _ctx(lsh, physics, shape, precision, nload, green="filtered", medium="phases"):
    if medium == "phases":
        ph = I.random_phases(shape, 3, seed=3)
        moduli = SCAL if physics == "scalar" else ELAS
        return context(lsh, ph, moduli, A0[physics], physics, green, precision, nload), \
            problem(ph, moduli, A0[physics], physics, green)
    rng = np.random.default_rng(5)
    E = 1.0 + 9.0 * rng.random(shape)
    ctx = lsh.Context(shape, physics, precision, max_loads=nload)
    ctx.set_reference(A0[physics])
    if physics == "scalar":
        ctx.set_voxel_moduli(E[None])
        vox = E[..., None, None] * np.eye(3)
    else:
        ctx.set_voxel_moduli(np.stack([E / 1.2, E / 2.6]))   # nu = 0.3
        vox = E[..., None, None] * I.elastic_from_young(1.0, 0.3)
    ctx.set_green(green)
    c = vox.shape[-1]
    return ctx, op.Problem(np.zeros(shape, np.uint8), np.zeros((1, c, c)), A0[physics], physics, green, voxel=vox)


@pytest.mark.parametrize("shape", [(2, 2, 4), (2, 4, 8), (4, 16, 16), (2, 32, 32), (2, 48, 48), (4, 48, 80), (2, 64, 64),
                                   (2, 80, 80), (16, 96, 96), (16, 128, 128), (16, 160, 160), (16, 80, 128),
                                   (2, 1024, 4), (2, 2, 1024)])
@pytest.mark.parametrize("physics,dtype,medium", [("scalar", "f64", "phases"), ("scalar", "f32", "voxel"),
                                                  ("elastic", "f32", "phases"), ("elastic", "f64", "voxel")])
def test_plane_operator_matches_oracle(lsh, shape, physics, dtype, medium):
    if shape[0] == 16 and physics == "elastic":
        shape = (8,) + shape[1:]   # 48 planes and components, the least that a large plane needs
    nload = 2 if np.prod(shape) < 40000 else 1
    ctx, pb = _ctx(lsh, physics, shape, "mixed" if dtype == "f32" else "fp64", nload, medium=medium)
    tau = I.random_field(shape, pb.c, nload, seed=7) * op.mask(pb)
    out = ctx.apply(to_dev(tau, dtype)).cpu().numpy()
    tol = 1e-12 if dtype == "f64" else 1e-5
    for l in range(nload):
        assert rel_max_err(out[l], op.apply(pb, tau[l])) <= tol


@pytest.mark.parametrize("shape", [(16, 16, 16), (4, 48, 80), (16, 64, 64), (16, 80, 80), (16, 96, 96), (16, 128, 128)])
@pytest.mark.parametrize("physics,precision,medium,solver", [
    ("scalar", "mixed", "phases", "cg"), ("scalar", "fp64", "voxel", "cg"), ("elastic", "mixed", "voxel", "cg"),
    ("elastic", "fp64", "phases", "cg"), ("scalar", "fp64", "phases", "minres"), ("scalar", "fp64", "phases", "basic")])
def test_plane_solve_equals_separate_passes(lsh, monkeypatch, shape, physics, precision, medium, solver):
    got = []
    for on in ("1", "0"):
        monkeypatch.setenv("LSH_PLANE", on)
        ctx, _ = _ctx(lsh, physics, shape, precision, 2, medium=medium)
        ctx.set_persistent(False)
        tol = 1e-10 if precision == "fp64" else 1e-6
        rep = ctx.solve(np.eye(ctx.c)[:2], solver, tol=tol, maxit=7 if solver == "basic" else 2000)
        got.append((rep["iterations"], ctx.effective(), ctx.field(1, "tau").cpu().numpy(),
                    ctx.field(0, "strain").cpu().numpy()))
    (i1, a1, t1, e1), (i0, a0, t0, e0) = got
    assert max(abs(x - y) for x, y in zip(i1, i0)) <= 1
    # the same recurrences up to rounding; a step more or less moves the result by the tolerance
    tol = 1e-8 if precision == "fp64" else 1e-4
    assert rel_max_err(a1, a0) <= tol and rel_max_err(t1, t0) <= tol and rel_max_err(e1, e0) <= tol


@pytest.mark.parametrize("shape", [(2, 4), (4, 16), (48, 64), (80, 48), (160, 96), (16, 128), (128, 80), (96, 160),
                                   (64, 192), (32, 256), (256, 16), (16, 512), (512, 8), (4, 1024), (1024, 16)])
@pytest.mark.parametrize("green", ["filtered", "truncated", "fd"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_2d_operator_matches_oracle(lsh, shape, green, dtype):
    # y transforms and the Green operator in one pass; x over blocks of rows
    ph = I.random_phases(shape, 2, seed=2)
    moduli = np.stack([I.scalar_isotropic(1.0, 2), I.scalar_isotropic(10.0, 2)])
    A0_ = I.scalar_isotropic(0.5, 2)
    pb = problem(ph, moduli, A0_, "scalar", green)
    ctx = context(lsh, ph, moduli, A0_, "scalar", green, "mixed" if dtype == "f32" else "fp64", 2)
    tau = I.random_field(shape, 2, 2, seed=7)
    out = ctx.apply(to_dev(tau, dtype)).cpu().numpy()
    for l in range(2):
        assert rel_max_err(out[l], op.apply(pb, tau[l])) <= (1e-12 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("shape", [(2, 16, 48), (4, 64, 80), (2, 32, 192), (4, 64, 256), (2, 16, 512), (2, 8, 1024),
                                   (16, 256, 96), (16, 192, 160), (8, 128, 128), (32, 256, 128),
                                   (64, 128), (128, 256), (32, 512), (16, 1024), (96, 192)])
@pytest.mark.parametrize("physics,precision", [("scalar", "mixed"), ("scalar", "fp64"), ("elastic", "mixed"),
                                               ("elastic", "fp64")])
def test_row_blocks_equal_the_passes_in_registers(lsh, monkeypatch, shape, physics, precision):
    if len(shape) == 2 and physics == "elastic":
        pytest.skip("elasticity is three-dimensional")
    d = len(shape)
    ph = I.random_phases(shape, 2, seed=4)
    moduli = ELAS[:2] if physics == "elastic" else np.stack([I.scalar_isotropic(a, d) for a in (1.0, 10.0)])
    ref = A0["elastic"] if physics == "elastic" else I.scalar_isotropic(0.5, d)
    got = []
    for on in ("1", "0"):
        monkeypatch.setenv("LSH_PLANE", on)
        ctx = context(lsh, ph, moduli, ref, physics, "filtered", precision, 2)
        rep = ctx.solve(np.eye(ctx.c)[:2], "cg", tol=1e-10 if precision == "fp64" else 1e-6, maxit=2000)
        got.append((rep["iterations"], ctx.effective(), ctx.field(1, "tau").cpu().numpy(),
                    ctx.field(0, "strain").cpu().numpy()))
    (i1, a1, t1, e1), (i0, a0, t0, e0) = got
    assert max(abs(x - y) for x, y in zip(i1, i0)) <= 1
    tol = 1e-8 if precision == "fp64" else 1e-4
    assert rel_max_err(a1, a0) <= tol and rel_max_err(t1, t0) <= tol and rel_max_err(e1, e0) <= tol
