"""Captured iterations are kept while the material's kernel arguments are the
same and captured anew when one of them changes: the same sequence of
materials with graphs on and off gives the same results bit for bit."""
import numpy as np
import pytest

from paper_1411_0330_amd import inputs as I

from .gpu_util import context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics,precision,solver", [("scalar", "fp64", "cg"), ("scalar", "mixed", "cg"),
                                                      ("elastic", "mixed", "cg"), ("elastic", "fp64", "cg"),
                                                      ("scalar", "fp64", "basic"), ("elastic", "fp64", "eyre_milton")])
def test_changing_materials_with_graphs_equals_eager(lsh, physics, precision, solver):
    shape = (8, 16, 32)
    el = physics == "elastic"
    iso = (lambda a: I.elastic_from_young(a, 0.3)) if el else (lambda a: I.scalar_isotropic(a, 3))
    c = 6 if el else 3
    full = np.eye(c) + 0.1 * np.ones((c, c))
    p0, p1, p3 = (I.random_phases(shape, k, seed=s) for k, s in ((2, 1), (2, 2), (3, 3)))
    vox = 1.0 + 4.0 * np.random.default_rng(4).random(shape)
    vox = np.stack([vox / 1.2, vox / 2.6]) if el else vox[None]
    greens = ["truncated", "consistent", "filtered"] if el else ["truncated", "fd", "consistent", "filtered"]
    steps = [lambda x: None,
             lambda x: x.set_phases(p1, np.stack([iso(1.0), iso(4.0)])),          # another map, the same scalars
             lambda x: x.set_phases(p1, np.stack([iso(1.0), iso(6.0)])),
             lambda x: x.set_reference(iso(0.6)),
             *[(lambda g: lambda x: x.set_green(g, series=2 if g == "consistent" else None))(g) for g in greens],
             lambda x: x.set_voxel_moduli(vox),
             lambda x: x.set_voxel_moduli(1.5 * vox),                             # other voxels, the same scalars
             lambda x: x.set_phases(p3, np.stack([iso(1.0), iso(6.0), iso(3.0)])),
             lambda x: x.set_phases(p0, np.stack([iso(1.0), iso(0.6) + full])),   # full matrices
             lambda x: x.set_phases(p0, np.stack([iso(1.0), iso(4.0)]))]
    ctxs = []
    for on in (True, False):
        ctx = context(lsh, p0, np.stack([iso(1.0), iso(4.0)]), iso(0.5), physics, "filtered", precision, 2)
        ctx.set_persistent(False)
        ctx.set_graphs(on)
        ctxs.append(ctx)
    fixed = solver != "cg"
    last = None
    for k, step in enumerate(steps):
        got = []
        for ctx in ctxs:
            step(ctx)
            rep = ctx.solve(np.eye(c)[:2], solver, tol=1e-6 if precision == "mixed" else 1e-10,
                            maxit=12 if fixed else 400)
            got.append((rep["iterations"], ctx.effective(), ctx.field(1, "tau").cpu().numpy()))
        assert got[0][0] == got[1][0], k
        assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2]), k
        assert last is None or not np.array_equal(last, got[0][1]), k   # the step had an effect
        last = got[0][1]
