"""Launch and byte counts of the kernel timing: every iteration once, each with
the loads that iterate in it."""
import numpy as np
import pytest

from paper_1411_0330_amd import inputs as I

from .gpu_util import context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("physics,solver,shape", [("scalar", "cg", (16, 32, 32)), ("elastic", "cg", (8, 16, 16)),
                                                  ("scalar", "minres", (16, 32, 32)), ("scalar", "basic", (8, 16, 16)),
                                                  ("scalar", "symmlq", (8, 16, 16)), ("scalar", "cg", (64, 128))])
def test_timed_launches_are_those_of_the_iterations(lsh, physics, solver, shape):
    iso = (lambda a: I.elastic_from_young(a, 0.3)) if physics == "elastic" else \
        (lambda a: I.scalar_isotropic(a, len(shape)))
    c = 6 if physics == "elastic" else len(shape)
    a0 = 3.0 if solver == "basic" else 0.5
    ph = I.random_phases(shape, 2, seed=3)
    ph[..., :, : shape[-1] // 2] = 0   # the loads converge at different steps
    ctx = context(lsh, ph, np.stack([iso(1.0), iso(5.0)]), iso(a0), physics, "filtered", "fp64", 2)
    ctx.set_persistent(False)
    names = ("xfwd_f64", "xinv_f64")

    def run(loads):
        ctx.set_timing(True)
        rep = ctx.solve(loads, solver, tol=1e-9, maxit=500)
        t = ctx.kernel_times()
        ctx.set_timing(False)
        return rep["iterations"], {k: t[k] for k in names}

    P = np.eye(c)[[0, c - 1]] * np.array([[1.0], [2.0]])
    i0, t0 = run(P[:1])
    i1, t1 = run(P[1:])
    both, t = run(P)
    assert both == i0 + i1 and both[0] != both[1]
    for its, times in ((i0, t0), (i1, t1), (both, t)):
        assert times["xinv_f64"][1] == max(its) + 1   # and the residual of the result
    for k in names:
        # a load's first CG step reads fewer fields, so the shared first step is counted once a load too
        assert t[k][2] == pytest.approx(t0[k][2] + t1[k][2], rel=1e-12)
