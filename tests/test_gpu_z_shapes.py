"""Tile shapes of the z pass with the stored operator: the operator against the
oracle for every length along z that has a shape of its own, on rows of 8 to 40
wave-vectors (a whole line of pencils, half a line, and a remainder).  Tolerances as for the operator elsewhere: 1e-12 in FP64,
1e-5 in FP32."""
import numpy as np
import pytest

from oracle import operator as op
from paper_1411_0330_amd import inputs as I

from .gpu_util import context, problem, rel_max_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [8, 16, 32, 48, 64, 80, 96, 128, 160, 192])
@pytest.mark.parametrize("ny,nx", [(2, 16), (2, 32), (4, 48), (2, 80)])
@pytest.mark.parametrize("physics,dtype", [("scalar", "f64"), ("scalar", "f32"), ("elastic", "f64"), ("elastic", "f32")])
def test_z_shapes_match_oracle(lsh, nz, ny, nx, physics, dtype):
    shape = (nz, ny, nx)
    if physics == "elastic":
        moduli = np.stack([I.elastic_from_young(1.0, 0.3), I.elastic_from_young(10.0, 0.2)])
        A0 = I.elastic_from_young(0.5, 0.3)
    else:
        moduli = np.stack([I.scalar_isotropic(1.0, 3), I.scalar_isotropic(10.0, 3)])
        A0 = I.scalar_isotropic(0.5, 3)
    ph = I.random_phases(shape, 2, seed=3)
    ctx = context(lsh, ph, moduli, A0, physics, "filtered", "mixed" if dtype == "f32" else "fp64", 2)
    pb = problem(ph, moduli, A0, physics, "filtered")
    tau = I.random_field(shape, pb.c, 2, seed=7) * op.mask(pb)
    out = ctx.apply(to_dev(tau, dtype)).cpu().numpy()
    for l in range(2):
        assert rel_max_err(out[l], op.apply(pb, tau[l])) <= (1e-12 if dtype == "f64" else 1e-5)
