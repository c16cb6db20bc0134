"""The separate x, y and z passes in registers where plane passes and row blocks
would take their place (LSH_PLANE=0): full-matrix phases, the fixed-point
schemes, unaligned tensors and larger planes still run them.  The operator
against the oracle on every row and column length, and every compiled kernel
shape of the 128- and 256-point passes."""
import numpy as np
import pytest

from oracle import operator as op
from paper_1411_0330_amd import inputs as I

from . import test_gpu_transform_operator as transform_operator
from .gpu_util import rel_max_err, to_dev
from .test_gpu_plane import _ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def separate(monkeypatch):
    monkeypatch.setenv("LSH_PLANE", "0")


@pytest.mark.parametrize("shape", [(2, 1024, 4), (2, 512, 8), (2, 256, 16), (4, 192, 32), (2, 160, 48), (8, 128, 64),
                                   (2, 96, 80), (2, 80, 96), (16, 64, 128), (4, 48, 160), (2, 32, 192), (2, 16, 256),
                                   (2, 8, 512), (4, 4, 1024), (8, 2, 64)])
@pytest.mark.parametrize("physics,dtype,medium", [("scalar", "f64", "phases"), ("scalar", "f32", "voxel"),
                                                  ("elastic", "f32", "phases"), ("elastic", "f64", "voxel")])
def test_separate_passes_match_oracle(lsh, shape, physics, dtype, medium):
    ctx, pb = _ctx(lsh, physics, shape, "mixed" if dtype == "f32" else "fp64", 2, medium=medium)
    tau = I.random_field(shape, pb.c, 2, seed=7) * op.mask(pb)
    ctx.set_timing(True)
    out = ctx.apply(to_dev(tau, dtype)).cpu().numpy()
    assert ctx.kernel_times()["y_" + dtype][1] == 2   # y forward and inverse, passes of their own
    for l in range(2):
        assert rel_max_err(out[l], op.apply(pb, tau[l])) <= (1e-12 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("variant", [1, 2, 3])
@pytest.mark.parametrize("physics,shape", [("scalar", (128, 8, 128)), ("scalar", (4, 128, 256)),
                                           ("elastic", (256, 4, 128)), ("elastic", (8, 256, 256))])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_kernel_shape_variants_of_the_separate_passes(lsh, monkeypatch, physics, shape, variant, dtype):
    transform_operator.test_operator_kernel_shape_variants(lsh, monkeypatch, physics, shape, variant, dtype)
