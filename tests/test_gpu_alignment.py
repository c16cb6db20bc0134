"""Tensors that do not start on 16 bytes: plane passes and row blocks need them
to, so the operator takes the passes in registers for such a field, in the
direction it belongs to.  Against the oracle, with the elements around the
output untouched."""
import ctypes as C

import numpy as np
import pytest

from oracle import operator as op
from paper_1411_0330_amd import inputs as I

from .gpu_util import rel_max_err
from .test_gpu_plane import _ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau_off,out_off", [(1, 0), (0, 1), (1, 1), (3, 2)])
@pytest.mark.parametrize("shape", [(4, 16, 16), (2, 48, 80), (4, 4, 256), (2, 32, 192)])
@pytest.mark.parametrize("physics,dtype,medium", [("scalar", "f64", "voxel"), ("scalar", "f32", "phases"),
                                                  ("elastic", "f64", "phases"), ("elastic", "f32", "voxel")])
def test_unaligned_fields_match_oracle(lsh, shape, physics, dtype, medium, tau_off, out_off):
    import torch
    ctx, pb = _ctx(lsh, physics, shape, "mixed" if dtype == "f32" else "fp64", 2, medium=medium)
    tau = I.random_field(shape, pb.c, 2, seed=7) * op.mask(pb)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    n = tau.size
    src = torch.full((n + 8,), 7.0, dtype=tdt, device="cuda:0")
    out = torch.full((n + 8,), -3.0, dtype=tdt, device="cuda:0")
    a, b = src[tau_off:tau_off + n], out[out_off:out_off + n]
    a.copy_(torch.from_numpy(tau).to(tdt).reshape(-1))
    size = a.element_size()
    assert src.data_ptr() % 16 == 0 and a.data_ptr() == src.data_ptr() + tau_off * size
    torch.cuda.synchronize()
    ctx._check(ctx.lib.lsh_apply(ctx.h, 2, C.c_void_p(a.data_ptr()), C.c_void_p(b.data_ptr()),
                                 lsh.F64 if dtype == "f64" else lsh.F32))
    tol = 1e-12 if dtype == "f64" else 1e-5
    got = b.cpu().numpy().reshape(tau.shape)
    for l in range(2):
        assert rel_max_err(got[l], op.apply(pb, tau[l])) <= tol
    assert torch.all(out[:out_off] == -3.0) and torch.all(out[out_off + n:] == -3.0)
    assert torch.equal(a.cpu(), torch.from_numpy(tau).to(tdt).reshape(-1))
    # the forward transform alone, from a field of the same alignment
    main, nyq = ctx.forward_dft(a.view(tau.shape))
    ref = np.fft.fftn(tau, axes=(-3, -2, -1))
    mx = shape[-1] // 2
    assert rel_max_err(main.cpu().numpy(), ref[..., :mx]) <= tol
    assert rel_max_err(nyq.cpu().numpy(), ref[..., mx]) <= tol
