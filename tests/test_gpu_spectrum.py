"""The Green spectrum call on ragged grids, where the operator pads its axes to
other lengths than the call's: values against the oracle with the bound of the
existing spectrum test, and no device memory taken, with the library's workspace
and with a caller's."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import fwi_oracle as O
from paper_2604_15796_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(37, 70), (130, 40), (150, 200), (40, 36, 30), (70, 20, 37)])
@pytest.mark.parametrize("caller", [False, True])
def test_spectrum_on_ragged_grids(shape, caller):
    from paper_2604_15796_amd import fwi
    nz, nx = shape[0], shape[-1]
    p = W.small2d(seed=1, nx=nx, nz=nz, ne=2, nf=2) if len(shape) == 2 else \
        W.small3d(seed=1, nx=nx, ny=shape[1], nz=nz, ne=2)
    ctx = fwi.Context(0)
    try:
        prob, l = fwi.ProblemArgs(p), p.nf - 1
        pad = [fwi.lib().fwi_padded_length(n) for n in (nz, p.ny if p.dim == 3 else 0, nx)]
        out = torch.empty([v for v in pad if v], dtype=torch.complex128, device="cuda:0")
        ws = torch.full((4096,), 7, dtype=torch.uint8, device="cuda:0")
        ctx.incident(p, 0)  # the problem's cache
        torch.cuda.synchronize()
        if caller:
            assert ctx.L.fwi_set_workspace(ctx.h, C.c_void_p(ws.data_ptr()), 4096) == 0
        free = torch.cuda.mem_get_info()[0]
        assert ctx.L.fwi_green_spectrum(ctx.h, prob.ref(), l, C.c_void_p(out.data_ptr())) == 0
        assert torch.cuda.mem_get_info()[0] == free and bool((ws == 7).all())
        # the table that the spectrum is of, offset by offset (-(n-1) .. n-1 per axis)
        got = np.fft.ifftn(out.cpu().numpy()) * out.numel()
        T = O.green_table(O.wavenumber(p.freqs[l], p.c0), p.dim, p.nx, p.ny, p.nz, p.dx)
        off = [np.arange(1 - n, n) for n in p.shape]
        ref = np.zeros_like(got)
        ref[np.ix_(*off)] = T[np.ix_(*off)]
        assert np.linalg.norm(got - ref) < 1e-13 * np.linalg.norm(ref)
        ctx.L.fwi_set_workspace(ctx.h, None, 0)
    finally:
        ctx.close()
