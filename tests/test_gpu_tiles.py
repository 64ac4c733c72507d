"""Complex128 strided passes on both sides of the sizes where their built-in tile
changes, against the oracle (bound of the operator tests, 1e-13), and the tuner
at a length that has one tile only."""
import numpy as np
import pytest
import torch

from oracle import fwi_oracle as O
from paper_2604_15796_amd import workloads as W

pytestmark = pytest.mark.gpu


# 16-column workgroups of the convolution, bound: 3 B, 800; 4 B, 800; 12 B, 256;
# 3D: 24 B of planes fewer than 8
@pytest.mark.parametrize("shape,batches", [((24, 24), (266, 267)), ((32, 32), (199, 200)), ((96, 96), (21, 22)),
                                           ((24, 20, 20), (7, 8))])
def test_operator_across_the_tile_bounds(shape, batches):
    from paper_2604_15796_amd import fwi
    p = W.small2d(seed=3, nx=shape[-1], nz=shape[0], ne=2, nf=1) if len(shape) == 2 else \
        W.small3d(seed=3, nx=shape[-1], ny=shape[1], nz=shape[0], ne=2)
    m = O.contrast(p.c, p.alpha, p.c0)
    Gh = O.green_spectrum(O.wavenumber(p.freqs[0], p.c0), p.dim, p.nx, p.ny, p.nz, p.dx)
    md = torch.as_tensor(m).to(torch.complex128).to("cuda:0")
    ctx = fwi.Context(0)
    try:
        for B in batches:
            x = W.random_complex(B, (B,) + p.shape)
            y = ctx.apply_operator(p, md, [0] * B, torch.as_tensor(x.reshape(B, -1)).to("cuda:0"), precision=0)
            y = y.cpu().numpy()
            for b in (0, B // 2, B - 1):
                ref = O.vie_apply(Gh, m, x[b]).ravel()
                assert np.linalg.norm(y[b] - ref) < 1e-13 * np.linalg.norm(ref), (B, b)
    finally:
        ctx.close()


def test_tuner_reports_the_built_in_tile_where_there_is_one():
    from paper_2604_15796_amd import fwi
    p = W.small2d(seed=3, nx=70, nz=75, ne=2, nf=1)  # lengths 144 and 160
    ctx = fwi.Context(0)
    try:
        for prec in (0, 1):
            for r in ctx.autotune(p, precision=prec, B=4, reps=1).values():
                assert r["chosen"] == r["default"], r
        assert all(v == 255 for v in ctx.get_tuning())  # no entries
    finally:
        ctx.close()
