"""Solves in the regimes of the Krylov step that differ in kernels, against the
oracle: coefficient sums in the orthogonalising pass, as a kernel of their own
(many right-hand sides, many parts, a tuned row tile) over ragged parts, and
fewer rows per right-hand side than a workgroup of the row pass has. The host
test of the same shapes (test_capi_host_paths.py, "sums") asserts which kernels
each one launches. Field error bound: the solve's tolerance, 1e-10, times 100."""
import numpy as np
import pytest
import torch

from oracle import fwi_oracle as O
from paper_2604_15796_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# shape (z .. x), elements, frequencies, padded x length, tuned row tile, sums fused, dots fused
CASES = [((70, 37), 5, 2, 80, False, True, True), ((50, 64), 5, 2, 128, True, False, True),
         ((210, 20, 16), 2, 1, 32, False, False, True), ((130, 120), 61, 4, 256, False, False, True),
         ((13, 20), 3, 1, 48, False, True, False)]


@pytest.mark.parametrize("shape,ne,nf,Lx,tuned,sums,dots", CASES)
@pytest.mark.parametrize("prec", [0, 1])
def test_solve_in_every_regime_vs_oracle(shape, ne, nf, Lx, tuned, sums, dots, prec):
    from paper_2604_15796_amd import fwi
    nz, nx = shape[0], shape[-1]
    p = W.small2d(seed=nx + nz, nx=nx, nz=nz, ne=ne, nf=nf) if len(shape) == 2 else \
        W.small3d(seed=nx + nz, nx=nx, ny=shape[1], nz=nz, ne=ne, nf=nf)
    # the regime: rows and parts of the built-in tile, its bounds
    rows, nl = p.n // nx, 2048 // Lx
    parts = -(-rows // nl)
    assert dots == (rows >= nl)
    assert sums == (not tuned and parts <= 64 and parts * ne * nf <= 4096)
    assert tuned or parts * nl != rows  # ragged
    ctx = fwi.Context(0)
    try:
        if tuned:
            table = bytearray([255] * fwi.TUNING_BYTES)
            table[0:22] = bytes([1] * 22)  # row pass, both precisions, every length
            ctx.set_tuning(bytes(table))
        tx = np.arange(ne) if ne < 10 else np.array([0, 31, ne - 1])
        _, ref, _ = O.forward(p.c, p.alpha, p.dim, p.nx, p.ny, p.nz, p.dx, p.c0, p.freqs, p.elems, tx=tx)
        opts = fwi.SolveOptions(precision=prec, rtol=1e-10, restart=16)
        ctx.profile(["dots_c64", "dots_c128"])
        _, F, st = ctx.forward(p, torch.as_tensor(p.c).to(DEV), torch.as_tensor(p.alpha).to(DEV), opts, fields=True)
        assert bool(ctx.profile_read()) == (not dots)
        err = np.linalg.norm(F.cpu().numpy()[:, tx] - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
        assert st["unconverged"] == 0 and err.max() < 1e-8
    finally:
        ctx.close()
