"""The Jacobian products at the edges of their matrix-core tiles: element and
transmit counts around multiples of 16 and 64, grids around the split sizes,
against the oracle. Tolerance: FP64 sums of up to n = 4099 terms in another
order, error below n eps = 1e-12 of the largest output."""
import numpy as np
import pytest
import torch

from oracle import fwi_oracle as O
from paper_2604_15796_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_15796_amd import fwi
    c = fwi.Context(0)
    yield c
    c.close()


def _err(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).to(torch.complex128).to(DEV)


@pytest.mark.parametrize("nx,nz,ne,nt", [(5, 3, 1, 1), (9, 7, 15, 4), (64, 1, 16, 16), (13, 10, 17, 2), (41, 5, 33, 32),
                                         (16, 16, 48, 21), (31, 9, 49, 48), (4099 // 11, 11, 65, 64),
                                         (64, 64, 80, 17)])
def test_jacobian_products_at_tile_edges_vs_oracle(ctx, nx, nz, ne, nt):
    p = W.small2d(seed=nx + ne, nx=nx, nz=nz, ne=ne, nf=2)
    tx, rx = W.random_complex(1, (p.nf, nt, p.n)), W.random_complex(2, (p.nf, ne, p.n))
    a = W.random_complex(3, (p.n,))
    ref = O.jacobian_apply_tx(tx, rx, a, p.freqs, p.c0, p.dx, 2)
    assert _err(ctx.jacobian_apply_tx(p, _dev(tx), _dev(rx), _dev(a)).cpu().numpy(), ref) < 1e-12


@pytest.mark.parametrize("nx,nz,ne", [(5, 3, 1), (9, 7, 15), (64, 1, 16), (13, 10, 17), (41, 5, 33), (16, 16, 48),
                                      (31, 9, 49), (4099 // 11, 11, 64), (64, 64, 65), (30, 20, 130)])
def test_symmetric_jacobian_products_at_tile_edges_vs_oracle(ctx, nx, nz, ne):
    """Element transmits: transmit and receiver fields are one array, so the
    products run on the unordered pairs of element blocks."""
    p = W.small2d(seed=nx + ne, nx=nx, nz=nz, ne=ne, nf=2)
    f, a, b = W.random_complex(1, (p.nf, ne, p.n)), W.random_complex(3, (p.n,)), W.random_complex(4, (p.nf, ne, ne))
    ref = O.jacobian_apply(f, a, p.freqs, p.c0, p.dx, 2)
    assert _err(ctx.jacobian_apply(p, _dev(f), _dev(a)).cpu().numpy(), ref) < 1e-12
    k2 = np.array([O.wavenumber(q, p.c0) ** 2 for q in p.freqs])
    ref = p.dx ** 2 * sum(k2[l] * np.conj(np.sum(f[l] * (np.conj(b[l]) @ f[l]), axis=0)) for l in range(p.nf))
    assert _err(ctx.jacobian_adjoint_apply(p, _dev(f), _dev(b)).cpu().numpy(), ref) < 1e-12


@pytest.mark.parametrize("dim,shape,ne", [(2, (37, 50), 3), (2, (5, 200), 2), (2, (64, 33), 5), (3, (11, 9, 20), 3),
                                          (2, (130, 120), 60)])
@pytest.mark.parametrize("prec", [0, 1])
def test_solver_with_ragged_rows_vs_oracle(ctx, dim, shape, ne, prec):
    """Rows per right-hand side that do not fill the row passes' workgroups (or
    fewer than one), so that the last part of the inner products is ragged; and
    enough right-hand sides (60) that the coefficient sums are a kernel of their
    own. Field error bound: the solve's tolerance, 1e-10, times 100."""
    from paper_2604_15796_amd import fwi
    nx, nz = shape[-1], shape[0]
    p = W.small2d(seed=nx + nz, nx=nx, nz=nz, ne=ne, nf=1) if dim == 2 else \
        W.small3d(seed=nx + nz, nx=nx, ny=shape[1], nz=nz, ne=ne)
    args = (dim, p.nx, p.ny, p.nz, p.dx, p.c0, p.freqs, p.elems)
    tx = np.arange(ne) if ne < 10 else np.array([0, 31, 59])
    _, ref, _ = O.forward(p.c, p.alpha, *args, tx=tx)
    opts = fwi.SolveOptions(precision=prec, rtol=1e-10, restart=16)
    _, F, st = ctx.forward(p, torch.as_tensor(p.c).to(DEV), torch.as_tensor(p.alpha).to(DEV), opts, fields=True)
    got = F.cpu().numpy()[:, tx]
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert st["unconverged"] == 0 and err.max() < 1e-8


@pytest.mark.parametrize("nx,nz,ne,nf,nbytes", [(64, 64, 64, 8, 39152128), (24, 40, 64, 8, 10118144)])
def test_forward_in_a_small_caller_workspace(ctx, nx, nz, ne, nf, nbytes):
    """A workspace that has no room for the partial sums of every split (the
    sizes are the plans with one split per 1024 points) is accepted, and the
    data are those of the full plan up to the order of the sums (n eps)."""
    import ctypes as C
    from paper_2604_15796_amd import fwi as F
    p = W.small2d(seed=5, nx=nx, nz=nz, ne=ne, nf=nf)
    o = F.SolveOptions(precision=F.FWI_FP32_REFINE, rtol=1e-8, restart=8, max_rhs=64)
    prob, co = F.ProblemArgs(p), o.c()
    full = C.c_size_t()
    assert ctx.L.fwi_workspace_size(prob.ref(), C.byref(co), 0, C.byref(full)) == 0 and full.value > nbytes
    cc = torch.as_tensor(np.ascontiguousarray(p.c)).to(torch.float64).to(DEV).reshape(-1)
    out = []
    for size in (full.value, nbytes):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        d = torch.empty((nf, ne, ne), dtype=torch.complex128, device=DEV)
        assert ctx.L.fwi_set_workspace(ctx.h, C.c_void_p(ws.data_ptr()), size) == 0
        rc = ctx.L.fwi_forward(ctx.h, prob.ref(), C.c_void_p(cc.data_ptr()), None, C.byref(co),
                               C.c_void_p(d.data_ptr()), None, None)
        torch.cuda.synchronize()
        ctx.L.fwi_set_workspace(ctx.h, None, 0)
        assert rc == 0
        out.append(d.cpu().numpy())
    assert _err(out[1], out[0]) < 1e-12
