"""The workloads whose speed is followed: the public entry points of the
package on the sizes its configurations, tests and benchmark use, from a
single small operator application to the 3D gradient.

listed() names the fixed cases, draw() makes more of the same ranges,
prepare() builds what a program has in hand before the call (context, problem,
device tensors, cached spectra), run() is one pass, work() the bytes and
operations a pass cannot do without, exact() the same outputs in plain
64-bit torch.

Solves run to a relative FP64 residual of 1e-11, so that the outputs are the
solution's and not the stopping point's, with the library's default inner
tolerance; the mixed form is the complex64 Krylov solve inside FP64 refinement.
"""
import math

import numpy as np
import torch

from paper_2604_15796_amd import fwi

C0 = 1540.0          # background speed of sound [m/s]
DX2, DX3 = 0.154e-3, 0.2e-3  # cell size [m], 2D and 3D
PITCH = 0.3e-3       # element pitch [m]
RHO, LAM, GAM, N_CG = 1e-2, 1e-3, 1e-5, 10  # ADMM weights and CG iterations
RTOL = 1e-11
MATVECS = 12         # operator applications that a solve to RTOL takes, about


def listed():
    return [
        # one operator application on the smallest grid: a caller's own Krylov loop
        dict(name="operator-64", kind="operator", nx=64, ny=1, nz=64, nf=1, batch=4, mixed=False),
        # the same on the 3D grid in complex64, a few right-hand sides
        dict(name="operator-3d", kind="operator", nx=128, ny=128, nz=96, nf=1, batch=8, mixed=True),
        # a new frequency list (frequency continuation): spectra and incident fields
        dict(name="setup-256", kind="setup", nx=256, ny=1, nz=256, nf=4, ne=64),
        # the smallest gradient: one frequency, plain FP64, latency counts
        dict(name="gradient-64", kind="gradient", nx=64, ny=1, nz=64, nf=1, ne=16, mixed=False, max_rhs=0),
        # forward and backward through automatic differentiation, ragged grid, odd element count
        dict(name="autograd-200x150", kind="autograd", nx=200, ny=1, nz=150, nf=3, ne=33, mixed=False),
        # the 2D gradient: every transmit of every frequency in one batch
        dict(name="gradient-256", kind="gradient", nx=256, ny=1, nz=256, nf=8, ne=64, mixed=True, max_rhs=0),
        # steered plane waves on a ragged grid, fewer transmits than elements
        dict(name="planewave-192x160", kind="planewave", nx=192, ny=1, nz=160, nf=5, ne=48, nt=21, mixed=True),
        # the largest 2D grid: forward data and complex64 fields
        dict(name="forward-512", kind="forward", nx=512, ny=1, nz=512, nf=2, ne=96, mixed=True),
        # Gauss-Newton products of an outer solver: J a and J^H b from stored fields
        dict(name="jacobian-256", kind="jacobian", nx=256, ny=1, nz=256, nf=8, ne=64),
        # one ADMM iteration of Algorithm 1 at full size
        dict(name="admm-384", kind="admm", nx=384, ny=1, nz=384, nf=12, ne=128, mixed=True, max_rhs=384),
        # a small ragged volume in plain FP64
        dict(name="gradient-40x36x30", kind="gradient", nx=40, ny=36, nz=30, nf=2, ne=8, mixed=False, max_rhs=0),
        # the 3D gradient, fields recomputed per frequency: the largest
        dict(name="gradient-3d", kind="gradient", nx=128, ny=128, nz=96, nf=4, ne=64, mixed=True, max_rhs=64),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    kind = rng.choice(["operator", "setup", "gradient", "autograd", "planewave", "forward", "jacobian", "admm"])
    mixed = rng.random() < 0.5
    volume = kind in ("operator", "gradient") and rng.random() < 0.4
    if volume:
        c = dict(kind=kind, nx=_log(rng, 24, 128), ny=_log(rng, 24, 128), nz=_log(rng, 20, 96))
    else:
        hi = dict(operator=512, setup=320, gradient=384, autograd=256, planewave=320, forward=512, jacobian=320,
                  admm=256)[kind]
        c = dict(kind=kind, nx=_log(rng, 40, hi), ny=1, nz=_log(rng, 40, hi))
    if kind == "operator":
        return dict(c, nf=rng.randint(1, 3), batch=_log(rng, 1, 16 if volume else 64), mixed=mixed)
    c["nf"] = rng.randint(1, 3 if volume else 6)
    c["ne"] = _log(rng, 5, 32 if volume else 96)
    while c["nf"] * c["ne"] * c["nx"] * c["ny"] * c["nz"] > 5e7:  # no more than the largest listed
        c["ne"] = 2 * c["ne"] // 3
    if kind == "planewave":
        c["nt"] = rng.randint(1, c["ne"])
    if kind not in ("setup", "jacobian"):
        c["mixed"] = mixed
    if kind in ("gradient", "admm"):
        c["max_rhs"] = c["ne"] if volume else rng.choice([0, 2 * c["ne"]])
    return c


# ------------------------------------------------------------------ inputs ---
class Problem:
    """Grid, array and frequencies, as the binding takes them."""

    def __init__(self, case, freqs=None):
        self.nx, self.ny, self.nz = case["nx"], case["ny"], case["nz"]
        self.dim = 2 if self.ny == 1 else 3
        self.dx, self.c0 = (DX2 if self.dim == 2 else DX3), C0
        self.n = self.nx * self.ny * self.nz
        self.shape = (self.nz, self.nx) if self.dim == 2 else (self.nz, self.ny, self.nx)
        lo, hi = (0.3e6, 1.0e6) if self.dim == 2 else (0.4e6, 0.8e6)
        self.freqs = np.linspace(lo, hi, case["nf"] + 1)[1:] if freqs is None else freqs
        ne, wx = case.get("ne", 1), self.nx * self.dx
        pitch = min(PITCH, 0.9 * wx / ne)
        x = wx / 2 + (np.arange(ne) - (ne - 1) / 2) * pitch
        y = np.full(ne, self.ny * self.dx / 2 if self.dim == 3 else 0.0)
        self.elems = np.stack([x, y, np.zeros(ne)], axis=1)


def _cells(p):
    """Cell-centre coordinates x, y, z, each [n]."""
    z, y, x = torch.meshgrid(*[(torch.arange(k, dtype=torch.float64) + 0.5) * p.dx for k in (p.nz, p.ny, p.nx)],
                             indexing="ij")
    return x.reshape(-1), y.reshape(-1) if p.dim == 3 else torch.zeros(p.n, dtype=torch.float64), z.reshape(-1)


def _phantom(p, rng):
    """Speed of sound [m/s] and attenuation [Np/m/Hz] of 2 to 5 soft-tissue
    inclusions (rotated ellipses or ellipsoids) with 0.5% speckle."""
    x, y, z = _cells(p)
    w = [p.nx * p.dx, p.ny * p.dx, p.nz * p.dx]
    c, a = torch.full((p.n,), C0, dtype=torch.float64), torch.zeros(p.n, dtype=torch.float64)
    for _ in range(int(rng.integers(2, 6))):
        semi = rng.uniform(0.05, 0.2, 3) * min(w[0], w[2])
        th, cs, al = rng.uniform(0, math.pi), rng.uniform(1480, 1600), rng.uniform(0, 0.5)
        cx, cy, cz = rng.uniform(0.1, 0.9) * w[0], rng.uniform(0.2, 0.8) * w[1], rng.uniform(0.15, 0.9) * w[2]
        u = (x - cx) * math.cos(th) + (z - cz) * math.sin(th)
        v = -(x - cx) * math.sin(th) + (z - cz) * math.cos(th)
        t = (y - cy) / semi[1] if p.dim == 3 else 0.0
        inside = (u / semi[0]) ** 2 + (v / semi[2]) ** 2 + t ** 2 <= 1
        c[inside], a[inside] = cs, al * 1e-4 * math.log(10.0) / 20.0  # dB/cm/MHz
    speckle = torch.from_numpy(rng.uniform(-0.005, 0.005, p.n))
    return c * (1 + speckle), a


def _contrast(c, a):
    return torch.complex(1 / c ** 2 - a ** 2 / (4 * math.pi ** 2), a / (math.pi * c)) * C0 ** 2 - 1


def _hankel0(x):
    """H0^(1) of real x > 0: the power series below 1, above it the integral
    of exp(-s^2) (1 + i s^2 / 2x)^(-1/2) over s by the trapezoidal rule, whose
    error falls like exp(-2 pi sqrt(x) / h)."""
    h, v = 0.15, x.clamp_min(1.0)
    acc = torch.full_like(v, 0.5, dtype=torch.complex128)
    for j in range(1, 43):
        s2 = (j * h) ** 2
        acc += math.exp(-s2) * torch.complex(torch.ones_like(v), 0.5 * s2 / v).rsqrt()
    big = torch.polar(2 * h * math.sqrt(2) / math.pi / v.sqrt(), v - math.pi / 4) * acc
    v = x.clamp_max(1.0)
    q, t, har = -v * v / 4, torch.ones_like(v), 0.0
    j0, tail = torch.ones_like(v), torch.zeros_like(v)
    for n in range(1, 12):
        t, har = t * q / n ** 2, har + 1 / n
        j0, tail = j0 + t, tail - har * t
    y0 = 2 / math.pi * ((torch.log(v / 2) + float(np.euler_gamma)) * j0 + tail)
    return torch.where(x < 1, torch.complex(j0, y0), big)


def _bessel1(x):
    """J1, Y1 of a small number, by their power series."""
    q, t, psi, j1, tail = -x * x / 4, 1.0, 1 - 2 * float(np.euler_gamma), 0.0, 0.0
    for n in range(14):
        j1, tail = j1 + t, tail + psi * t
        psi, t = psi + 1 / (n + 1) + 1 / (n + 2), t * q / ((n + 1) * (n + 2))
    j1 *= x / 2
    return j1, -2 / (math.pi * x) + 2 / math.pi * math.log(x / 2) * j1 - x / (2 * math.pi) * tail


def _green(k, r, dim):
    if dim == 2:
        return 0.25j * _hankel0(k * r)
    return torch.polar(1 / (4 * math.pi * r), k * r)


def _observed(p, rng, c, a, weights=None):
    """Scattered data [nf, nt, ne] of a medium near this one: the Born sum over
    a random subset of its cells, with 2% noise."""
    x, y, z = _cells(p)
    cells = torch.from_numpy(rng.choice(p.n, min(p.n, 512), replace=False))
    m = _contrast(c, a)[cells] * torch.from_numpy(rng.uniform(0.7, 1.3, len(cells)))
    e = torch.from_numpy(p.elems)
    r = torch.sqrt((x[cells] - e[:, :1]) ** 2 + (y[cells] - e[:, 1:2]) ** 2 + z[cells] ** 2)
    out = []
    for l, f in enumerate(p.freqs):
        k = 2 * math.pi * f / C0
        G = _green(k, r, p.dim)
        T = G if weights is None else weights[l] @ G
        out.append(k ** 2 * p.dx ** p.dim * p.n / len(cells) * (T * m) @ G.T)
    d = torch.stack(out)
    noise = torch.view_as_complex(torch.from_numpy(rng.standard_normal((*d.shape, 2))))
    return d + 0.02 * d.abs().square().mean().sqrt() / math.sqrt(2) * noise


def _plane_waves(p, nt):
    """Element weights [nf, nt, ne] of nt plane waves steered over -60 to 60 degrees."""
    x = torch.from_numpy(p.elems[:, 0] - p.elems[:, 0].mean())
    s = torch.sin(torch.linspace(-math.pi / 3, math.pi / 3, nt, dtype=torch.float64)) if nt > 1 else torch.zeros(1).double()
    k = 2 * math.pi * torch.from_numpy(np.asarray(p.freqs)) / C0
    ph = k[:, None, None] * s[None, :, None] * x[None, None, :]
    return torch.polar(torch.ones_like(ph), ph)


def _inputs(case, seed):
    """Everything a pass takes, on the CPU, from the seed alone."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "setup":  # two stages of a frequency continuation
        lo = rng.uniform(0.25e6, 0.35e6)
        return dict(problems=[Problem(case, np.linspace(a * lo, 3 * a * lo, case["nf"] + 1)[1:]) for a in (1.0, 1.3)])
    p = Problem(case)
    s = dict(problem=p)
    c, a = _phantom(p, rng)
    if kind in ("gradient", "planewave", "forward"):
        s.update(c=c.reshape(p.shape), a=a.reshape(p.shape))
    else:
        s["m"] = _contrast(c, a).reshape(p.shape)
    if kind == "operator":
        x = torch.view_as_complex(torch.from_numpy(rng.standard_normal((case["batch"], p.n, 2))))
        s["x"] = x.to(torch.complex64 if case["mixed"] else torch.complex128)
        s["fi"] = [int(v) for v in np.sort(rng.integers(0, case["nf"], case["batch"]))]
    if kind == "planewave":
        s["w"] = _plane_waves(p, case["nt"])
    if kind in ("gradient", "planewave", "autograd", "admm"):
        s["d"] = _observed(p, rng, c, a, s.get("w"))
    if kind == "jacobian":  # fields of point sources seen through a random medium
        x, y, z = _cells(p)
        amp = 1 + 0.1 * torch.from_numpy(rng.standard_normal(p.n))
        e = torch.from_numpy(p.elems)
        r = torch.sqrt((x - e[:, :1]) ** 2 + z ** 2)
        s["fields"] = torch.stack([torch.polar(amp / torch.sqrt(8 * math.pi * k * r), k * r)
                                   for k in 2 * math.pi * np.asarray(p.freqs) / C0])
        s["b"] = torch.view_as_complex(torch.from_numpy(rng.standard_normal((case["nf"], case["ne"], case["ne"], 2))))
    if kind == "admm":  # a started inversion: the iterate is half way to the medium
        s["m"] = 0.5 * s["m"]
        s["g"] = torch.stack(_diff(s["m"]))
        s["u"] = 1e-2 * s["g"]
    return s


def _diff(m):
    """Forward differences along x and z, zero at the last index."""
    dx, dz = torch.zeros_like(m), torch.zeros_like(m)
    dx[:, :-1], dz[:-1] = m[:, 1:] - m[:, :-1], m[1:] - m[:-1]
    return [dx, dz]


def prepare(case, seed):
    ctx = fwi.Context(0)
    s = {k: v.to(ctx.device) if isinstance(v, torch.Tensor) else v for k, v in _inputs(case, seed).items()}
    s.update(kind=case["kind"], ctx=ctx)
    if case["kind"] == "setup":
        s["problems"] = [fwi.ProblemArgs(p) for p in s["problems"]]
        return s
    s["problem"] = fwi.ProblemArgs(s["problem"])
    restart = 16 if case["ny"] > 1 or case["kind"] == "admm" else 32  # basis memory of the largest cases
    s["opts"] = fwi.SolveOptions(precision=fwi.FWI_FP32_REFINE if case.get("mixed") else fwi.FWI_FP64, rtol=RTOL, restart=restart,
                                 max_rhs=case.get("max_rhs", 0), fields_c64=1 if case["kind"] == "forward" else 0)
    ctx.green_spectrum(s["problem"], 0)  # spectra and incident fields of this problem, kept in the context
    return s


def run(s):
    ctx, kind = s["ctx"], s["kind"]
    if kind == "setup":
        return [[ctx.incident(p, p.nf - 1), ctx.green_spectrum(p, 0)] for p in s["problems"]]
    p, o = s["problem"], s["opts"]
    if kind == "operator":
        return ctx.apply_operator(p, s["m"], s["fi"], s["x"], precision=o.precision)
    if kind == "gradient":
        return list(ctx.adjoint_gradient(p, s["c"], s["a"], s["d"], o)[:4])
    if kind == "planewave":
        return list(ctx.adjoint_gradient_tx(p, s["c"], s["a"], s["w"], s["d"], o)[:4])
    if kind == "forward":
        return list(ctx.forward(p, s["c"], s["a"], o, fields=True)[:2])
    if kind == "jacobian":
        return [ctx.jacobian_apply(p, s["fields"], s["m"]), ctx.jacobian_adjoint_apply(p, s["fields"], s["b"])]
    if kind == "autograd":
        m = s["m"].clone().requires_grad_(True)
        d = fwi.fwi_data(m, ctx, p, o)
        d.backward(d.detach() - s["d"])
        return [d.detach(), m.grad]
    m, g, u = s["m"].clone(), s["g"].clone(), s["u"].clone()
    rep, _ = ctx.tv_admm_step(p, m, g, u, s["d"], LAM, RHO, GAM, N_CG, m_ref=s["m"], opts=o)
    return [m, g, u, rep["misfit"], rep["tv"], rep["dm_norm"]]


def work(case):
    p, kind = Problem(case), case["kind"]
    n, nf, ne = p.n, case["nf"], case.get("ne", 0)
    pad = [1 << (2 * k - 1).bit_length() for k in p.shape]
    N = math.prod(pad)
    apply = 2 * 5 * N * math.log2(N) + 14 * n + 6 * N  # two transforms, contrast, spectrum product, difference
    nt = case.get("nt", ne)
    sample = 8 * nf * nt * ne * n  # one complex contraction of fields with element fields
    if kind == "operator":
        es = 8 if case["mixed"] else 16
        return dict(bytes=2 * case["batch"] * n * es + 16 * n + nf * N * es, flops=case["batch"] * apply)
    if kind == "setup":
        return dict(bytes=2 * nf * (N + ne * n) * 16, flops=2 * nf * (5 * N * math.log2(N) + 60 * (N + ne * n)))
    if kind == "jacobian":
        return dict(bytes=2 * nf * ne * n * 16 + 32 * n + 32 * nf * ne * ne, flops=2 * sample)
    solve = nf * nt * MATVECS * apply
    if kind == "forward":
        return dict(bytes=16 * n + 8 * nf * nt * n + 16 * nf * ne * n + 16 * nf * nt * ne, flops=solve + sample)
    if kind == "admm":
        return dict(bytes=16 * n * 11 + 16 * nf * ne * n + 16 * nf * ne * ne,
                    flops=solve + sample + (2 * N_CG + 1) * sample)
    return dict(bytes=64 * n + 16 * nf * ne * n + 16 * nf * nt * ne, flops=2 * solve + 2 * sample)


# -------------------------------------------------- the outputs in 64 bits ---
def _padded(n):
    return min(2 ** a * 3 ** b for a in range(5, 11) for b in range(0, 2) if 2 * n <= 2 ** a * 3 ** b) if n > 24 else \
        min(L for L in (32, 48) if L >= 2 * n)


def _spectrum(k, p, lengths):
    """FFT of k^2 times the integral of the Green's function over a cell (the
    disk of equal area, the ball of equal volume), on the circulant grid."""
    off, use = [], []
    for n, L in zip(p.shape, lengths):
        i = torch.arange(L)
        d = torch.where(i < L // 2 + (L % 2), i, i - L)
        off.append(d.double())
        use.append(d.abs() < n)
    sq = sum(o.reshape([-1 if j == q else 1 for j in range(p.dim)]) ** 2 for q, o in enumerate(off))
    ok = math.prod([u.reshape([-1 if j == q else 1 for j in range(p.dim)]).double() for q, u in enumerate(use)])
    r = (p.dx * torch.sqrt(sq)).to(_DEV)
    zero = (0,) * p.dim
    r[zero] = 1.0
    if p.dim == 2:
        a = p.dx / math.sqrt(math.pi)
        j1, y1 = _bessel1(k * a)
        W = (2 * math.pi * a / k) * j1 * _green(k, r, 2)
        W[zero] = complex(1j * math.pi * a / (2 * k) * complex(j1, y1) - 1 / k ** 2)
    else:
        a = p.dx * (3 / (4 * math.pi)) ** (1 / 3)
        ka = k * a
        W = 4 * math.pi / k ** 3 * (math.sin(ka) - ka * math.cos(ka)) * _green(k, r, 3)
        W[zero] = ((1 - 1j * ka) * complex(math.cos(ka), math.sin(ka)) - 1) / k ** 2
    return torch.fft.fftn(k ** 2 * W * ok.to(_DEV))


_DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _apply(G, m, x, p):
    """x - k^2 sum W m x for x [B, n]."""
    d = tuple(range(1, 1 + p.dim))
    y = torch.fft.ifftn(torch.fft.fftn((m * x).reshape(-1, *p.shape), s=G.shape, dim=d) * G, dim=d)
    return x - y[(slice(None),) + tuple(slice(0, k) for k in p.shape)].reshape(x.shape)


def _solve(G, m, b, p, steps=16):
    """Restarted GMRES for every row of b, to a residual near 1e-14."""
    if len(b) > 64:
        return torch.cat([_solve(G, m, q, p, steps) for q in b.split(64)])
    x = b.clone()
    norm = lambda v: torch.linalg.vector_norm(v, dim=1)
    for _ in range(6):
        r = b - _apply(G, m, x, p)
        beta = norm(r)
        if float((beta / norm(b)).max()) < 2e-14:
            break
        V = [r / beta.clamp_min(1e-300)[:, None]]
        H = torch.zeros(len(b), steps + 1, steps, dtype=torch.complex128, device=b.device)
        for j in range(steps):
            w = _apply(G, m, V[j], p)
            for i in range(j + 1):
                H[:, i, j] = (V[i].conj() * w).sum(1)
                w = w - H[:, i, j, None] * V[i]
            h = norm(w)
            H[:, j + 1, j] = h
            V.append(w / h.clamp_min(1e-300)[:, None])
        e = torch.zeros(len(b), steps + 1, 1, dtype=torch.complex128)
        e[:, 0, 0] = beta.cpu()
        y = (torch.linalg.pinv(H.cpu(), rtol=1e-13) @ e).to(b.device)
        for j in range(steps):
            x = x + y[:, j] * V[j]
    return x


def exact(case, seed):
    kind = case["kind"]
    lengths = [_padded(k) for k in ((case["nz"], case["nx"]) if case["ny"] == 1 else (case["nz"], case["ny"], case["nx"]))]
    rows = case["nf"] * case.get("nt", case.get("ne", 0))
    cost = rows * math.prod(lengths) * dict(gradient=2, planewave=2, autograd=2, admm=2).get(kind, 1)
    if kind not in ("operator", "setup", "jacobian") and cost > 2.5e9:
        return None  # minutes
    s = {k: v.to(_DEV) if isinstance(v, torch.Tensor) else v for k, v in _inputs(case, seed).items()}

    def fields0(p, k):
        x, y, z = _cells(p)
        e = torch.from_numpy(p.elems)
        r = torch.sqrt((x - e[:, :1]) ** 2 + (y - e[:, 1:2]) ** 2 + z ** 2).to(_DEV)
        return torch.cat([_green(k, q, p.dim) for q in r.split(16)])

    wave = lambda f: float(2 * math.pi * f / C0)
    if kind == "setup":
        return [[fields0(p, wave(p.freqs[-1])), _spectrum(wave(p.freqs[0]), p, lengths) / math.prod(lengths)]
                for p in s["problems"]]
    p = s["problem"]
    ks, dV = [wave(f) for f in p.freqs], p.dx ** p.dim
    if kind in ("gradient", "planewave", "forward"):
        c, a = s["c"].reshape(-1), s["a"].reshape(-1)
        m = _contrast(c, a)
    else:
        m = s["m"].reshape(-1)
    if kind == "operator":
        Gs = [_spectrum(k, p, lengths) for k in ks]
        return torch.cat([_apply(Gs[f], m, s["x"][b:b + 1].to(torch.complex128), p) for b, f in enumerate(s["fi"])])
    J = lambda F, v: torch.stack([k ** 2 * dV * (F[l] * v) @ F[l].T for l, k in enumerate(ks)])
    JH = lambda F, b: sum(k ** 2 * dV * (F[l] * (b[l].conj() @ F[l])).sum(0).conj() for l, k in enumerate(ks))
    if kind == "jacobian":
        return [J(s["fields"], m), JH(s["fields"], s["b"])]
    Gs = [_spectrum(k, p, lengths) for k in ks]
    P0 = [fields0(p, k) for k in ks]
    src = [s["w"][l] @ P0[l] for l in range(len(ks))] if kind == "planewave" else P0
    F = [_solve(Gs[l], m, src[l], p) for l in range(len(ks))]
    d = torch.stack([k ** 2 * dV * (F[l] * m) @ P0[l].T for l, k in enumerate(ks)])
    if kind == "forward":
        return [d, torch.stack(F)]
    r = d - s["d"]
    if kind != "admm":
        g = torch.zeros_like(m)
        for l, k in enumerate(ks):
            lam = _solve(Gs[l], m, r[l].conj() @ P0[l], p)
            g += dV * k ** 2 * (F[l] * lam).sum(0).conj()
        if kind == "autograd":
            return [d, g.reshape(p.shape)]
        dc = torch.complex(-2 / c ** 3, -a / (math.pi * c ** 2)) * C0 ** 2
        da = torch.complex(-2 * a / (4 * math.pi ** 2), 1 / (math.pi * c)) * C0 ** 2
        return [0.5 * float(r.abs().square().sum()), g, (g.conj() * dc).real, (g.conj() * da).real]
    # one ADMM iteration, the Gauss-Newton system by N_CG steps of CG
    grad = lambda v: torch.stack(_diff(v))

    def grad_t(v):
        out = torch.zeros_like(v[0])
        out[:, 1:] += v[0][:, :-1]
        out[:, :-1] -= v[0][:, :-1]
        out[1:] += v[1][:-1]
        out[:-1] -= v[1][:-1]
        return out

    dot = lambda v, w: float((v.conj() * w).sum().real)
    m0, g, u, sc = m.reshape(p.shape), s["g"], s["u"], 1 / float(s["d"].abs().square().sum())
    A = lambda v: sc * JH(F, J(F, v.reshape(-1))).reshape(p.shape) + RHO * grad_t(grad(v)) + GAM * v
    b = -sc * JH(F, r).reshape(p.shape) + RHO * grad_t(g + u - grad(m0))
    x, res, q = torch.zeros_like(b), b, b
    rs = dot(b, b)
    for _ in range(N_CG):
        Aq = A(q)
        al = rs / dot(q, Aq)
        x, res = x + al * q, res - al * Aq
        new = dot(res, res)
        q, rs = res + new / rs * q, new
    m1 = m0 + x
    gm = grad(m1)
    w = gm - u
    nw = w.abs().square().sum(0).sqrt()
    g1 = (1 - LAM / RHO / nw.clamp_min(1e-300)).clamp_min(0) * w
    return [m1, g1, u + RHO * (g1 - gm), 0.5 * float(r.abs().square().sum()),
            float(gm.abs().square().sum(0).sqrt().sum()), math.sqrt(dot(x, x))]
