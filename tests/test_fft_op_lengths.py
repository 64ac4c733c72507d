"""The operator's FFT lengths between the powers of two and their 3/2 multiples
(72 ... 864): every plan on the CPU against a direct DFT, in the tile shapes the
passes use, and the operator on the GPU against the oracle at the smallest and
the largest grid of each length (2D lateral and depth axes, 3D elevation and
depth). Bounds of the existing plan and operator tests (2e-6 complex64, 1e-14
and 1e-13 complex128 relative)."""
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

from oracle import fwi_oracle as O
from paper_2604_15796_amd import workloads as W

ROOT = pathlib.Path(__file__).resolve().parents[1]
EMU = ROOT / "tests" / "host_emu"
CSRC = ROOT / "paper_2604_15796_amd" / "csrc"
LENGTHS = [72, 80, 144, 160, 216, 288, 320, 432, 576, 640, 864]

SOURCE = r"""
#define FWI_EMU_PART 99
#define main plans_main
#include "fft_plans.cpp"
#undef main
template <int L>
void one() {
  constexpr int R = 2048 / L;
  all_modes<float, L, R, 256, false>("float");        // rows
  all_modes<double, L, R, 256, false>("double");
  all_modes<float, L, 16, 256, true>("float");        // strided
  all_modes<float, L, L <= 576 ? 16 : 8, 512, true>("float");
  all_modes<double, L, L <= 288 ? 16 : L <= 576 ? 8 : 4, 256, true>("double");
  all_modes<double, L, 8, 512, true>("double");
}
int main() { FWI_ALL }
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_operator_length_plans_on_host(tmp_path):
    parts = [LENGTHS[k::4] for k in range(4)]
    builds, exes = [], []
    for k, ls in enumerate(parts):
        src, exe = tmp_path / f"p{k}.cpp", tmp_path / f"p{k}"
        src.write_text(SOURCE.replace("FWI_ALL", " ".join(f"one<{L}>();" for L in ls)))
        exes.append(exe)
        builds.append(subprocess.Popen(["g++", "-std=c++20", "-O1", "-fsanitize=address", f"-I{EMU}", f"-I{CSRC}",
                                        str(src), "-o", str(exe), "-lpthread"]))
    assert all(b.wait(timeout=900) == 0 for b in builds)
    runs = [subprocess.Popen([str(e)], stdout=subprocess.PIPE, text=True) for e in exes]
    lines = [l for r in runs for l in r.communicate(timeout=900)[0].splitlines() if l.strip()]
    assert all(r.returncode == 0 for r in runs) and len(lines) == 6 * len(LENGTHS)
    assert not [l for l in lines if not l.endswith(" ok")], "\n".join(lines)


@pytest.mark.gpu
@pytest.mark.parametrize("L", LENGTHS)
@pytest.mark.parametrize("case", ["2d", "3d"])
def test_operator_at_every_length_vs_oracle(L, case):
    import torch

    from paper_2604_15796_amd import fwi
    below = max([v for v in [32, 48, 64, 72, 80, 96, 128, 144, 160, 192, 216, 256, 288, 320, 384, 432, 512, 576, 640,
                             768, 864] if v < L])
    ctx = fwi.Context(0)
    try:
        for n in (below // 2 + 1, L // 2):
            # lateral and depth axis of a 2D grid; elevation and depth axis of a 3D one
            probs = [W.small2d(seed=n, nx=n, nz=11, nf=1), W.small2d(seed=n, nx=13, nz=n, nf=1)] if case == "2d" else \
                [W.small3d(seed=n, nx=9, ny=n, nz=7), W.small3d(seed=n, nx=18, ny=5, nz=n)]
            for p in probs:
                m = O.contrast(p.c, p.alpha, p.c0)
                x = W.random_complex(n, (3,) + p.shape)
                Gh = O.green_spectrum(O.wavenumber(p.freqs[0], p.c0), p.dim, p.nx, p.ny, p.nz, p.dx)
                ref = np.stack([O.vie_apply(Gh, m, x[b]).ravel() for b in range(3)])
                for wide in (False, True):  # 64-bit addressing form of the strided passes too
                    ctx.set_addressing(wide)
                    for prec in (0, 1):
                        dt = torch.complex64 if prec else torch.complex128
                        xd = torch.as_tensor(x.reshape(3, -1)).to(dt).to("cuda:0")
                        md = torch.as_tensor(m).to(torch.complex128).to("cuda:0")
                        y = ctx.apply_operator(p, md, [0, 0, 0], xd, precision=prec).cpu().numpy()
                        err = np.linalg.norm(y - ref, axis=1) / np.linalg.norm(ref, axis=1)
                        assert err.max() < (2e-6 if prec else 1e-13), (p.name, wide, prec, err)
    finally:
        ctx.close()
