"""Registers of the orthogonalising row pass, from the compiler's resource
report: the kind that reads its coefficients runs on full batches and with every
row tile, so it must not pay for the kind that sums them (short launches). With
both in one kernel the bounds below were missed: 5 waves per SIMD instead of 8
and 7, one instead of two, and 148 bytes of scratch per lane in the largest
complex128 tile."""
import pathlib
import re
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2604_15796_amd" / "csrc"
HIPCC = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if pathlib.Path("/opt/rocm/bin/hipcc").exists() else None)
# type, length, rows per workgroup, kind, least waves per SIMD
KERNELS = [("float", 256, 8, "RI_ORTH_ONLY", 8), ("float", 48, 42, "RI_ORTH", 7), ("float", 256, 32, "RI_ORTH", 2),
           ("double", 384, 10, "RI_ORTH", 2), ("double", 192, 42, "RI_ORTH", 1)]


@pytest.mark.skipif(HIPCC is None, reason="hipcc not available")
def test_orthogonalising_row_pass_keeps_its_registers(tmp_path):
    src = tmp_path / "row.hip"
    src.write_text('#include "fft_passes.hpp"\nnamespace fwi {\n' + "".join(
        f"template __global__ void k_row_fwd<{t}, {L}, {nl}, true, {k}>(RowFwdArgs<{t}>);\n"
        for t, L, nl, k, _ in KERNELS) + "}\n")
    p = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", f"-I{ROOT / 'include'}", f"-I{CSRC}", "--cuda-device-only", "-c", str(src),
                        "-o", str(tmp_path / "row.o"), "-Rpass-analysis=kernel-resource-usage"],
                       capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stderr[-3000:]
    seen = {}
    for line in p.stderr.splitlines():
        m = re.search(r"remark: .*?(Function Name|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\S+)", line)
        if m and m[1] == "Function Name":
            cur = seen.setdefault(re.search(r"k_row_fwdI([fd])Li(\d+)ELi(\d+)", m[2]).groups(), {})
        elif m:
            cur[m[1].split()[0]] = int(m[2])
    for t, L, nl, kind, waves in KERNELS:
        r = seen[(t[0], str(L), str(nl))]
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= waves, (t, L, nl, kind, r)
