"""Every FFT plan on the CPU in the tiles that the passes launch: lines and
threads come from the launchers' own tables (csrc/fft_tiles.hpp), for the row
passes, the convolution, the elevation passes and the 64-bit-addressing tile,
in both precisions; against a direct DFT, under the address sanitizer, with the
bounds of the existing plan test (2e-6 complex64, 1e-14 complex128 relative)."""
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
EMU = ROOT / "tests" / "host_emu"
CSRC = ROOT / "paper_2604_15796_amd" / "csrc"
OP_LENGTHS = [72, 80, 144, 160, 216, 288, 320, 432, 576, 640, 864]
ABI_LENGTHS = [32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024]

SOURCE = r"""
#define FWI_EMU_PART 99
#define main plans_main
#include "fft_plans.cpp"
#undef main
#include "fft_tiles.hpp"
template <typename T, int L, int V, bool LF = true>
void tile(const char* name) {
  if constexpr (LF) all_modes<T, L, col_nl<T, L, V>(), col_nt<V>(), true>(name);
  else all_modes<T, L, row_nl<T, L, V>(), fwi::NT, false>(name);
}
template <typename T, int L>
void op(const char* name) {  // one tile per pass; 0: 64-bit addressing
  constexpr int c = op_conv_variant<T>(L), s = op_strided_variant<T>(L);
  tile<T, L, 0, false>(name);
  tile<T, L, c>(name);
  if constexpr (s != c) tile<T, L, s>(name);
  if constexpr (c != 0 && s != 0) tile<T, L, 0>(name);
}
template <typename T, int L>
void abi(const char* name) {  // every variant
  tile<T, L, 0, false>(name);
  tile<T, L, 1, false>(name);
  tile<T, L, 0>(name);
  tile<T, L, 1>(name);
  tile<T, L, 2>(name);
}
template <int L> void one_op() { op<float, L>("float"); op<double, L>("double"); }
template <int L> void one_abi() { abi<float, L>("float"); abi<double, L>("double"); }
int main() { FWI_ALL }
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_plans_in_launched_tiles_on_host(tmp_path):
    calls = [f"one_op<{L}>();" for L in OP_LENGTHS] + [f"one_abi<{L}>();" for L in ABI_LENGTHS]
    builds, exes = [], []
    for k in range(6):
        src, exe = tmp_path / f"p{k}.cpp", tmp_path / f"p{k}"
        src.write_text(SOURCE.replace("FWI_ALL", " ".join(calls[k::6])))
        exes.append(exe)
        builds.append(subprocess.Popen(["g++", "-std=c++20", "-O1", "-fsanitize=address", f"-I{EMU}", f"-I{CSRC}",
                                        str(src), "-o", str(exe), "-lpthread"]))
    assert all(b.wait(timeout=900) == 0 for b in builds)
    runs = [subprocess.Popen([str(e)], stdout=subprocess.PIPE, text=True) for e in exes]
    lines = [l for r in runs for l in r.communicate(timeout=900)[0].splitlines() if l.strip()]
    assert all(r.returncode == 0 for r in runs)
    assert not [l for l in lines if not l.endswith(" ok")], "\n".join(lines)
    tiles = [tuple(l.replace("=", " ").split()[i] for i in (0, 2, 4, 6, 8)) for l in lines]  # type, L, NL, NT, LF
    assert len(tiles) == 10 * len(ABI_LENGTHS) + sum(t[1] in map(str, OP_LENGTHS) for t in tiles)
    # tiles that a list of numbers beside this test once missed
    for t in [("double", "144", "16", "512", "1"), ("double", "576", "4", "256", "1"), ("float", "576", "8", "512", "1"),
              ("float", "864", "8", "256", "1"), ("double", "640", "4", "512", "1")]:
        assert t in tiles, (t, tiles)
