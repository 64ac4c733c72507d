"""Single conditions of the library's host code on the CPU: capi.cpp with the
stand-ins of tests/host_capi/ (see test_capi_host_emulation.py), under the
address and undefined-behaviour sanitizers. Each name is a function of
tests/host_capi/paths.cpp."""
import os
import pathlib
import shutil
import subprocess

import pytest

ROOT = pathlib.Path(__file__).resolve().parents[1]
HOST = ROOT / "tests" / "host_capi"
CSRC = ROOT / "paper_2604_15796_amd" / "csrc"
SOURCES = [CSRC / "capi.cpp", HOST / "emu_runtime.cpp", HOST / "stub_kernels.cpp", HOST / "paths.cpp"]


@pytest.fixture(scope="module")
def paths(tmp_path_factory):
    probe = subprocess.run(["g++", "-fsanitize=address", "-x", "c++", "-", "-o", os.devnull],
                           input="int main(){return 0;}", capture_output=True, text=True) if shutil.which("g++") else None
    if probe is None or probe.returncode != 0:
        pytest.skip("g++ with the address sanitizer not available")
    out = tmp_path_factory.mktemp("paths")
    flags = ["-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
             "-fno-sanitize-recover=undefined", "-DFWI_WORKSPACE_GUARD", f"-I{HOST}", f"-I{ROOT / 'include'}",
             f"-I{CSRC}"]
    procs = [subprocess.Popen(["g++", *flags, "-c", str(s), "-o", str(out / (s.stem + ".o"))], stderr=subprocess.PIPE,
                              text=True) for s in SOURCES]
    for p in procs:
        _, err = p.communicate(timeout=900)
        assert p.returncode == 0, err
    exe = out / "paths"
    subprocess.run(["g++", "-fsanitize=address,undefined", *[str(out / (s.stem + ".o")) for s in SOURCES], "-o",
                    str(exe)], check=True, timeout=300)
    return exe


@pytest.mark.parametrize("name,checks", [("spectrum", 4), ("launches", 6), ("tiles", 4), ("splits", 8),
                                         ("batch", 3), ("sums", 6)])
def test_host_path(paths, name, checks):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    p = subprocess.run([str(paths), name], capture_output=True, text=True, timeout=600, env=env)
    text = p.stdout + p.stderr
    assert p.returncode == 0 and "AddressSanitizer" not in text and "runtime error" not in text, text[-6000:]
    assert text.count("ok ") == checks and "FAILED" not in text, text
