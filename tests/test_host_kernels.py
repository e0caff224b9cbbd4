"""The solver kernels' own source, run on the CPU block by block (tests/host/
block_emu.hpp), for what a run on the GPU shows only by chance or not at all."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="clang not available")
@pytest.mark.parametrize("name", ["inner_stop", "rho_updates", "rho_stencil"])
def test_kernels_on_the_host(tmp_path, name):
    exe = tmp_path / name
    # (the launch functions of the sources are compiled with the kernels but never called)
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROCM, "include"),
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1709_08785_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", str(exe),
           "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
