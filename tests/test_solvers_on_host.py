"""The conjugate residual solvers' kernels, compiled for the CPU with a stand-in for the HIP runtime
(tests/simt): the order in which wavefronts and workgroups run can be chosen there, so that decisions
that must not depend on it can be tested; and any operator can take the place of H."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang")
@pytest.mark.parametrize("name,opt", [("cr", "-O1"), ("coarse_cr", "-O0")])
def test_solver_on_host(name, opt, tmp_path):
    exe = tmp_path / name
    cmd = [CLANG, "-x", "c++", "-std=c++17", opt, "-Wno-unknown-attributes", "-I" + os.path.join(ROOT, "tests", "simt"),
           "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "simt", name + "_main.cpp"), "-o", str(exe),
           "-lpthread"]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and f"{name} ok" in r.stdout, r.stdout + r.stderr
