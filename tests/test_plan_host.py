"""The backward's host side on the CPU (no GPU): plan_check.cpp compiles vpce_api.cpp with the
kernels replaced by recorders and checks what 600 random problems would launch."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("g++")


@pytest.mark.skipif(CXX is None, reason="no g++")
def test_backward_plans_cover_the_problem(tmp_path):
    exe = str(tmp_path / "plan_check")
    subprocess.run([CXX, "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O1", "-Wall",
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    os.path.join(HERE, "plan_check.cpp"), "-o", exe, "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib"], check=True)
    out = subprocess.run([exe, "3"], stdout=subprocess.PIPE, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    print(out.stdout)
