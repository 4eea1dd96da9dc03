"""The plan of the several-sweeps launches, checked on the host through C++
programs linked with libj3d.so."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_check(tmp_path, name):
    pkg = os.path.join(ROOT, "paper_2202_11819_amd")
    exe = tmp_path / name
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(pkg, "csrc"), "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", name + ".cpp"), "-o", str(exe),
                           "-L", pkg, "-lj3d", f"-Wl,-rpath,{pkg}"])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout[-2000:]
    assert " 0 bad" in out.stdout


@pytest.mark.parametrize("name", ["cut_axis_check", "mshape_check", "dense_route_check",
                                  "launch_choice_check", "scratch_check"])
def test_host_check(tmp_path, name):
    run_check(tmp_path, name)
