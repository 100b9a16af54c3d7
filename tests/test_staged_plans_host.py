"""Plans of the FC kernels, on the host.  Of those that stage their source through LDS, the index arithmetic: every workgroup number of plans up to the
largest tensors that they take, against plain division (tests/host/staged_plans.cpp).  Of the weight gradient without a window: tiles that
read more than they must, and workgroups beyond the compute units (tests/host/wgrad_plans.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2304_07741_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, name):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    B.load()
    libdir = os.path.dirname(B.LIB_PATH)
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "host", name + ".cpp"),
                    "-o", exe, f"-L{libdir}", "-lcanvas_dag", f"-Wl,-rpath,{libdir}", "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
    return [int(v) for v in re.findall(r"\d+", p.stdout.splitlines()[-1])]


def test_workgroup_numbers(tmp_path):
    plans, slices, tiles, wrong = _run(tmp_path, "staged_plans")
    assert plans > 1000 and slices > 50 and tiles > 1 << 17 and wrong == 0


def test_weight_gradient_tiles(tmp_path):
    plans, wrong = _run(tmp_path, "wgrad_plans")
    assert plans > 5000 and wrong == 0
