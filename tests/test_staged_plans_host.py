"""Index arithmetic of the FC kernels that stage their source through LDS, on the host: every workgroup number of plans up to the largest
tensors that they take, against plain division (tests/host/staged_plans.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2304_07741_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workgroup_numbers(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    B.load()
    libdir = os.path.dirname(B.LIB_PATH)
    exe = str(tmp_path / "staged_plans")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "host", "staged_plans.cpp"),
                    "-o", exe, f"-L{libdir}", "-lcanvas_dag", f"-Wl,-rpath,{libdir}", "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
    plans, slices, tiles, wrong = map(int, re.findall(r"\d+", p.stdout.splitlines()[-1]))
    assert plans > 1000 and slices > 50 and tiles > 1 << 17 and wrong == 0, p.stdout
