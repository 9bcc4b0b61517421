"""The grouped weight-gradient plans against the workspace laid out for them,
over widths, depths and token counts, on the host (tests/native/plan_check.cpp
replaces the launches with recorders)."""
import os
import shutil
import subprocess

import pytest

from paper_2609_28568_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_bias_rows_and_slices_fit_their_areas(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "plan_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    os.path.join(HERE, "native", "plan_check.cpp"), binding.LIB_PATH, f"-L{ROCM}/lib", "-lamdhip64",
                    f"-Wl,-rpath,{os.path.dirname(binding.LIB_PATH)}", f"-Wl,-rpath,{ROCM}/lib", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
