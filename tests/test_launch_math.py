"""The launch arithmetic shared by kernels and host code, checked by brute force on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_math(tmp_path):
    exe = str(tmp_path / "launch_math")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                            "-I", os.path.join(ROOT, "include"),
                            "-I", os.path.join(ROOT, "paper_2505_14022_amd", "csrc"),
                            os.path.join(ROOT, "tests", "launch_math.cpp"), "-o", exe],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "failures: 0" in run.stdout, run.stdout[-2000:]


# The macros that arrange the gather kernels' work in another way (microbench/ablation.py), and the product.
ARRANGEMENTS = ["product", "NO_XCD_REMAP", "HEAD_FASTEST", "SLAB_RANGES", "QUERY_EIGHTHS", "INDEX_EIGHTHS"]


@pytest.mark.parametrize("variant", ARRANGEMENTS)
def test_gather_work_is_done_once(tmp_path, variant):
    exe = str(tmp_path / "gather_work")
    macro = [] if variant == "product" else [f"-DMSDA_ABLATE_{variant}=1"]
    csrc = os.path.join(ROOT, "paper_2505_14022_amd", "csrc")
    build = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include"] + macro +
                           ["-I", os.path.join(ROOT, "include"), "-I", csrc,
                            os.path.join(ROOT, "tests", "gather_work.cpp"), os.path.join(csrc, "msda_arrange.cpp"),
                            "-o", exe], capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "failures: 0" in run.stdout, run.stdout[-2000:]
