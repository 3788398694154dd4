"""The launch arithmetic shared by kernels and host code, checked by brute force on the CPU."""
import os
import subprocess

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
