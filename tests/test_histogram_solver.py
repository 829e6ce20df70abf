"""The kernels' histogram solver for general alpha, compiled for the host (tests/host/histogram_main.cpp): its
root and the bracket it promises against a float64 bisection, alpha from 1.001 to 1.999, up to 131072 counts."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_general_alpha_root_is_reached(tmp_path):
    exe = str(tmp_path / "histogram")
    res = subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_15180_amd", "csrc"),
                          os.path.join(ROOT, "tests", "host", "histogram_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout
