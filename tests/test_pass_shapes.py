"""Launch shapes of the fused passes, computed on the CPU."""
import os
import subprocess

from paper_2609_07172_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shapes_fit_the_kernels_they_launch(tmp_path):
    exe = str(tmp_path / "pass_shapes")
    subprocess.run([build.hipcc(), "--cuda-host-only", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(build.PKG, "csrc"), "-o", exe, "-x", "hip",
                    os.path.join(ROOT, "tests", "pass_shapes_host.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr
