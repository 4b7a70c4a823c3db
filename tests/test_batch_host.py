"""The batch's host code without a GPU: what a lane's lost stream costs."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_07172_amd", "csrc")


def test_a_lost_stream_loses_its_own_answers_only(tmp_path):
    """The problems that a failed wait covers are reported, with the failure's
    text; every other lane's problems keep their status."""
    exe = str(tmp_path / "batch_lanes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-o", exe, "-x", "c++",
                    os.path.join(CSRC, "batch.hip"), os.path.join(ROOT, "tests", "batch_lanes_host.cpp"),
                    "-pthread"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr[-4000:]
