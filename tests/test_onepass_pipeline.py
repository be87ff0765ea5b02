"""CPU: the order of the exchange where two gradients of a group are in it at a time, and of the wavefronts of a block that leaves it
(csrc/onepass.hpp, kernels_onepass.hip, onepass_pipeline_check.cpp)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_two_gradients_in_the_exchange(tmp_path):
    from paper_1710_06952_amd import build
    exe = str(tmp_path / "check")
    csrc = os.path.join(ROOT, "paper_1710_06952_amd", "csrc")
    subprocess.check_call([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip",
                           os.path.join(HERE, "onepass_pipeline_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    sys.stdout.write(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("ok, ")
