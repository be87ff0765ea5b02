"""CPU: every shape that is accepted for the linear gradients in one pass has a kernel, on any number of compute units
(csrc/onepass.cpp, onepass_shape_check.cpp)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_accepted_shapes_are_built(tmp_path):
    from paper_1710_06952_amd import build
    exe = str(tmp_path / "check")
    csrc = os.path.join(ROOT, "paper_1710_06952_amd", "csrc")
    subprocess.check_call([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip",
                           os.path.join(HERE, "onepass_shape_check.cpp"), os.path.join(csrc, "onepass.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    sys.stdout.write(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("ok, ")
