"""CPU: the layouts of calls that go in one launch (csrc/strips.cpp, pack_columns) against the serial semantics: random
schedules through the checks that ADPSGD_FLAG_VERIFY_PLAN runs (verify_strips, verify_columns), and planted mistakes that
these have to find (strips_layout_check.cpp)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_layouts_reproduce_the_serial_order(tmp_path):
    from paper_1710_06952_amd import build
    exe = str(tmp_path / "check")
    csrc = os.path.join(ROOT, "paper_1710_06952_amd", "csrc")
    subprocess.check_call([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip",
                           os.path.join(HERE, "strips_layout_check.cpp"), os.path.join(csrc, "planner.cpp"), os.path.join(csrc, "strips.cpp"),
                           "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    sys.stdout.write(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("ok")
