"""CPU: the layout of a call as one persistent launch (csrc/strips.cpp) against the serial semantics: random schedules
with stale reads, carried and looked-ahead events, extra pairs, the wait-free variant, few slots and all numbers of
teams are executed entry by entry (strips_layout_check.cpp): every read sees exactly the updates before it, every update
finds its gradient, batches name a row once, rows are requested before they are used, slots are not given away."""
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
