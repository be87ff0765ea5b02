"""CPU: rounds whose updates come in chains and the tables of these chains (csrc/planner.cpp, chains_layout_check.cpp,
chains_table_check.cpp), and records of the strip kernel that request rows and use them at once (csrc/strips.cpp,
strips_holders_check.cpp), against the serial order."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("check", ["chains_layout_check", "chains_table_check", "strips_holders_check"])
def test_layouts_reproduce_the_serial_order(tmp_path, check):
    from paper_1710_06952_amd import build
    exe = str(tmp_path / "check")
    csrc = os.path.join(ROOT, "paper_1710_06952_amd", "csrc")
    subprocess.check_call([build.hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip",
                           os.path.join(HERE, check + ".cpp"), os.path.join(csrc, "planner.cpp"), os.path.join(csrc, "strips.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    sys.stdout.write(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("ok")
