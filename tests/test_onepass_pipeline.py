"""CPU: the order of the exchange where two gradients of a group are in it at a time (onepass_pipeline_check.cpp)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))


def test_two_gradients_in_the_exchange(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", os.path.join(HERE, "onepass_pipeline_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    sys.stdout.write(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("ok, ")
