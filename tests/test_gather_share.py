"""The HBM part of the launch that runs both gathers (csrc/launch_rules.hpp,
built with g++): its share of the grid follows the step's own lists, not those
of another step."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_share_follows_the_steps_own_lists(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path / "gather_share_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                           os.path.join(HERE, "native", "gather_share_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "wrong 0" in out.stdout
