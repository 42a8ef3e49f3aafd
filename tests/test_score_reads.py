"""Where a round's select pass reads its 16-byte vectors of scores
(csrc/launch_rules.hpp), built with g++: inside the array's allocation also
where the halo (or the global id space) has fewer than four entries."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_vectors_stay_inside_the_allocation(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path / "score_reads_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                           os.path.join(HERE, "native", "score_reads_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "past 0 wrong 0" in out.stdout
