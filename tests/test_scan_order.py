"""Single-pass scans that run at once (a context's rounds beside its sampling,
several contexts) never wait for blocks that they keep off the chip: the
library's rule for taking tiles (csrc/launch_rules.hpp), built with g++ and run
on a model of the chip's dispatch; and every scan of the sources takes its tile
by that rule."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2410_22697_amd", "csrc")


def test_mixes_of_scans_end(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path / "scan_order_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror",
                           os.path.join(HERE, "native", "scan_order_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "stuck 0 seen 1" in out.stdout


def test_every_scan_takes_its_tile_by_the_rule():
    text = ""
    for name in ("sample_kernels.hpp", "buffer_kernels.hpp"):
        with open(os.path.join(CSRC, name)) as f:
            text += re.sub(r"//[^\n]*", "", f.read())
    kernels = re.split(r"(?=__global__)", text)[1:]
    scans = [k for k in kernels if "lookback_exclusive(" in k or "fr_lookback<" in k]
    names = {re.search(r"void\s+(k_\w+)", k).group(1) for k in scans}
    assert names == {"k_seed_rows", "k_frontier", "k_round_evict", "k_rank_emit", "k_gsel_emit", "k_sort_scan"}
    for k in scans:
        name = re.search(r"void\s+(k_\w+)", k).group(1)
        assert "scan_tile<TICKETS>(" in k, name
        assert "blockIdx" not in k.split("\n}\n")[0], name + " uses its block index as a tile"
