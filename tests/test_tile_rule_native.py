"""The default tiles (csrc/tile_rule.h) on the CPU, for M up to 46340, every padded
number of states, both precisions and one to many systems: tiles and slabs that the
kernels are compiled for, slabs that do not depend on the number of systems, the
allocation-free call's limit and the row thresholds (tests/native/tile_rule_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_default_tiles(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "tile_rule_check")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_1912_01491_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "tile_rule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and ", 0 bad" in r.stdout, r.stdout + r.stderr
