"""The packed word of the one-workgroup scan (csrc/scan_pack.h) on the CPU, under the
address and undefined-behaviour sanitizers: steps of 8192 counts that are all nonzero,
partly and hardly, sums up to its range (tests/native/scan_pack_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_packed_scan(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "scan_pack_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_1912_01491_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "scan_pack_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout + r.stderr
