"""Limit and shape of the on-chip row layout on the CPU: tests/cpp/
test_resident_limits.cpp and test_resident_shape.cpp, under AddressSanitizer
and UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("name", ["test_resident_limits", "test_resident_shape"])
def test_resident_layout_limits(tmp_path, name):
    exe = str(tmp_path / name)
    csrc = os.path.join(ROOT, "paper_2212_09642_amd", "csrc")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "cpp", name + ".cpp"),
                    os.path.join(csrc, "resident_layout.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
