"""Limit of the on-chip row layout on the CPU: tests/cpp/
test_resident_limits.cpp, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_word_rows_stay_within_32_bit_offsets(tmp_path):
    exe = str(tmp_path / "test_resident_limits")
    csrc = os.path.join(ROOT, "paper_2212_09642_amd", "csrc")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "cpp", "test_resident_limits.cpp"),
                    os.path.join(csrc, "resident_layout.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
