"""Where a step's long rows run, on the CPU: tests/cpp/test_long_rows.cpp,
under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_long_rows_first(tmp_path):
    exe = str(tmp_path / "test_long_rows")
    csrc = os.path.join(ROOT, "paper_2212_09642_amd", "csrc")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "cpp", "test_long_rows.cpp"),
                    os.path.join(csrc, "host_graph.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
