"""The bins of the truncation's sort, compiled for the host with the compiler's check of float-to-integer conversions."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_values_far_beyond_the_bins(tmp_path):
    exe = tmp_path / "bins_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=float-cast-overflow", "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2512_16273_amd", "csrc"), "-o", str(exe), os.path.join(ROOT, "tests", "bins_check.cpp")], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "wrong 0", r.stdout + r.stderr
