"""What the kernels' tables are made of, compiled for the host."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tables_match_what_they_are_made_of(tmp_path):
    exe = tmp_path / "tables_check"
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-mfma", "-I", os.path.join(ROOT, "paper_2512_16273_amd", "csrc"),
                    "-o", str(exe), os.path.join(ROOT, "tests", "tables_check.cpp")], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    m = re.search(r"differ (\d+) max_ulp ([0-9.]+)", out)
    # one rounding at full size (half an ulp), a quarter for r, and a little for the series; exp64 itself: 0.9
    assert m and m.group(1) == "0" and float(m.group(2)) < 0.9, out
