"""The table-driven exponential of the fp64 sweeps, compiled for the host, against libm's long-double exp."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pow_exp_matches_libm(tmp_path):
    """Half an ulp each for the table entry and for the last fma, and a little for what lies between: 1.3 measured."""
    exe = tmp_path / "pow_exp_check"
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-mfma", "-I", os.path.join(ROOT, "paper_2512_16273_amd", "csrc"),
                    "-o", str(exe), os.path.join(ROOT, "tests", "pow_exp_check.cpp")], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    m = re.search(r"max_ulp ([0-9.]+) edge (\d)", out)
    assert m and float(m.group(1)) < 1.5 and m.group(2) == "1", out
