"""Registers of kernels that the compiler makes for gfx950: those that have come to spill where nothing needed it."""
import os
import re
import subprocess

import pytest

from paper_2512_16273_amd import build

FORMS = ["tree_node_kernel<float, PowTerms<float>, kShared>(const TreeParams)",
         "verify_resample_kernel<float, PowTerms<float>, kShared>(const VerifyParams)"]


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("form", FORMS)
def test_fp32_rows_two_to_a_compute_unit_do_not_spill(tmp_path, form):
    """Each row's workgroup has 64 registers a thread; what is asked for early is held in them through all that comes before the sweep."""
    src, asm = tmp_path / "form.hip", tmp_path / "form.s"
    src.write_text('#include "tree.h"\n#include "verify.h"\nnamespace tslt {\ntemplate __global__ void %s;\n}\n' % form)
    flags = [f for f in build.hipcc_command()[1:] if f not in ("-fPIC", "-shared") and not f.endswith((".hip", ".so")) and f != "-o"]
    subprocess.run([build.hipcc_command()[0], *flags, "--cuda-device-only", "-S", "-o", str(asm), str(src)], check=True, stderr=subprocess.DEVNULL)
    name = form.split("<")[0]
    made = [k for k in asm.read_text().split(".agpr_count")[1:] if re.search(r"\.symbol:\s+\S*" + name, k)]
    assert len(made) == 1 and re.search(r"\.vgpr_spill_count:\s+(\d+)", made[0]).group(1) == "0"
