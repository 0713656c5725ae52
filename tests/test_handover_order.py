"""The order in which a workgroup's results leave it, read off the code that the compiler makes for gfx950."""
import os
import re
import subprocess

import pytest

from paper_2512_16273_amd import build

FORMS = [f"{t}, {terms}<{t}>, {waves}" for t, terms in (("float", "PowTerms"), ("F16", "PowTerms"), ("Bf16", "PowTerms"), ("Bf16", "BitTerms"))
         for waves in ("kAlone", "kShared", "kAlone, true")]
SOURCE = """#include "tree.h"
namespace tslt {
template __global__ void tree_node_kernel<%s>(const TreeParams);
}
"""


def instructions(text):
    """[(instruction, indices of those that may follow it)]"""
    lines, labels = [], {}
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:", line):
            labels[line[:-1]] = len(lines)
        elif line and line[0] != "." and not line.endswith(":"):
            lines.append(line)
    out = []
    for i, line in enumerate(lines):
        branch = re.match(r"s_(c?)branch\S*\s+(\.LBB\w+)", line)
        after = [] if line.startswith("s_endpgm") else [i + 1]
        if branch:
            after = [labels[branch.group(2)]] + ([i + 1] if branch.group(1) else [])
        out.append((line, [j for j in after if j < len(lines)]))
    return out


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("form", FORMS)
def test_ratios_arrive_before_the_words_of_a_node(tmp_path, form):
    """A path's candidates: their ratios go to memory before the node's words are stored, on every way through the kernel.  Whoever
    finds the words writes NaN over the ratios of nodes that are not on the path."""
    src, asm = tmp_path / "node.hip", tmp_path / "node.s"
    src.write_text(SOURCE % form)
    flags = [f for f in build.hipcc_command()[1:] if f not in ("-fPIC", "-shared") and not f.endswith((".hip", ".so")) and f != "-o"]
    subprocess.run([build.hipcc_command()[0], *flags, "--cuda-device-only", "-S", "-o", str(asm), str(src)], check=True, stderr=subprocess.DEVNULL)
    code = instructions(asm.read_text())
    ratios = [i for i, (line, _) in enumerate(code) if re.match(r"global_store_dword\s.*\bsc1\b", line)]
    words = {i for i, (line, _) in enumerate(code) if re.match(r"global_store_dwordx2\s.*\bsc1\b", line)}
    assert len(ratios) >= 2 and len(words) >= 2                  # the ratio and the rate; the two words
    seen, todo = set(), [j for i in ratios for j in code[i][1]]
    while todo:
        i = todo.pop()
        if i in seen:
            continue
        seen.add(i)
        assert i not in words, "a word can be stored while a ratio is on its way"
        if not re.match(r"s_waitcnt\b.*vmcnt\(0\)", code[i][0]):
            todo += code[i][1]
    assert seen
