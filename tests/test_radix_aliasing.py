"""The radix scatter's 16-bit digit counts may alias the words they lie in.

Lanes clear the counts as 32-bit words and count in 16 bits between barriers of the wave,
which order no memory for the compiler: with a type of its own for the 16-bit accesses it
may move one past the other. Compiles radix.hip (this repository's code only) to LLVM IR
and checks the alias class of every 16-bit LDS access.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2107_05681_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


def test_digit_counts_may_alias_words(tmp_path):
    out = tmp_path / "radix.ll"
    subprocess.check_call(
        [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", "--offload-device-only", "-S",
         "-emit-llvm", os.path.join(CSRC, "radix.hip"), "-o", str(out)],
        stderr=subprocess.DEVNULL)
    ir = out.read_text()
    nodes = dict(re.findall(r"^!(\d+) = (.*)$", ir, flags=re.M))
    lines = [ln for ln in ir.splitlines()
             if re.search(r"\b(load i16|store i16)\b.*addrspace\(3\)", ln)]
    assert lines
    for ln in lines:
        tag = re.search(r"!tbaa !(\d+)", ln)
        if tag is None:
            continue  # no class: may alias anything
        access = re.match(r"!\{!(\d+), ", nodes[tag.group(1)]).group(1)
        assert "omnipotent char" in nodes[access], (ln, nodes[access])
