"""Loads whose address starts at any word must not be promised to the compiler
as 16-byte aligned: rows of the boundary distances in the first products (they start
at a group's first boundary vertex) and blocks of the distance store in a query.
Read from the compiler's intermediate form; no GPU."""
import os
import re
import subprocess

import pytest

from paper_1503_07192_amd import build as B

# source and kernels that read no 16-byte aligned global memory at all
CASES = [("hier.hip", ["k_mp_statsILi0E", "k_mp_prodILi0E"]), ("kernels.hip", ["k_query"])]


@pytest.mark.parametrize("source,names", CASES)
def test_loads_promise_no_more_than_a_word(source, names, tmp_path):
    out = str(tmp_path / "kernel.ll")
    cmd = [c for c in B.command(out) if not c.endswith(".hip") and c != "-shared"]
    subprocess.run(cmd + ["--offload-device-only", "-S", "-emit-llvm", os.path.join(B.CSRC, source)],
                   check=True, capture_output=True)
    wide, kernel, seen = [], "", set()
    for line in open(out):
        m = re.match(r"define .*@(\w+)\(", line)
        if m:
            kernel = m.group(1)
        if any(n in kernel for n in names):
            seen.add(kernel)
            if re.search(r"= load .* ptr addrspace\(1\) .*align (16|32)", line):
                wide.append((kernel, line.strip()))
    assert len(seen) == len(names)
    assert not wide, wide[:3]
