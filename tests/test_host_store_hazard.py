"""gfx950 wants two wait states between a store of more than 64 bits and an instruction that
writes the store's data registers again.  The compiler adds them behind stores of its own, but
not behind one that stands in inline assembly, so every such block has to end with them:
otherwise a change of the code around it could put other bytes into the store.  Read from the
assembly that the compiler makes of the kernels."""
import os
import re
import subprocess

import pytest

from paper_2510_09665_amd import build as B


def test_wide_stores_in_inline_assembly_are_followed_by_two_wait_states(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = str(tmp_path / "kernels.s")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc] + flags + ["--cuda-device-only", "-S", os.path.join(B.CSRC, "lmc_kernels.hip"), "-o", out],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    with open(out) as f:
        blocks = re.findall(r";;#ASMSTART\n(.*?);;#ASMEND", f.read(), re.S)
    stores = 0
    for block in blocks:
        lines = [l.strip() for l in block.splitlines() if l.strip()]
        for i, line in enumerate(lines):
            if not re.match(r"(global|flat|buffer|scratch)_store_dwordx[34]\b", line):
                continue
            stores += 1
            # "s_nop n" is n + 1 wait states
            waits = sum(int(l.split()[1]) + 1 for l in lines[i + 1:] if l.startswith("s_nop"))
            assert waits >= 2, block
    assert stores > 0                # the kernels have such stores: the search still finds them
