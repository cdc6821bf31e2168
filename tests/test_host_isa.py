"""What the compiler makes of the block kernels, where their speed hangs on it and no result shows it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_03644_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_restored_blocks_know_their_address_before_their_rows(tmp_path):
    # The address of a block inside one tensor comes by a scalar load: as a vector load it is issued among the rows,
    # done when they are, and the workgroup's barrier waits for it.
    asm = str(tmp_path / "blocks.s")
    subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-S", "-o", asm,
                                              os.path.join(build.CSRC, "blocks.hip")],
                   check=True, capture_output=True, text=True)
    loads, name = {}, None
    for line in open(asm):
        m = re.match(r"(_Z\S+):", line)
        if m:
            name = m.group(1)
        m = re.match(r"\s+(global_load_\w+|s_barrier)\b", line)
        if m and name:
            loads.setdefault(name, []).append(m.group(1))
    restores = [k for k in loads if re.search(r"block_kernel(_listed)?ILi1E|block_kernel_heldILi", k)]
    assert len(restores) == 8
    for k in restores:
        text = " ".join(loads[k])
        assert re.search("(^| )" + " ".join(["global_load_dwordx4"] * 8) + " s_barrier", text), k
