"""What the compiler makes of the kernels, where their speed hangs on it and no result shows it."""
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


@pytest.fixture(scope="module")
def step_asm(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("needs hipcc")
    asm = str(tmp_path_factory.mktemp("step") / "fused.s")
    subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-S", "-o", asm,
                                              os.path.join(build.CSRC, "fused.hip")],
                   check=True, capture_output=True, text=True)
    return asm


@pytest.fixture(scope="module")
def step_registers(step_asm):
    used, name = {}, None
    for line in open(step_asm):
        m = re.match(r"\s+\.amdhsa_(kernel|next_free_vgpr|private_segment_fixed_size) (\S+)", line)
        if m and m.group(1) == "kernel":
            name = m.group(2)
        elif m:
            used.setdefault(name, {})[m.group(1)] = int(m.group(2))
    return used


def test_long_chained_steps_leave_room_for_seven_wavefronts_on_a_simd(step_registers):
    # 512 registers a SIMD, handed out in eights: 72 for seven wavefronts, none of them in scratch memory.
    # <F16, CHAINED, BC2, N, TALLY>
    bf16 = {k: v for k, v in step_registers.items() if re.search(r"fused_kernelILb0ELb1ELb[01]ELj\d+ELb0EE", k)}
    assert len(bf16) == 6
    for k, v in bf16.items():
        assert v["next_free_vgpr"] <= 72 and v["private_segment_fixed_size"] == 0, (k, v)


def test_steps_keep_nothing_in_scratch_memory(step_registers):
    # six wavefronts on a SIMD, short steps and long ones, both halves
    steps = {k: v for k, v in step_registers.items() if re.search(r"fused_kernel(_warm)?ILb[01]E", k)}
    assert sum("fused_kernel_warm" in k for k in steps) == 24 and len(steps) == 60
    for k, v in steps.items():
        assert v["next_free_vgpr"] <= 80 and v["private_segment_fixed_size"] == 0, (k, v)


def test_short_steps_load_through_the_caches(step_asm):
    # what a short step reads, its tensors that are only copied included, is in the last-level cache or would be by the next step
    nt, name = {}, None
    for line in open(step_asm):
        m = re.match(r"(_Z\S+):", line)
        if m:
            name = m.group(1)
        m = re.match(r"\s+(global|flat|buffer)_load_\w+", line)
        if m and name:
            nt.setdefault(name, []).append(bool(re.search(r"\bnt\b", line)))
    warm = [k for k in nt if "fused_kernel_warm" in k]
    long = [k for k in nt if re.search(r"fused_kernelILb", k)]
    assert len(warm) == 24 and len(long) == 36
    for k in warm:
        assert not any(nt[k]), k
    for k in long:
        assert any(nt[k]), k
