"""Wait states that the compiler does not insert, in the built code: a lane swap
(v_permlane16_swap, v_permlane32_swap) reads a register that a vector
instruction wrote fewer than two wait states before. The compiler keeps that
distance after its own instructions; it does not see that inline assembly
writes registers with vector instructions, so code built around such a block
has to."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2404_16208_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SWAP_WAIT_STATES = 2


def swaps_too_early(lines):
    """(kernel, writer, swap) of every swap that follows a vector write of one of
    its registers too closely (in program order; a label starts afresh)."""
    kernel, before, bad = "", [], []
    for line in lines:
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            kernel, before = head.group(1), []
            continue
        ins = line.split("//")[0].strip()
        if not ins:
            continue
        if re.match(r"v_permlane(16|32)_swap", ins):
            regs = set(re.findall(r"\bv\d+\b", ins))
            states = 0
            for earlier in reversed(before):
                if states >= SWAP_WAIT_STATES:
                    break
                if earlier.startswith("v_") and regs & set(re.findall(r"\bv\d+\b", earlier.split(",")[0])):
                    bad.append((kernel, earlier, ins))
                states += int(earlier.split()[1]) + 1 if earlier.startswith("s_nop") else 1
        before = (before + [ins])[-SWAP_WAIT_STATES:]
    return bad


def test_the_scan_finds_a_missing_wait():
    near = ["0 <k>:", "v_addc_co_u32_e32 v62, vcc, v62, v62, vcc", "s_nop 0", "v_permlane32_swap_b32_e32 v169, v62"]
    assert len(swaps_too_early(near)) == 1
    near[2] = "s_nop 1"
    assert not swaps_too_early(near)


def test_lane_swaps_wait_for_vector_writes(tmp_path):
    if not os.path.exists(OBJDUMP) or not os.path.exists(build.LIB):
        pytest.skip("needs llvm-objdump and the built library")
    lib = shutil.copy(build.LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objects = [str(tmp_path / f) for f in os.listdir(tmp_path) if f.endswith(build.ARCH)]
    assert objects
    swaps, bad = 0, []
    for obj in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        swaps += len(re.findall(r"\tv_permlane(?:16|32)_swap", text))
        bad += swaps_too_early(text.splitlines())
    assert swaps > 100
    assert not bad, f"{len(bad)} lane swaps too early, first: {bad[0]}"
