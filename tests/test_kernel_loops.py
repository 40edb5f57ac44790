"""What the compiler made of the staged BF16 kernels: their K loops move no accumulator between the two kinds of register.  Quads stored
straight from accumulation registers had the compiler keep half of the accumulators in each kind and move all of
them twice per K step (three moves per MFMA), which the sums' bits do not show.  Read from the library that was built here."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_20315_amd import _lib

TOOLS = "/opt/rocm/llvm/bin/"


def _innermost_mfma_loops(text):
    """(MFMAs, accumulator moves) of each innermost loop of one disassembled kernel that holds MFMAs."""
    ins = [(int(at, 16), op, line) for line in text.splitlines()[1:]
           for op, at in re.findall(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", line)]
    loops = []
    for at, op, line in ins:
        to = re.search(r"<.*\+0x([0-9a-f]+)>", line)
        if op.startswith(("s_cbranch", "s_branch")) and to and ins[0][0] + int(to.group(1), 16) <= at:
            loops.append((ins[0][0] + int(to.group(1), 16), at))
    inner = [a for a in loops if not any(b != a and a[0] <= b[0] and b[1] <= a[1] for b in loops)]
    bodies = [[op for at, op, _ in ins if lo <= at <= hi] for lo, hi in inner]
    counts = [(sum("mfma" in op for op in b), sum("accvgpr" in op for op in b)) for b in bodies]
    return [c for c in counts if c[0]]


@pytest.mark.skipif(not os.path.exists(TOOLS + "llvm-objdump"), reason="no disassembler")
def test_staged_bf16_loops_move_no_accumulators(tmp_path):
    lib = tmp_path / "lib.so"
    shutil.copy(_lib.LIB_PATH, lib)
    subprocess.run([TOOLS + "llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    seen = {}
    for part in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([TOOLS + "llvm-objdump", "-d", "--demangle", str(part)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            name = re.match(r"[0-9a-f]{16} <(?:void )?(?:mq::)?(?:\(anonymous namespace\)::)?(bf16_stage_kernel<.*?>)", kernel)
            if name:
                seen[name.group(1)] = _innermost_mfma_loops(kernel)
    assert len(seen) >= 32 and all(len(loops) == 1 for loops in seen.values()), seen
    assert not {n: c for n, c in seen.items() if c[0][1]}, "accumulator moves in a K loop (MFMAs, moves)"
