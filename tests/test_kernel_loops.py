"""What the compiler made of some kernels, read from the library that was built here; the results' bits do not show it.  The K loops of
the staged BF16 kernels move no accumulator between the two kinds of register (quads stored straight from accumulation registers had the
compiler keep half of them in each kind and move all of them twice per K step).  The direct NVFP4 kernels (K whole or in halves) start on
their first K step without a wait for the second one's loads.  The conversion exists with non-temporal
loads and stores, stores alone and neither."""
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


def _kernels(tmp_path, part_of_name):
    """{name: disassembly} of the library's kernels with this in their names."""
    if not os.path.exists(TOOLS + "llvm-objdump"):
        pytest.skip("no disassembler")
    lib = tmp_path / "lib.so"
    shutil.copy(_lib.LIB_PATH, lib)
    subprocess.run([TOOLS + "llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    found = {}
    for part in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([TOOLS + "llvm-objdump", "-d", "--demangle", str(part)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            name = re.match(r"[0-9a-f]{16} <.*?(" + part_of_name + r"<.*?>)\(", kernel)
            if name:
                found[name.group(1)] = kernel
    return found


def test_staged_bf16_loops_move_no_accumulators(tmp_path):
    seen = {name: _innermost_mfma_loops(text) for name, text in _kernels(tmp_path, "bf16_stage_kernel").items()}
    # eight tiles in both output types, and with K slabs all but 256x192, which no long K reaches
    assert len(seen) == 23 and all(len(loops) == 1 for loops in seen.values()), seen
    assert not [n for n in seen if n.startswith("bf16_stage_kernel<8, 6,") and ", true, false>" in n]
    assert not {n: c for n, c in seen.items() if c[0][1]}, "accumulator moves in a K loop (MFMAs, moves)"


def test_direct_fp4_starts_with_the_second_k_step_in_flight(tmp_path):
    kernels = _kernels(tmp_path, "gemm_fp4_direct")
    assert len(kernels) == 6
    for name, text in kernels.items():
        if name.endswith(", 4>"):  # a wave has a quarter of K: faster with both steps' loads mixed
            continue
        before = text[:text.index("v_mfma")]
        after_loads = before[before.rindex("buffer_load"):]
        waits = [int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\)", after_loads)]
        assert before.count("buffer_load") == 32 and min(waits, default=16) >= 16, (name, waits)


def test_conversion_past_the_cache_only_where_it_pays(tmp_path):
    kernels = _kernels(tmp_path, "relayout_kernel")
    streamed = {name: (len(re.findall(r"global_load_dwordx4.* nt", text)), len(re.findall(r"global_store_dwordx4.* nt", text)))
                for name, text in kernels.items()}
    assert streamed == {f"relayout_kernel<{to}, {i}, {o}>": (4 * (i == "true"), 4 * (o == "true"))
                        for to in ("true", "false") for i, o in (("true", "true"), ("false", "true"), ("false", "false"))}
