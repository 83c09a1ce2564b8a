"""Waits that count loads, looked at in the library as built.  In the in-tile kernel: while one of the first stages is waited for, the bias and residual
loads behind it may stay in flight, and they are taken to be as many as the kernel asks for (NI + ME * NI).  In the tiles of few rows they count nowhere."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2407_02031_amd", "libswiftdiff.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def kernels(tmp_path, name):
    """(template arguments, instructions) of every instance of a kernel in the library as built"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(LIB):
        from paper_2407_02031_amd import build
        build.build(verbose=False)
    shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", "libswiftdiff.so"], cwd=tmp_path, check=True, capture_output=True)
    for obj in sorted(tmp_path.glob("libswiftdiff.so.*gfx950")):
        if name.encode() not in obj.read_bytes():
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--demangle", str(obj)], check=True, capture_output=True, text=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <.*" + name + r"<([\d, ]+)>.*>:\n((?:.+\n)*)", text, re.M):
            yield tuple(map(int, m.group(1).split(","))), [line.split("//")[0].strip() for line in m.group(2).splitlines()]


def test_bias_and_residual_loads_are_as_many_as_the_waits_count(tmp_path):
    seen = 0
    for args, ops in kernels(tmp_path, "gemm16_kernel"):
        BM, BN, WGM, WGN, WGK, _, RES, _ = args
        NI, ME = BN // WGN // 16, BM // WGM // 16 // WGK
        loads = [i for i, op in enumerate(ops) if op.startswith("global_load") and "_lds_" not in op]
        assert len(loads) == NI + (ME * NI if RES else 0), args
        # all of them between the first stage's barrier and the next wait
        assert sum(op.startswith("s_barrier") for op in ops[:loads[0]]) == 1, args
        assert not any(op.startswith("s_barrier") or "vmcnt" in op for op in ops[loads[0]:loads[-1]]), args
        assert not any(op.startswith(("flat_load", "buffer_load")) for op in ops), args
        seen += 1
    assert seen >= 30


def test_few_row_tiles_count_on_no_load_of_the_compiler(tmp_path):
    """Up to the end of the K loop (the first barrier) they wait for all loads, or for all but a slice's."""
    seen = 0
    for args, ops in kernels(tmp_path, "gemm_thin_kernel"):
        BM, BN, RT, _ = args
        loop = ops[:next(i for i, op in enumerate(ops) if op.startswith("s_barrier"))]
        waits = {int(m.group(1)) for op in loop if (m := re.search(r"vmcnt\((\d+)\)", op))}
        assert waits <= {0, (BM + BN + 16 * RT) // 8}, args
        # ... which are in flight behind the wait; the epilogue's, ahead of them, in front of the loop
        loads = [i for i, op in enumerate(ops) if op.startswith("global_load") and "_lds_" not in op]
        assert loads[-1] < next(i for i, op in enumerate(ops) if "vmcnt" in op), args
        seen += 1
    assert seen >= 30
