"""The in-tile kernel's waits count loads: while one of the first stages is waited for, the bias and residual loads behind it may
stay in flight, and they are taken to be as many as the kernel asks for (NI + ME * NI).  Here they are counted in the library as built."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2407_02031_amd", "libswiftdiff.so")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def test_bias_and_residual_loads_are_as_many_as_the_waits_count(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(LIB):
        from paper_2407_02031_amd import build
        build.build(verbose=False)
    shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", "libswiftdiff.so"], cwd=tmp_path, check=True, capture_output=True)
    seen = 0
    for obj in sorted(tmp_path.glob("libswiftdiff.so.*gfx950")):
        if b"gemm16_kernel" not in obj.read_bytes():
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--demangle", str(obj)], check=True, capture_output=True, text=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <.*gemm16_kernel<([\d, ]+)>.*>:\n((?:.+\n)*)", text, re.M):
            BM, BN, WGM, WGN, WGK, _, RES, _ = map(int, m.group(1).split(","))
            NI, ME = BN // WGN // 16, BM // WGM // 16 // WGK
            ops = [line.split("//")[0].strip() for line in m.group(2).splitlines()]
            loads = [i for i, op in enumerate(ops) if op.startswith("global_load") and "_lds_" not in op]
            assert len(loads) == NI + (ME * NI if RES else 0), m.group(1)
            # all of them between the first stage's barrier and the next wait
            assert sum(op.startswith("s_barrier") for op in ops[:loads[0]]) == 1, m.group(1)
            assert not any(op.startswith("s_barrier") or "vmcnt" in op for op in ops[loads[0]:loads[-1]]), m.group(1)
            assert not any(op.startswith(("flat_load", "buffer_load")) for op in ops), m.group(1)
            seen += 1
    assert seen >= 30
