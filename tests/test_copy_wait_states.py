"""Wait states of the hand-written global -> LDS copies (no GPU needed).

A copy into LDS takes its LDS address from m0, and gfx9 needs one wait state
between a scalar write of m0 and the copy.  The compiler inserts it for its own
instructions, not inside the assembly blocks of gemm.hip and attention.hip, so
this test reads the built library's own gfx950 code and checks every copy.  It
also checks that no vector instruction writes a copy's scalar base address in
the five wait states before it.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_2411_06465_amd as L

LLVM = "/opt/rocm/llvm/bin"
VALU_SGPR_TO_VMEM = 5          # wait states between a vector write of a scalar register and its use by a memory access

pytestmark = pytest.mark.skipif(not os.path.exists(L.LIB_PATH) or not os.path.exists(f"{LLVM}/llvm-objdump"),
                                reason="libl4d.so not built, or no llvm-objdump")


def scalar_registers(token):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", token)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def hazards(listing):
    """(copies, messages) of a disassembly: instructions as text lines, kernels headed by <name>:."""
    copies, found, kernel, before = 0, [], "", []
    for line in listing.splitlines():
        head = re.search(r"<(.*)>:$", line)
        if head:
            kernel, before = head[1], []
            continue
        ins = line.split("//")[0].replace(",", " ").split()
        if not ins or not ins[0].startswith(("s_", "v_", "ds_", "global_", "buffer_", "flat_", "scratch_")):
            continue
        if "_load_lds" in ins[0]:
            copies += 1
            if before and before[-1][0].startswith("s_") and "m0" in before[-1][1:2]:
                found.append(f"{kernel}: m0 written right before a copy")
            base, waits = set().union(*(scalar_registers(t) for t in ins[1:])), 0
            for b in reversed(before):
                if waits >= VALU_SGPR_TO_VMEM:
                    break
                if b[0].startswith("v_") and len(b) > 1 and scalar_registers(b[1]) & base:
                    found.append(f"{kernel}: {b[0]} writes a copy's base {waits} wait states before it")
                waits += int(b[1]) + 1 if b[0] == "s_nop" else 1
        before = (before + [ins])[-8:]
    return copies, found


def test_the_check_sees_a_missing_wait():
    bad = "<k>:\n\ts_mov_b32 m0, s4\n\tglobal_load_lds_dwordx4 v[2:3], off\n"
    good = "<k>:\n\ts_mov_b32 m0, s4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v[2:3], off\n"
    base = "<k>:\n\tv_readfirstlane_b32 s6, v1\n\ts_mov_b32 m0, s4\n\ts_nop 0\n\tglobal_load_lds_dword v2, s[6:7]\n"
    assert hazards(bad)[0] == 1 and len(hazards(bad)[1]) == 1
    assert hazards(good) == (1, [])
    assert len(hazards(base)[1]) == 1


def test_every_copy_into_lds_waits_for_m0(tmp_path):
    lib = shutil.copy(L.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    images = glob.glob(str(tmp_path / "*gfx950*"))
    assert images
    copies = 0
    for image in images:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", image],
                              check=True, capture_output=True, text=True).stdout
        n, found = hazards(text)
        copies += n
        assert not found, found[:3]
    assert copies > 100          # the GEMM and attention kernels are there
