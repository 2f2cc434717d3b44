"""The gfx950 instructions of the built library (its own sources, compiled here) around LDS-DMA transfers.

The transfers that stand in inline assembly are invisible to the compiler's own hazard handling, so what gfx950 asks for
before them is checked on what was built: one wait state between a scalar write of M0 and the transfer that takes its LDS
address from it, and five between a vector instruction that writes a scalar register and a transfer that takes its address
from that register.

Likewise for matrix instructions: two wait states after a vector instruction that writes one of their operands.  The compiler keeps them
for the instructions it emits itself, not for those of inline assembly.
"""
import os
import re
import shutil
import subprocess

import pytest

import paper_2506_23025_amd as tl

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
TRANSFER = re.compile(r"^(global|buffer)_load_lds_|^buffer_load_.* lds\b")


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def hazards(lines):
    """(kernel, instruction, what it follows too closely) of every unguarded transfer in a listing, and the number of transfers."""
    kernel, before, found, count = None, [], [], 0
    for line in lines:
        m = re.match(r"^[0-9a-f]+ <(.+)>:", line)
        if m:
            kernel, before = m[1], []
            continue
        text = line.split("//")[0].strip()
        if not text or not re.match(r"^[a-z]", text):
            continue
        name, _, rest = text.partition(" ")
        operands = [o.strip() for o in rest.replace(" off", ",off").split(",") if o.strip()]
        if TRANSFER.match(text):
            count += 1
            reads = set().union(*(scalar_registers(o) for o in operands))
            states = 0                                     # wait states between the earlier instruction and this one
            for name0, ops0 in reversed(before):
                if states >= 5:
                    break
                if states < 1 and name0.startswith("s_") and ops0 and ops0[0] == "m0":
                    found.append((kernel, text, f"{name0} {', '.join(ops0)}"))
                if name0.startswith("v_") and any(scalar_registers(o) & reads for o in ops0[:2 if "_co_" in name0 else 1]):
                    found.append((kernel, text, f"{name0} {', '.join(ops0)}"))
                states += int(ops0[0], 0) + 1 if name0 == "s_nop" else 1
        before = (before + [(name, operands)])[-8:]
    return found, count


def test_the_check_sees_unguarded_transfers():
    listing = """
0000000000001000 <k>:
	s_mov_b32 m0, s4   // 0
	global_load_lds_dwordx4 v1, s[2:3]  // 1
	s_mov_b32 m0, s4   // 2
	s_nop 0
	global_load_lds_dwordx4 v1, s[2:3]
	v_readfirstlane_b32 s3, v0
	s_mov_b32 m0, s4
	s_nop 2
	global_load_lds_dword v1, s[2:3] offset:16
	v_readfirstlane_b32 s3, v0
	s_mov_b32 m0, s4
	s_nop 3
	global_load_lds_ushort v1, s[2:3]
"""
    found, count = hazards(listing.splitlines())
    assert count == 4
    assert [f[2].split()[0] for f in found] == ["s_mov_b32", "v_readfirstlane_b32"]


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_transfers_wait_for_their_scalar_operands(tmp_path):
    lib = str(tmp_path / "lib.so")
    shutil.copy(tl.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(f for f in os.listdir(tmp_path) if "gfx950" in f)
    assert objects, "no code objects found"
    total = 0
    for f in objects:
        text = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        found, count = hazards(text.splitlines())
        total += count
        assert not found, f"{len(found)} of {count} transfers unguarded, first: {found[0]}"
    assert total > 0, "no transfer in the library"


def vector_registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m[1])} if m else set()


def matrix_hazards(lines):
    """(kernel, instruction, what it follows too closely) of every matrix instruction that reads a vector register too early, and their number."""
    kernel, before, found, count = None, [], [], 0
    for line in lines:
        m = re.match(r"^[0-9a-f]+ <(.+)>:", line)
        if m:
            kernel, before = m[1], []
            continue
        text = line.split("//")[0].strip()
        if not text or not re.match(r"^[a-z]", text):
            continue
        name, _, rest = text.partition(" ")
        operands = [o.split()[0] for o in rest.split(",") if o.strip()]
        if name.startswith("v_mfma"):
            count += 1
            reads = set().union(*(vector_registers(o) for o in operands[1:4]))
            states = 0
            for name0, ops0 in reversed(before):
                if states >= 2:
                    break
                if name0.startswith("v_") and not name0.startswith("v_mfma") and ops0 and vector_registers(ops0[0]) & reads:
                    found.append((kernel, text, f"{name0} {', '.join(ops0)}"))
                states += int(ops0[0], 0) + 1 if name0 == "s_nop" else 1
        before = [] if name in ("s_branch", "s_endpgm") else (before + [(name, operands)])[-4:]
    return found, count


def test_the_check_sees_matrix_operands_written_too_late():
    listing = """
0000000000001000 <k>:
	v_and_b32_e32 v4, s0, v4   // 0
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[0:3]
	v_and_b32_e32 v6, s0, v6
	s_nop 0
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[0:3]
	v_and_b32_e32 v6, s0, v6
	s_nop 1
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], 0
	v_and_b32_e32 v12, s0, v6
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], 0
	v_perm_b32 v9, v1, v2, s3
	v_mov_b32_e32 v12, 0
	s_waitcnt lgkmcnt(0)
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], 0
"""
    found, count = matrix_hazards(listing.splitlines())
    assert count == 5
    assert [f[2].split()[1] for f in found] == ["v4,", "v6,"]


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_matrix_instructions_wait_for_their_operands(tmp_path):
    lib = str(tmp_path / "lib.so")
    shutil.copy(tl.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for f in sorted(f for f in os.listdir(tmp_path) if "gfx950" in f):
        text = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        found, count = matrix_hazards(text.splitlines())
        total += count
        assert not found, f"{len(found)} of {count} matrix instructions read an operand too early, first: {found[0]}"
    assert total > 0, "no matrix instruction in the library"


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_operands_of_a_pass_are_built_in_one_place(tmp_path):
    # the streaming kernel of several passes, items of one tile: three copies of an item, 16 products each, and 16 for the sums over x.  Built in two places
    # (32), the operands were copied from one to the other in every pass
    lib = str(tmp_path / "lib.so")
    shutil.copy(tl.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    counts = {}
    for f in sorted(f for f in os.listdir(tmp_path) if "gfx950" in f):
        kernel = None
        for line in subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout.splitlines():
            m = re.match(r"^[0-9a-f]+ <(.+)>:", line)
            if m:
                kernel = m[1] if re.search(r"gemv_lean_kernelILi1ELb1ELi(0|256)E", m[1]) else None
                if kernel:
                    counts[kernel] = 0
            elif kernel and "v_mfma" in line:
                counts[kernel] += 1
    assert len(counts) >= 8 and set(counts.values()) == {64}, counts
