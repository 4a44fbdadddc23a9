"""Wait states in front of matrix instructions, in the library as it is built.  A matrix instruction must not issue within two wait states of
a vector instruction that wrote one of its operands; nothing in the hardware holds it back.  The compiler counts for what it writes
itself but does not look into inline assembly, so an exchange of registers written that way has to bring its own wait.  Read from the
disassembly of every kernel, in the order of the instructions."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2605_17415_amd", "libivftq.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
WAIT = 2


def device_code(path):
    """The gfx950 code objects of a library: every translation unit has left a bundle of (host, device)."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        entry = at + len(MAGIC) + 8
        for _ in range(count if count < 16 else 0):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + name]:
                yield data[at + offset:at + offset + size]
            entry += 24 + name
        at = data.find(MAGIC, at + len(MAGIC))


def registers(operand):
    m = re.match(r"v(?:(\d+)$|\[(\d+):(\d+)\]$)", operand)
    if not m:
        return range(0)
    return range(int(m[1]), int(m[1]) + 1) if m[1] else range(int(m[2]), int(m[3]) + 1)


def too_early(lines):
    """(kernel, writer, matrix instruction) of every matrix instruction with fewer than WAIT states between"""
    kernel, recent, found = "", [], []            # recent: (states since, instruction), at most WAIT of them
    for line in lines:
        if line[:1] == "<":
            kernel, recent = line.strip(), []
            continue
        text = line.split("//")[0].strip()
        if not text:
            continue
        op, _, rest = text.partition(" ")
        if op.startswith("v_mfma") and recent:
            operands = [a.strip() for a in rest.split(",")]
            read = {r for a in operands[1:4] for r in registers(a)}
            for _, w in recent:
                w_op, _, w_rest = w.partition(" ")
                written = [a.strip() for a in w_rest.split(",")][:2 if "swap" in w_op else 1]
                if any(r in read for a in written for r in registers(a)):
                    found.append((kernel, w, text))
        passed = int(rest.split()[0], 0) + 1 if op == "s_nop" else 1
        recent = [(n + passed, w) for n, w in recent if n + passed < WAIT]
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readlane", "v_readfirstlane")):
            recent.append((0, text))
    return found


def test_the_check_itself():
    swap, one, product = "v_swap_b32_e32 v3, v4", "s_mov_b32 s0, 0", "v_mfma_f32_16x16x32_f16 v[8:11], v[12:15], v[0:3], 0"
    assert too_early(["<k>:", swap, product]) and too_early(["<k>:", swap, one, product]) and too_early(["<k>:", swap, "s_nop 0", product])
    assert not too_early(["<k>:", swap, one, one, product]) and not too_early(["<k>:", swap, "s_nop 1", product])
    assert too_early(["<k>:", "v_mov_b32_e32 v15, v20", product]) and not too_early(["<k>:", "v_mov_b32_e32 v4, v20", product])


@pytest.mark.skipif(OBJDUMP is None, reason="llvm-objdump not available")
def test_operands_of_matrix_instructions_are_there(tmp_path):
    if not os.path.exists(LIB):
        from paper_2605_17415_amd import build
        build.build_library(verbose=False)
    units = list(device_code(LIB))
    assert len(units) >= 8, "the library holds a bundle for every source file"
    products = 0
    for i, code in enumerate(units):
        unit = tmp_path / f"unit{i}.o"
        unit.write_bytes(code)
        run = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(unit)], capture_output=True, text=True)
        assert run.returncode == 0, run.stderr
        lines = run.stdout.splitlines()
        products += sum("v_mfma" in line for line in lines)
        found = too_early(lines)
        assert not found, f"{len(found)} operands read too early, the first: {found[:3]}"
    assert products > 1000
