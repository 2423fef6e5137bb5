"""What the kernels' sources have to keep to, seen without a GPU."""
import os
import re

import pytest

from paper_2212_05231_amd import build as b

FILES = sorted(f for f in os.listdir(b.CSRC) if f.endswith((".hip", ".h")))


def test_asm_statements_hold_no_instruction():
    """The compiler puts the wait states that a matrix instruction needs in front of its own instructions only: one written in
    asm text may be given a register that the matrix instruction is still to write, among them those of a result that nobody
    reads.  So an asm statement is an empty barrier to the optimiser, in every kernel, whatever registers it is given."""
    found = 0
    for name in FILES:
        with open(os.path.join(b.CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for statement in re.finditer(r"\b(?:asm|__asm__)\s*(?:volatile\s*)?\(\s*(\"(?:[^\"\\]|\\.)*\")", text):
            found += 1
            line = text[:statement.start()].count("\n") + 1
            assert statement.group(1) == '""', f"{name}:{line}: asm text {statement.group(1)}"
        assert len(re.findall(r"\b(?:asm|__asm__)\b", text)) == len(re.findall(r"\b(?:asm|__asm__)\s*(?:volatile\s*)?\(\s*\"", text)), name
    assert found > 0


def kernels_of(library):
    """name -> what the compiler noted of every kernel of a library built here (the metadata notes of its gfx950 code object)."""
    import struct
    msgpack = pytest.importorskip("msgpack")
    with open(library, "rb") as f:
        data = f.read()
    kernels, magic = {}, b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            if "gfx950" not in target or size == 0:
                continue
            elf = data[at + offset:at + offset + size]
            table, = struct.unpack_from("<Q", elf, 0x28)
            width, sections = struct.unpack_from("<HH", elf, 0x3a)
            for k in range(sections):
                kind, _, _, start, length_ = struct.unpack_from("<IQQQQ", elf, table + k * width + 4)
                if kind != 7:                                   # notes
                    continue
                name_size, note_size, note_type = struct.unpack_from("<III", elf, start)
                if note_type == 32:                             # the metadata, as a message pack
                    first = start + 12 + (name_size + 3) // 4 * 4
                    for kernel in msgpack.unpackb(elf[first:first + note_size])["amdhsa.kernels"]:
                        kernels[kernel[".name"]] = kernel
        at = data.find(magic, at + 1)
    return kernels


def test_no_kernel_keeps_registers_in_memory():
    """A register spilled inside a tile loop is stored and fetched for every tile.  Only the SDF backward kernel without given
    masks, which carries both orders of a tile in one wavefront, keeps some loop-invariant ones in memory."""
    kernels = kernels_of(b.LIB)
    assert len(kernels) > 30
    spilled = {name: k[".vgpr_spill_count"] for name, k in kernels.items() if k[".vgpr_spill_count"] > 0}
    allowed = {"sdf_bwd_kernelILi32ELi3EE": 18}
    for name, count in spilled.items():
        assert any(part in name and count <= most for part, most in allowed.items()), (name, count)
