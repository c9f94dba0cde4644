"""Where lanes that a branch had switched off meet the others again, nothing may be computed for all lanes before they are switched on:
the compiler once put copies of registers there that live on, and lanes of rows outside the problem, or all lanes after them, worked with
what a register held before.  Looks for that in the kernels of the built library."""
import os
import re
import struct
import subprocess

import pytest

from test_kernel_resources import LIB

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
VECTOR = re.compile(r"v_(?!writelane|readlane|readfirstlane)|global_|ds_|buffer_|scratch_|flat_")


def code_objects():
    data = open(LIB, "rb").read()
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        count, = struct.unpack_from("<Q", data, m.start() + 24)
        pos = m.start() + 32
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + idlen] and size:
                yield data[m.start() + off:m.start() + off + size]
            pos += 24 + idlen


def suspects(listing):
    """(kernel, instructions) between a branch target that lanes skip to and the instruction that switches them on."""
    joins = set(re.findall(r"s_cbranch_execz .*<(\S+\+0x[0-9a-f]+)>", listing, re.IGNORECASE))
    kernel, start, pending = None, 0, None
    for line in listing.split("\n"):
        head = re.match(r"([0-9a-f]+) <(\S+)>:$", line)
        if head:
            start, kernel, pending = int(head.group(1), 16), head.group(2), None
            continue
        m = re.match(r"\t(\S+)(.*?)// ([0-9A-F]+):", line)
        if not m:
            continue
        op, operands, at = m.group(1), m.group(2), int(m.group(3), 16)
        if f"{kernel}+0x{at - start:x}" in joins:
            pending = []
        if pending is None:
            continue
        if op == "s_or_b64" and operands.split()[0] == "exec,":
            if pending:
                yield kernel, pending
            pending = None
        elif op.startswith(("s_cbranch", "s_branch", "s_endpgm")) or "exec" in op + operands:
            pending = None
        elif VECTOR.match(op):
            pending.append(f"{op} {operands.strip()}")


def test_nothing_is_computed_before_lanes_are_switched_on(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    listings = 0
    for i, image in enumerate(code_objects()):
        path = tmp_path / f"{i}.o"
        path.write_bytes(image)
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], check=True, capture_output=True, text=True).stdout
        listings += "s_cbranch_execz" in listing
        assert list(suspects(listing)) == []
    assert listings > 5
