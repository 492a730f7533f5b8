"""The device code of the built library, read back as AMD assembly: what the compiler does not see to itself on gfx950."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2006_02230_amd as P

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/lib/llvm/bin/llvm-objdump", shutil.which("llvm-objdump"))
                if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 ELF images inside a library's offload bundles."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        count, pos = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + n].decode()
            pos += 24 + n
            if size and "gfx950" in triple:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, pos)


SHIFT = re.compile(r"\bv_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)(?:_e64)? v\[\d+:\d+\], v(\d+),")


def hazards(lines):
    """(kernel, instruction) of every 64-bit shift whose amount is the last register of a block of eight."""
    kernel, out = None, []
    for l in lines:
        m = re.match(r"[0-9a-f]+ <(\w+)>:", l)
        if m:
            kernel = m.group(1)
            continue
        m = SHIFT.search(l)
        if m and int(m.group(1)) % 8 == 7:
            out.append((kernel, l.split("//")[0].strip()))
    return out


def test_hazards_are_recognised():
    text = ["0000000000001900 <k>:", "\tv_lshrrev_b64 v[4:5], v70, v[2:3]  // 00", "\tv_lshrrev_b64 v[4:5], s7, v[2:3]  // 00",
            "\tv_lshlrev_b64 v[4:5], 7, v[2:3]  // 00", "\tv_lshrrev_b32_e32 v4, v71, v2  // 00", "\tv_lshrrev_b64 v[4:5], v71, v[2:3]  // 00"]
    assert hazards(text) == [("k", "v_lshrrev_b64 v[4:5], v71, v[2:3]")]


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_no_64bit_shift_by_a_register_that_can_be_the_last(tmp_path):
    # Registers are allocated in blocks of eight.  On gfx950 a per-lane 64-bit shift whose amount lies in the last register of the
    # allocation uses another wave's value now and then (measured: a quarter of such shifts wrong on a full card, none with the
    # amount one register lower or with one block more); the compiler avoids that on gfx90a only.  Whether register 8 n + 7
    # is the last one depends on everything else in a kernel, so no such shift may use one.
    found, kernels = [], 0
    for i, elf in enumerate(code_objects(P.LIB_PATH)):
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(elf)
        lines = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout.splitlines()
        kernels += sum(l.endswith(">:") for l in lines)
        found += hazards(lines)
    assert kernels > 300          # the library was read
    assert not found, "%d, first: %s" % (len(found), found[0])
