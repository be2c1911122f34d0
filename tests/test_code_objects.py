"""The built library's gfx950 code: no 64-bit shift takes its amount from the last
vector register allocated to the wavefront (allocated in eights).  Such a shift
has given wrong sums on the GPU when another workgroup shared the compute unit."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

import paper_2608_07971_amd as esp

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
SHIFT = re.compile(r"\bv_(?:lshlrev|lshrrev|ashrrev)_[bi]64(?:_e64)? v\[\d+:\d+\], v(\d+),")


def _code_objects(path):
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        q = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, q)
        q += 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, q)
            name = data[q + 24:q + 24 + n].decode()
            q += 24 + n
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _offending(code, registers):
    """(kernel, instruction) of the shifts; `registers`: kernel -> VGPR count."""
    found, kernel, last, seen = [], None, -1, 0
    for line in code.splitlines():
        m = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if m:
            kernel = m.group(1)
            last = (registers.get(kernel, 0) + 7) // 8 * 8 - 1
            continue
        m = SHIFT.search(line)
        if m:
            seen += 1
            if int(m.group(1)) == last:
                found.append((kernel, line.strip()))
    return found, seen


def test_the_scan_finds_a_shift_by_the_last_register():
    code = "0000 <k>:\n\tv_lshlrev_b64 v[50:51], v71, v[2:3]\n\tv_lshrrev_b64 v[50:51], v70, v[2:3]\n"
    assert _offending(code, {"k": 72}) == ([("k", "v_lshlrev_b64 v[50:51], v71, v[2:3]")], 2)
    assert _offending(code, {"k": 73})[0] == []


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")), reason="needs ROCm's llvm-objdump")
def test_no_64_bit_shift_by_the_last_register():
    total = kernels = 0
    with tempfile.TemporaryDirectory() as tmp:
        for i, blob in enumerate(_code_objects(esp.LIB_PATH)):
            f = os.path.join(tmp, f"{i}.o")
            with open(f, "wb") as out:
                out.write(blob)
            notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f], capture_output=True, text=True,
                                   check=True).stdout
            registers = {}
            for block in notes.split("- .agpr_count")[1:]:
                name, count = (re.search(rf"\.{key}:\s+(\S+)", block).group(1) for key in ("name", "vgpr_count"))
                registers[name] = int(count)
            code = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", f],
                                  capture_output=True, text=True, check=True).stdout
            found, seen = _offending(code, registers)
            assert not found
            total += seen
            kernels += len(registers)
    assert kernels > 300 and total > 1000
