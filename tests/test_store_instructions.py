"""The device code that was built: no store of more than 8 bytes has a scalar offset. Such a store still
reads its data registers in the cycle after it was issued, and the compiler keeps the next instruction
from overwriting them only where there is no scalar offset: with one, the first word of a store came out
as another's now and then, too rarely for a test of results to rely on."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2505_11329_amd as tw

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def gfx950_code_objects():
    """The gfx950 code objects of libtw.so, one per source file: its offload bundles list (offset, size, target)."""
    data = open(tw.library_path(), "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + name_len].decode()
            pos += 24 + name_len
            if "gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def objdump():
    for path in (shutil.which("llvm-objdump"), "/opt/rocm/llvm/bin/llvm-objdump"):
        if path and os.path.exists(path):
            return path
    pytest.skip("no llvm-objdump")


# one operand after the descriptor: the scalar offset, 0 where there is none
WIDE_STORE = re.compile(r"\bbuffer_store_(?:dwordx[34]|b96|b128|format_d16_xyzw|format_xyzw?)\s+(.*)")


def scalar_offset(operands):
    ops = [o.strip() for o in operands.split("//")[0].split(",")]
    i = next(k for k, o in enumerate(ops) if re.match(r"s\[\d+:\d+\]", o))
    return ops[i + 1].split()[0]


def test_no_wide_store_has_a_scalar_offset(tmp_path):
    lib, wide = tw.lib(), 0
    assert lib is not None
    assert scalar_offset("v[8:11], v0, s[4:7], s9 offen sc1") == "s9"
    assert scalar_offset("v[8:11], v0, s[4:7], 0 offen offset:16  // 0000: E07C") == "0"
    objects = list(gfx950_code_objects())
    assert len(objects) >= 4
    for i, code in enumerate(objects):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(code)
        p = subprocess.Popen([objdump(), "-d", "--mcpu=gfx950", str(path)], stdout=subprocess.PIPE, text=True)
        for line in p.stdout:
            m = WIDE_STORE.search(line)
            if m:
                wide += 1
                assert scalar_offset(m.group(1)) == "0", line
        assert p.wait() == 0
    assert wide > 500      # the kernels' own stores were seen
