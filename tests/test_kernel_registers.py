"""The attention kernels keep what their loops need in registers: spills of the built library, from the metadata of its code object.

A reload from scratch memory waits for every load issued before it, so a spill around the tiles costs far more than its instructions.
The limits are what the kernels stood at when the times beside them were measured; the instance that launches with a work list use for
heads of 64 on the fp8 pool lost 7 % of a step at 31."""
import os
import re
import shutil
import struct
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_00023_amd", "libprefixattn.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
LIST, WIDE, NARROW = 0, 1, 2          # launches with a work list; without one, of wide tiles; of narrow tiles only
MOST = {LIST: 10, WIDE: 25, NARROW: 4}


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{(head dimension, fp8 pool, form): vector registers spilled}"""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    data = open(LIB, "rb").read()
    found = {}
    for m in re.finditer(re.escape(MAGIC), data):
        at = m.start()
        (n,), pos = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            code = data[at + off:at + off + size]
            if b"gfx950" not in name or b"extend_bf16_kernel" not in code:
                continue
            path = tmp_path_factory.mktemp("code") / "kernels.elf"
            path.write_bytes(code)
            notes = subprocess.check_output([READELF, "--notes", str(path)], text=True)
            for k in notes.split("- .agpr_count:")[1:]:
                name = re.search(r"\.name:\s+_ZN2pa18extend_bf16_kernelILi(\d+)ELb(\d)ELi(\d)", k)
                if name:
                    found[int(name[1]), name[2] == "1", int(name[3])] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", k)[1])
    return found


@pytest.mark.parametrize("form", [LIST, WIDE, NARROW])
@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_attention_kernels_hardly_spill(spills, D, kv8, form):
    assert spills[D, kv8, form] <= MOST[form]
