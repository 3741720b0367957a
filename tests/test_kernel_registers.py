"""Registers that the kernels keep in memory, from the metadata of the built library: a key loop that spills runs at half its speed.  No GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2605_03644_amd import build as hip_build

LLVM = os.path.join(os.path.dirname(os.path.realpath(hip_build.hipcc())), "..", "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _tool(name):
    for d in (LLVM, "/opt/rocm/llvm/bin"):
        if os.path.exists(os.path.join(d, name)):
            return os.path.join(d, name)
    pytest.skip(name + " is not here")


def _spills(tmp_path):
    """{kernel: (registers spilled, bytes of scratch per lane)}"""
    fat = str(tmp_path / "fat")
    subprocess.run([_tool("llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, hip_build.LIB, str(tmp_path / "copy")], check=True)
    data, found = open(fat, "rb").read(), {}
    for m in re.finditer(MAGIC, data):
        n, at = struct.unpack_from("<Q", data, m.start() + len(MAGIC))[0], m.start() + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in triple or size == 0:
                continue
            elf = tmp_path / "code"
            elf.write_bytes(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([_tool("llvm-readelf"), "--notes", str(elf)], check=True, capture_output=True, text=True).stdout
            for part in notes.split("  - .agpr_count:")[1:]:
                name = re.search(r"^    \.name:\s+(\S+)", part, re.M).group(1)
                found[name] = tuple(int(re.search(r"\." + key + r":\s+(\d+)", part).group(1))
                                    for key in ("vgpr_spill_count", "private_segment_fixed_size"))
    return found


def test_no_kernel_keeps_more_than_a_few_registers_in_memory(tmp_path):
    spills = _spills(tmp_path)
    assert sum("attn_stream_kernel" in k for k in spills) >= 30 and any("attn_mfma_kernel" in k for k in spills)
    assert {k: v for k, v in spills.items() if v[0] > 24 or v[1] > 100} == {}  # (the widest head spills a few, outside its loop)
