"""Rules of the gfx9 ISA that the assembler does not enforce inside inline asm,
checked on the instructions of the library built here (no GPU needed)."""

import os
import shutil
import struct
import subprocess

import pytest

from paper_2607_00501_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 code objects of the library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + n]
            p += 24 + n
            if size and b"gfx950" in triple:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def test_lds_dma_waits_for_m0(tmp_path):
    """One wait state stands between a scalar write of M0 and the LDS DMA that
    reads it."""
    if not os.path.exists(B.LIB_PATH) or shutil.which(OBJDUMP) is None:
        pytest.skip("library or llvm-objdump not there")
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    dma = 0
    for i, co in enumerate(_code_objects(data)):
        if b"qgemm_kernel" not in co:
            continue
        path = tmp_path / f"{i}.co"
        path.write_bytes(co)
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                              stdout=subprocess.PIPE, text=True) as p:
            before = ""
            for line in p.stdout:
                ins = line.strip()
                if ins.startswith("global_load_lds"):
                    dma += 1
                    assert not (before.startswith("s_") and " m0," in before), f"{before} | {ins}"
                before = ins
        assert p.returncode == 0
    assert dma > 0
