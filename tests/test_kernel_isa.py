"""Rules of the gfx9 ISA that the assembler does not enforce inside inline asm,
checked on the instructions of the library built here (no GPU needed)."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2607_00501_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
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


def _gemm_instructions(tmp_path):
    """The instructions of the built GEMM kernels, one stripped line each."""
    if not os.path.exists(B.LIB_PATH) or shutil.which(OBJDUMP) is None:
        pytest.skip("library or llvm-objdump not there")
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    for i, co in enumerate(_code_objects(data)):
        if b"qgemm_kernel" not in co:
            continue
        path = tmp_path / f"{i}.co"
        path.write_bytes(co)
        with subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                              stdout=subprocess.PIPE, text=True) as p:
            yield from (line.strip() for line in p.stdout)
        assert p.returncode == 0


def test_lds_dma_waits_for_m0(tmp_path):
    """One wait state stands between a scalar write of M0 and the LDS DMA that
    reads it."""
    dma, before = 0, ""
    for ins in _gemm_instructions(tmp_path):
        if ins.startswith("global_load_lds"):
            dma += 1
            assert not (before.startswith("s_") and " m0," in before), f"{before} | {ins}"
        before = ins
    assert dma > 0


def test_lds_dma_waits_for_fragment_reads(tmp_path):
    """No LDS DMA is issued while an LDS read of the step before is pending (it
    may overwrite the stage that the read comes from).  Checked on the kernels of
    one wavefront per K slice, whose K steps read nothing but activation
    fragments from LDS and have no barrier."""
    dma, pending, kernel, one_wave = 0, None, "", False
    for ins in _gemm_instructions(tmp_path):
        if ins.endswith(">:"):
            kernel, pending, one_wave = ins, None, re.search(r"qgemm_kernelILi\d+ELi1E", ins) is not None
        elif not one_wave:
            continue
        elif ins.startswith("ds_read"):
            pending = ins
        elif ins.startswith("s_waitcnt") and "lgkmcnt(0)" in ins:
            pending = None
        elif ins.startswith("global_load_lds"):
            dma += 1
            assert pending is None, f"{kernel} {pending} | {ins}"
    assert dma > 0


def test_matrix_and_attention_kernels_do_not_spill(tmp_path):
    """No GEMM, few-row, expert or attention kernel keeps registers in scratch
    memory (its loads would also count in the waits for the LDS DMA)."""
    if not os.path.exists(B.LIB_PATH) or shutil.which(READELF) is None:
        pytest.skip("library or llvm-readelf not there")
    with open(B.LIB_PATH, "rb") as f:
        data = f.read()
    sizes = {}
    for i, co in enumerate(_code_objects(data)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"^ +\.symbol: +(\S+)\.kd$", notes, re.M)
        scratch = re.findall(r"\.private_segment_fixed_size: (\d+)", notes)
        assert len(names) == len(scratch)
        sizes.update((n, int(c)) for n, c in zip(names, scratch) if re.search("qgemm|fewrow|attn", n))
    assert len(sizes) > 100 and not [n for n, s in sizes.items() if s]
